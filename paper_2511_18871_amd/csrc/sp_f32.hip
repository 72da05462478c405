// float32 path of shared-prompt attention, the segment-table upload
// and the backward preprocess D = rowsum(dO * O).
//
// These kernels give the eight wavefronts of a workgroup a single (row, head) or (key, kv head), or 16 of them, and walk
// the allowed keys / rows of the Section 4.3 mask in chunks, in float32 throughout: they exist to cross-check the bf16 path and to serve float32 callers.
#include "sp_common.hpp"
#include "sp_launch.hpp"
#include <algorithm>
#include <type_traits>

namespace sp {
namespace {

__device__ __forceinline__ float wave_max(float x) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x = fmaxf(x, __shfl_xor(x, o, 64));
    return x;
}
__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) x += __shfl_xor(x, o, 64);
    return x;
}

__global__ void upload_table_kernel(TabChunk chunk, int* __restrict__ dst, int offset, int count) {
    for (int i = threadIdx.x; i < count; i += blockDim.x) dst[offset + i] = chunk.w[i];
}

// One thread per packed token writes its segment bounds, one per work tile its descriptor (see Schedule).
__device__ __forceinline__ void schedule_body(const int* __restrict__ tab, int n_groups, int64_t T_total, int n256,
                                              int n128, TileDesc* __restrict__ tiles256, TileDesc* __restrict__ tiles128,
                                              TileDesc* __restrict__ key_tiles, int* __restrict__ key_lo,
                                              int* __restrict__ row_hi, int key_order) {
    const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
    if (i < T_total) {
        const GroupDesc gd = load_group(tab, find_group_of_token(tab, i));
        const int t = (int)(i - gd.tok_base);
        int lo = 0, hi = gd.Tg;
        if (t >= gd.Lp) {
            const int tq[1] = {t};
            int sq[1], eq[1];
            seg_bounds<1>(gd, tq, sq, eq);
            lo = sq[0]; hi = eq[0];
        }
        key_lo[i] = lo;
        row_hi[i] = hi;
    }
    auto describe = [&](auto bt_tag, int n, TileDesc* out) -> TileDesc {
        constexpr int BT = decltype(bt_tag)::value;
        TileDesc td{0, 0, 0, 0, 0, 0, 0, 0};
        if (i >= n) return td;
        find_tile<BT>(tab, n_groups, (int)i, td.g, td.ti);
        if (td.g < 0) td.g = n_groups - 1;             // cannot happen: n is the exact tile count
        const GroupDesc gd = load_group(tab, td.g);
        td.tok_base = gd.tok_base; td.Lp = gd.Lp; td.Tg = gd.Tg;
        out[i] = td;
        return td;
    };
    describe(std::integral_constant<int, 256>{}, n256, tiles256);
    if ((int64_t)blockIdx.x * 256 >= n128) return;     // the whole block
    const TileDesc td = describe(std::integral_constant<int, 128>{}, n128, tiles128);
    if (key_order == KEYS_AS_PACKED) return;
    // place among the key tiles: the number of prompt tiles, and of those ahead of this block's first tile, by a strided
    // sum over the groups; within the block by a scan
    __shared__ int part[3][4], first[2];
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    const bool prompt = i < n128 && 128 * td.ti < td.Lp;
    if (threadIdx.x == 0) { first[0] = td.g; first[1] = min(td.ti, (td.Lp + 127) / 128); }
    __syncthreads();
    int before = 0, all = 0;
    for (int g = threadIdx.x; g < n_groups; g += 256) {
        const int c = (tab[TAB_HEADER + TAB_GROUP_WORDS * g + 1] + 127) / 128;
        all += c;
        before += g < first[0] ? c : 0;
    }
#pragma unroll
    for (int o = 32; o >= 1; o >>= 1) { all += __shfl_xor(all, o, 64); before += __shfl_xor(before, o, 64); }
    const uint64_t mine = __builtin_amdgcn_ballot_w64(prompt);
    if (l == 0) { part[0][w] = all; part[1][w] = before; part[2][w] = __popcll(mine); }
    __syncthreads();
    const int n_prompt = part[0][0] + part[0][1] + part[0][2] + part[0][3];
    int rank = first[1] + part[1][0] + part[1][1] + part[1][2] + part[1][3] + __popcll(mine & ((1ull << l) - 1));
    for (int v = 0; v < w; ++v) rank += part[2][v];    // prompt tiles ahead of tile i
    int at = prompt ? rank : n_prompt + (int)i - rank;
    if (prompt && key_order == KEYS_BY_ROWS) {         // prompt tiles with more rows, or as many in an earlier group
        at = 0;
        for (int g = 0; g < n_groups; ++g) {
            const int* e = tab + TAB_HEADER + TAB_GROUP_WORDS * g;
            const int more = e[2] - (td.Tg - 128 * td.ti) + (g < td.g ? 1 : 0);
            at += min((e[1] + 127) / 128, max(0, (more + 127) / 128));
        }
    }
    if (i < n128) key_tiles[at] = td;
}

__global__ __launch_bounds__(256) void schedule_kernel(const int* __restrict__ tab, int n_groups, int64_t T_total,
                                                       int n256, int n128, TileDesc* __restrict__ tiles256,
                                                       TileDesc* __restrict__ tiles128, TileDesc* __restrict__ key_tiles,
                                                       int* __restrict__ key_lo, int* __restrict__ row_hi, int key_order) {
    schedule_body(tab, n_groups, T_total, n256, n128, tiles256, tiles128, key_tiles, key_lo, row_hi, key_order);
}

__global__ __launch_bounds__(64) void reserve_tag_kernel(uint32_t* __restrict__ blk, ReserveTag want, int mode) {
    reserve_tag_body(blk, want, mode, threadIdx.x);
}

// Everything a call does ahead of its attention kernels, in one launch, for segment tables that fit one
// kernel-argument block: block 0 stores the table into the workspace and (first wave) maintains the tag
// block; every block works out its part of the schedule from a copy of the table in its own LDS, since the
// copy in memory is only complete when the kernel has ended.  Small problems, whose attention kernels run
// for tens of microseconds, otherwise spend a fifth of a call in three tiny launches and the gaps between them.
__global__ __launch_bounds__(256) void prepare_kernel(PrepChunk chunk, int n_words, int* __restrict__ dev_tab,
                                                      uint32_t* __restrict__ tag_blk, ReserveTag want, int tag_mode,
                                                      int with_schedule, int n_groups, int64_t T_total, int n256,
                                                      int n128, TileDesc* __restrict__ tiles256,
                                                      TileDesc* __restrict__ tiles128, TileDesc* __restrict__ key_tiles,
                                                      int* __restrict__ key_lo, int* __restrict__ row_hi, int key_order) {
    __shared__ int tab_s[PREP_WORDS];
    for (int i = threadIdx.x; i < n_words; i += 256) {
        const int x = chunk.w[i];
        tab_s[i] = x;
        if (blockIdx.x == 0) dev_tab[i] = x;
    }
    if (blockIdx.x == 0 && threadIdx.x < 64 && tag_mode != TAG_KEEP) reserve_tag_body(tag_blk, want, tag_mode, threadIdx.x);
    __syncthreads();
    if (with_schedule) schedule_body(tab_s, n_groups, T_total, n256, n128, tiles256, tiles128, key_tiles, key_lo, row_hi, key_order);
}

template <typename T>
__global__ __launch_bounds__(256) void rowsum_kernel(const T* __restrict__ d_o, const T* __restrict__ o,
                                                     const float* __restrict__ lse, float* __restrict__ D,
                                                     int64_t T_total, int Hq, int dh,
                                                     const int* __restrict__ tab, int resp_only,
                                                     const T* __restrict__ o_lo) {
    constexpr bool BF = std::is_same<T, __bf16>::value;        // the bf16 planes hold -D and lse * log2(e)
    const int64_t gw = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int l = threadIdx.x & 63;
    if (gw >= T_total * Hq) return;
    const int64_t tok = gw / Hq;
    const int h = (int)(gw % Hq);
    if (resp_only) {
        // prompt rows take no part: their o / lse may hold anything, so they are not read, and the
        // planes get finite placeholders (rows of a partly used tile are masked, not skipped)
        const GroupDesc gd = load_group(tab, find_group_of_token(tab, (int)tok));
        if ((int)tok - gd.tok_base < gd.Lp) {
            if (l == 0) {
                D[(int64_t)h * T_total + tok] = 0.f;
                D[(int64_t)Hq * T_total + (int64_t)h * T_total + tok] = 0.f;
            }
            return;
        }
    }
    const T* a = d_o + gw * dh;
    const T* b = o + gw * dh;
    float acc = 0.f;
    if (o_lo) {          // o was stored with its rounding residual: D from the unrounded value
        const T* c = o_lo + gw * dh;
        for (int i = l; i < dh; i += 64) acc += (float)a[i] * ((float)b[i] + (float)c[i]);
    } else {
        for (int i = l; i < dh; i += 64) acc += (float)a[i] * (float)b[i];
    }
    acc = wave_sum(acc);
    if (l == 0) {
        D[(int64_t)h * T_total + tok] = BF ? -acc : acc;
        if (BF) D[(int64_t)Hq * T_total + (int64_t)h * T_total + tok] = lse[(int64_t)h * T_total + tok] * LOG2E;
    }
}

// The same rowsum for bf16 rows of 128 elements, laid out for bandwidth.  A block owns RS_TOK
// consecutive tokens x all q heads, which is one contiguous stretch of d_o and of o; 16 lanes read
// a (token, head) row as 16-byte pieces and add up over the lanes.  The sums pass through LDS so
// that each head's RS_TOK tokens leave as one contiguous store into the [Hq, T] planes.  In
// response-rows mode the prompt rows are still read (the buffers are whole) but their values are
// discarded by a select, never used in arithmetic that reaches the output.
constexpr int RS_TOK = 16;      // rowsum_fast_path() in sp_launch.hpp assumes this value
template <bool HAS_LO>
__global__ __launch_bounds__(256) void rowsum_bf16_kernel(const __bf16* __restrict__ d_o, const __bf16* __restrict__ o,
                                                          const float* __restrict__ lse, float* __restrict__ D,
                                                          int64_t T_total, int Hq, const int* __restrict__ tab,
                                                          int resp_only, const __bf16* __restrict__ o_lo,
                                                          const uint32_t* __restrict__ lo_flag) {
    extern __shared__ float rs_sum[];                  // [Hq][RS_TOK]
    __shared__ int rs_skip[RS_TOK];
    // the residual is the workspace's reserve: usable only if the tag check of this call said so
    const bool use_lo = HAS_LO && (lo_flag == nullptr || __builtin_amdgcn_readfirstlane((int)*lo_flag) != 0);
    const int64_t tok0 = (int64_t)blockIdx.x * RS_TOK;
    const int ntok = (int)(T_total - tok0 < RS_TOK ? T_total - tok0 : RS_TOK);
    const int tid = threadIdx.x, sub = tid & 15, grp = tid >> 4;
    if (tid < RS_TOK) {
        int sk = 0;
        if (resp_only && tid < ntok) {
            const GroupDesc gd = load_group(tab, find_group_of_token(tab, tok0 + tid));
            sk = (int)(tok0 + tid - gd.tok_base) < gd.Lp;
        }
        rs_skip[tid] = sk;
    }
    __syncthreads();
    const int nrows = ntok * Hq;
    const int64_t base = tok0 * Hq * 128 + 8 * sub;
    auto row_dot = [&](int r) -> float {
        const int64_t off = base + (int64_t)r * 128;
        const bf16x8 a = *reinterpret_cast<const bf16x8*>(d_o + off);
        const bf16x8 b = *reinterpret_cast<const bf16x8*>(o + off);
        float acc = dot8(a, b, 0.f);
        // o was stored with its rounding residual: D from the unrounded value
        if (HAS_LO && use_lo) acc = dot8(a, *reinterpret_cast<const bf16x8*>(o_lo + off), acc);
        return acc;
    };
    auto put = [&](int r, float acc) {
#pragma unroll
        for (int sh = 8; sh >= 1; sh >>= 1) acc += __shfl_xor(acc, sh, 16);
        const int tl = r / Hq, h = r - tl * Hq;
        if (sub == 0) rs_sum[h * RS_TOK + tl] = rs_skip[tl] ? 0.f : acc;
    };
    for (int r = grp; r < nrows; r += 32) {            // two rows per trip: four to six loads in flight per lane
        const bool two = r + 16 < nrows;
        const float x0 = row_dot(r), x1 = row_dot(two ? r + 16 : r);
        put(r, x0);
        if (two) put(r + 16, x1);
    }
    __syncthreads();
    for (int i = tid; i < Hq * RS_TOK; i += 256) {
        const int h = i / RS_TOK, tl = i % RS_TOK;
        if (tl < ntok) {
            const int64_t idx = (int64_t)h * T_total + tok0 + tl;
            D[idx] = -rs_sum[i];
            // second plane: the row's logsumexp in base-2 units, as the dkdv pass consumes it
            const float l2 = lse[idx] * LOG2E;
            D[(int64_t)Hq * T_total + idx] = rs_skip[tl] ? 0.f : l2;
        }
    }
}

// Few rows (keys): a workgroup of eight waves per (row, head) or (key, kv head), bound by latency: every wave takes each eighth chunk
// of 32 keys, two lanes per key, with one batch of loads for the scores and one (rows 32 at a time, lanes along a row) for
// the sums.  The waves' sums meet in LDS, in a fixed order.  (WIDE; else one wave and chunks of 64 keys, a lane per key, the wave's
// own row in scalar registers: where rows see few keys, and for single rows of the blocks below.  Which shape: f32_shape().)
// With the rowsum within the dq kernel and the table as an argument, a training pass of 64 + 4 x 32 tokens, 2 heads of 64: 54.0 ->
// 33.0 us.
constexpr int F32_WAVES = 8;
template <bool WIDE> constexpr int CHUNK = WIDE ? 32 : 64;
template <bool WIDE> constexpr int F32_BLOCK = WIDE ? 64 * F32_WAVES : 256;
// dot product of two rows in the lane, or (WIDE) half of it in each lane of the pair (l, l ^ 32)
template <int DH, bool WIDE>
__device__ __forceinline__ float dot_row(const float* __restrict__ x, const float* __restrict__ y, int l) {
    constexpr int N = WIDE ? DH / 8 : DH / 4;
    const int at = WIDE ? DH / 2 * (l >> 5) : 0;
    f32x4 v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) v[i] = *reinterpret_cast<const f32x4*>(y + at + 4 * i);
    f32x4 part = {0.f, 0.f, 0.f, 0.f};             // four short sums, as in the blocks below
    if constexpr (WIDE) {
        f32x4 u[N];
#pragma unroll
        for (int i = 0; i < N; ++i) u[i] = *reinterpret_cast<const f32x4*>(x + at + 4 * i);
        __builtin_amdgcn_sched_barrier(0);         // all loads in flight: left alone, each waited for the products of the one before
#pragma unroll
        for (int i = 0; i < 4 * N; ++i) part[i & 3] = __builtin_fmaf(u[i >> 2][i & 3], v[i >> 2][i & 3], part[i & 3]);
        return pair_sum((part[0] + part[1]) + (part[2] + part[3]));
    }
#pragma unroll
    for (int i = 0; i < 4 * N; ++i) part[i & 3] = __builtin_fmaf(x[i], v[i >> 2][i & 3], part[i & 3]);
    return (part[0] + part[1]) + (part[2] + part[3]);
}
__device__ __forceinline__ float lane_value(float x, int lane) {      // of a wave-uniform lane
    return __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(x), lane));
}
// acc[e] += sum over j < n of lane j's p * row j's element l + 64 e; p is 0 in the lanes from n on.  Row j at base + j * stride.
// The rows of a batch past n repeat row n - 1 with weight 0, which is nothing unless that row holds an
// infinity (0 * inf).  A sum that became NaN is therefore taken once more over the n rows alone, one by one; excluding the
// repeated rows with a select per row instead costs a tenth of the kernel.
template <int PER>
__device__ __forceinline__ void add_rows(float (&acc)[PER], float p, const float* __restrict__ base, int64_t stride, int n, int l) {
    constexpr int ROWS = 32;
    float start[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) start[e] = acc[e];
    for (int j0 = 0; j0 < n; j0 += ROWS) {
        float x[ROWS][PER];
#pragma unroll
        for (int u = 0; u < ROWS; ++u)
#pragma unroll
            for (int e = 0; e < PER; ++e) x[u][e] = base[min(j0 + u, n - 1) * stride + l + 64 * e];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const float pj = lane_value(p, j0 + u);
#pragma unroll
            for (int e = 0; e < PER; ++e) acc[e] = __builtin_fmaf(pj, x[u][e], acc[e]);
        }
    }
    bool is_nan = false;             // by its bits: the build takes float comparisons to see no NaN
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        asm volatile("" : "+v"(acc[e]));
        is_nan |= (__float_as_uint(acc[e]) & 0x7fffffffu) > 0x7f800000u;
    }
    if (__builtin_amdgcn_ballot_w64(is_nan)) {
#pragma unroll
        for (int e = 0; e < PER; ++e) acc[e] = start[e];
        for (int j = 0; j < n; ++j) {
            const float pj = lane_value(p, j);
#pragma unroll
            for (int e = 0; e < PER; ++e) acc[e] = __builtin_fmaf(pj, base[j * stride + l + 64 * e], acc[e]);
        }
    }
}
// The chunks of keys that row t sees: those of the prompt, then those of its response from its first token on.
template <int C>
struct KeyChunks {
    int n1, n, end1, st, end;
    __device__ __forceinline__ KeyChunks(const GroupDesc& gd, int t) {
        st = seg_start(gd, t);
        end1 = min(gd.Lp, t + 1);
        end = t + 1;
        n1 = (end1 + C - 1) / C;
        n = n1 + (t >= gd.Lp ? (end - st + C - 1) / C : 0);
    }
    __device__ __forceinline__ int first(int i) const { return i < n1 ? C * i : st + C * (i - n1); }
    __device__ __forceinline__ int count(int i) const { return min(C, (i < n1 ? end1 : end) - first(i)); }
};

// The row (key) and head of a workgroup, or of its wave w; false past the last one
template <bool WIDE>
__device__ __forceinline__ bool row_and_head(int w, int64_t T_total, int heads, int& tok, int& h) {
    if constexpr (WIDE) {
        tok = (int)(blockIdx.x / (unsigned)heads); h = (int)(blockIdx.x % (unsigned)heads);
        return true;
    }
    const int64_t item = (int64_t)blockIdx.x * 4 + w;
    tok = (int)(item / heads); h = (int)(item % heads);
    return item < T_total * heads;
}

// One row of one head: by one wave, or (WIDE) by the workgroup's eight
template <int DH, bool WIDE>
__device__ __forceinline__ void fwd_f32_row(const GroupDesc& gd, int tok, int h, int w, int l, const float* __restrict__ q, const float* __restrict__ k,
                                            const float* __restrict__ v, float* __restrict__ o, float* __restrict__ lse, int64_t T_total,
                                            int Hq, int Hkv, float scale, int resp_only) {
    constexpr int PER = DH / 64;
    __shared__ float sh_m[F32_WAVES], sh_l[F32_WAVES], sh_acc[WIDE ? F32_WAVES : 1][DH];
    const int t = tok - gd.tok_base;
    if (resp_only && t < gd.Lp) return;
    constexpr int C = CHUNK<WIDE>;
    const KeyChunks<C> ch(gd, t);
    const int kvh = h / (Hq / Hkv);
    const float* qrow = q + ((int64_t)tok * Hq + h) * DH;
    const float* kb = k + ((int64_t)gd.tok_base * Hkv + kvh) * DH;
    const float* vb = v + ((int64_t)gd.tok_base * Hkv + kvh) * DH;
    const int64_t kvs = (int64_t)Hkv * DH;

    float m = -INFINITY, lsum = 0.f, acc[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] = 0.f;
    for (int i = WIDE ? w : 0; i < ch.n; i += WIDE ? F32_WAVES : 1) {
        const int s0 = ch.first(i), nk = ch.count(i), key = l & (C - 1);
        const bool ok = key < nk;
        const float dot = dot_row<DH, WIDE>(qrow, kb + (int64_t)(s0 + min(key, nk - 1)) * kvs, l);
        const float sc = ok ? scale * dot : -INFINITY;
        const float mnew = fmaxf(m, wave_max(sc));
        // (nothing but masked keys and scores of -inf so far.  A NaN, which the maximum ignores, goes on: both sums become NaN)
        unsigned bits = __float_as_uint(sc);
        asm volatile("" : "+v"(bits));
        if (mnew == -INFINITY && !__builtin_amdgcn_ballot_w64((bits & 0x7fffffffu) > 0x7f800000u)) continue;
        const float alpha = expf(m - mnew);
        const float p = ok ? expf(sc - mnew) : 0.f;
        lsum = lsum * alpha + wave_sum(l < C ? p : 0.f);
        m = mnew;
#pragma unroll
        for (int e = 0; e < PER; ++e) acc[e] *= alpha;
        add_rows<PER>(acc, p, vb + (int64_t)s0 * kvs, kvs, nk, l);
    }
    if constexpr (!WIDE) {
        float* const orow = o + ((int64_t)tok * Hq + h) * DH;
#pragma unroll
        for (int e = 0; e < PER; ++e) orow[l + 64 * e] = acc[e] / lsum;
        if (l == 0) lse[(int64_t)h * T_total + tok] = m + logf(lsum);
        return;
    }
    if (l == 0) { sh_m[w] = m; sh_l[w] = lsum; }
#pragma unroll
    for (int e = 0; e < PER; ++e) sh_acc[w][l + 64 * e] = acc[e];
    __syncthreads();
    if ((int)threadIdx.x >= DH) return;
    float mt = sh_m[0];
#pragma unroll
    for (int i = 1; i < F32_WAVES; ++i) mt = fmaxf(mt, sh_m[i]);
    float ls = 0.f, x = 0.f;
#pragma unroll
    for (int i = 0; i < F32_WAVES; ++i) {
        if (__float_as_uint(sh_l[i]) == 0u) continue;    // a wave without a key (or with scores of -inf only)
        const float f = expf(sh_m[i] - mt);
        ls = __builtin_fmaf(sh_l[i], f, ls);
        x = __builtin_fmaf(sh_acc[i][threadIdx.x], f, x);
    }
    o[((int64_t)tok * Hq + h) * DH + threadIdx.x] = x / ls;
    if (threadIdx.x == 0) lse[(int64_t)h * T_total + tok] = mt + logf(ls);
}

template <int DH, bool WIDE>
__global__ __launch_bounds__(F32_BLOCK<WIDE>) void fwd_f32_kernel(TabArg table, const float* __restrict__ q, const float* __restrict__ k,
                                                                 const float* __restrict__ v, float* __restrict__ o,
                                                                 float* __restrict__ lse, int64_t T_total, int Hq, int Hkv,
                                                                 float scale, int resp_only) {
    const int* const tab = table_of(table);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    int tok, h;
    if (!row_and_head<WIDE>(w, T_total, Hq, tok, h)) return;
    fwd_f32_row<DH, WIDE>(load_group(tab, find_group_of_token(tab, tok)), tok, h, w, l, q, k, v, o, lse, T_total, Hq, Hkv, scale, resp_only);
}

// dQ[t,h] = scale * sum_s dS[t,s] K[s],  dS = P * (dP - D)
// `o` (a call that runs the rowsum stage too): D is formed here, with the arithmetic of rowsum_kernel, and written for the
// dkdv kernel.  `tag`: cleared (a call without a preparation launch).
template <int DH, bool WIDE>
__device__ __forceinline__ void dq_f32_row(const GroupDesc& gd, int tok, int h, int w, int l, const float* __restrict__ q, const float* __restrict__ k,
                                           const float* __restrict__ v, const float* __restrict__ d_o, const float* __restrict__ o,
                                           const float* __restrict__ lse, float* __restrict__ D, float* __restrict__ dq,
                                           int64_t T_total, int Hq, int Hkv, float scale, int resp_only) {
    constexpr int PER = DH / 64;
    __shared__ float sh_acc[WIDE ? F32_WAVES : 1][DH];
    const int t = tok - gd.tok_base;
    if (resp_only && t < gd.Lp) return;
    constexpr int C = CHUNK<WIDE>;
    const KeyChunks<C> ch(gd, t);
    const int kvh = h / (Hq / Hkv);
    const int64_t row = (int64_t)tok * Hq + h, word = (int64_t)h * T_total + tok;
    const float* kb = k + ((int64_t)gd.tok_base * Hkv + kvh) * DH;
    const float* vb = v + ((int64_t)gd.tok_base * Hkv + kvh) * DH;
    const int64_t kvs = (int64_t)Hkv * DH;
    const float L = lse[word];
    float Dt;
    if (o) {
        Dt = 0.f;
#pragma unroll
        for (int e = 0; e < PER; ++e) Dt += d_o[row * DH + l + 64 * e] * o[row * DH + l + 64 * e];
        Dt = wave_sum(Dt);
        if ((WIDE ? (int)threadIdx.x : l) == 0) D[word] = Dt;
    } else {
        Dt = D[word];
    }

    float acc[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] = 0.f;
    for (int i = WIDE ? w : 0; i < ch.n; i += WIDE ? F32_WAVES : 1) {
        const int s0 = ch.first(i), nk = ch.count(i), key = l & (C - 1);
        const int64_t at = (int64_t)(s0 + min(key, nk - 1)) * kvs;
        const float dot = dot_row<DH, WIDE>(q + row * DH, kb + at, l);
        if (WIDE) __builtin_amdgcn_sched_barrier(0);       // (a second row in flight beside these spills)
        const float dp = dot_row<DH, WIDE>(d_o + row * DH, vb + at, l);
        const float ds = key < nk ? expf(scale * dot - L) * (dp - Dt) : 0.f;
        add_rows<PER>(acc, ds, kb + (int64_t)s0 * kvs, kvs, nk, l);
    }
    if constexpr (!WIDE) {
#pragma unroll
        for (int e = 0; e < PER; ++e) dq[row * DH + l + 64 * e] = scale * acc[e];
        return;
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) sh_acc[w][l + 64 * e] = acc[e];
    __syncthreads();
    if ((int)threadIdx.x >= DH) return;
    float x = 0.f;
#pragma unroll
    for (int i = 0; i < F32_WAVES; ++i) x += sh_acc[i][threadIdx.x];
    dq[row * DH + threadIdx.x] = scale * x;
}

template <int DH, bool WIDE>
__global__ __launch_bounds__(F32_BLOCK<WIDE>, WIDE && DH == 64 ? 4 : 1) void bwd_dq_f32_kernel(TabArg table, const float* __restrict__ q, const float* __restrict__ k,
                                                                    const float* __restrict__ v, const float* __restrict__ d_o,
                                                                    const float* __restrict__ o, const float* __restrict__ lse,
                                                                    float* __restrict__ D, float* __restrict__ dq, uint32_t* __restrict__ tag,
                                                                    int64_t T_total, int Hq, int Hkv, float scale, int resp_only) {
    const int* const tab = table_of(table);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    int tok, h;
    if (!row_and_head<WIDE>(w, T_total, Hq, tok, h)) return;
    if (tag && blockIdx.x == 0 && w == 0) tag[l] = 0u;
    dq_f32_row<DH, WIDE>(load_group(tab, find_group_of_token(tab, tok)), tok, h, w, l, q, k, v, d_o, o, lse, D, dq, T_total, Hq, Hkv, scale, resp_only);
}

// dK[s,g] = scale * sum_{h in g} sum_t dS[t,s] Q[t,h];  dV[s,g] = sum_{h in g} sum_t P[t,s] dO[t,h].
// The rows that see key s are contiguous: [s, Tg) for a prompt key (later prompt rows and
// every row of every response), [s, end of its response) otherwise.
template <int DH, bool WIDE>
__device__ __forceinline__ void dkdv_f32_key(const GroupDesc& gd, int tok, int kvh, int w, int l, const float* __restrict__ q, const float* __restrict__ k,
                                             const float* __restrict__ v, const float* __restrict__ d_o, const float* __restrict__ lse,
                                             const float* __restrict__ D, float* __restrict__ dk, float* __restrict__ dv,
                                             int64_t T_total, int Hq, int Hkv, float scale, int resp_only, int accumulate) {
    constexpr int PER = DH / 64;
    __shared__ float sh_acc[2][WIDE ? F32_WAVES : 1][DH];
    constexpr int C = CHUNK<WIDE>;
    const int s = tok - gd.tok_base;
    const int row_end = s < gd.Lp ? gd.Tg : seg_end(gd, s), row_lo = resp_only ? max(s, gd.Lp) : s;
    const int rep = Hq / Hkv, n = (row_end - row_lo + C - 1) / C;
    const float* krow = k + ((int64_t)tok * Hkv + kvh) * DH;
    const float* vrow = v + ((int64_t)tok * Hkv + kvh) * DH;

    float ak[PER], av[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) { ak[e] = 0.f; av[e] = 0.f; }
    for (int hr = 0, i = WIDE ? w : 0; hr < rep; ++hr, i -= n) {      // chunk i of the n * rep, counted within the head
        for (; i < n; i += WIDE ? F32_WAVES : 1) {
            const int h = kvh * rep + hr, r0 = row_lo + C * i, nr = min(C, row_end - r0), r = l & (C - 1);
            const int64_t row0 = ((int64_t)(gd.tok_base + r0) * Hq + h) * DH, rs = (int64_t)Hq * DH;
            const int64_t at = row0 + min(r, nr - 1) * rs, word = (int64_t)h * T_total + gd.tok_base + r0 + min(r, nr - 1);
            const float L = lse[word], Dt = D[word];
            const float dot = dot_row<DH, WIDE>(krow, q + at, l);
            if (WIDE && DH == 128) __builtin_amdgcn_sched_barrier(0);
            const float dp = dot_row<DH, WIDE>(vrow, d_o + at, l);
            const float p = r < nr ? expf(scale * dot - L) : 0.f, ds = r < nr ? p * (dp - Dt) : 0.f;
            if (WIDE && DH == 128) __builtin_amdgcn_sched_barrier(0);
            add_rows<PER>(av, p, d_o + row0, rs, nr, l);
            if (WIDE && DH == 128) __builtin_amdgcn_sched_barrier(0);
            add_rows<PER>(ak, ds, q + row0, rs, nr, l);
        }
    }
    if constexpr (!WIDE) {
        float* const okr = dk + ((int64_t)tok * Hkv + kvh) * DH;
        float* const ovr = dv + ((int64_t)tok * Hkv + kvh) * DH;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            okr[l + 64 * e] = scale * ak[e] + (accumulate ? okr[l + 64 * e] : 0.f);
            ovr[l + 64 * e] = av[e] + (accumulate ? ovr[l + 64 * e] : 0.f);
        }
        return;
    }
#pragma unroll
    for (int e = 0; e < PER; ++e) { sh_acc[0][w][l + 64 * e] = ak[e]; sh_acc[1][w][l + 64 * e] = av[e]; }
    __syncthreads();
    for (int i = threadIdx.x; i < 2 * DH; i += 64 * F32_WAVES) {
        const int which = i / DH, e = i - which * DH;
        float x = 0.f;
#pragma unroll
        for (int j = 0; j < F32_WAVES; ++j) x += sh_acc[which][j][e];
        float* const out = (which == 0 ? dk : dv) + ((int64_t)tok * Hkv + kvh) * DH + e;
        *out = (which == 0 ? scale * x : x) + (accumulate ? *out : 0.f);
    }
}

template <int DH, bool WIDE>
__global__ __launch_bounds__(F32_BLOCK<WIDE>) void bwd_dkdv_f32_kernel(TabArg table, const float* __restrict__ q, const float* __restrict__ k,
                                                                      const float* __restrict__ v, const float* __restrict__ d_o,
                                                                      const float* __restrict__ lse, const float* __restrict__ D,
                                                                      float* __restrict__ dk, float* __restrict__ dv,
                                                                      int64_t T_total, int Hq, int Hkv, float scale,
                                                                      int resp_only, int accumulate) {
    const int* const tab = table_of(table);
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63;
    int tok, kvh;
    if (!row_and_head<WIDE>(w, T_total, Hkv, tok, kvh)) return;
    dkdv_f32_key<DH, WIDE>(load_group(tab, find_group_of_token(tab, tok)), tok, kvh, w, l, q, k, v, d_o, lse, D, dk, dv, T_total, Hq, Hkv, scale,
                           resp_only, accumulate);
}

// ------------------------------------------------------------------------------------
// Matrix instructions: 16 rows (keys) to a workgroup of eight waves, each of which takes every eighth chunk of 64 keys (rows).
// ------------------------------------------------------------------------------------
// A row per wave read every key's row for itself: L2 traffic bound, 1 MB for a row of 1000 keys.  v_mfma_f32_16x16x4_f32 multiplies in
// float32 and takes operands straight from the rows: lane (i, g) = (l % 16, l / 16) holds elements 16 j + 4 g + e of row i, and the sums
// of 16 x 16 tiles, element 4 g + e of column i, are the operand of the product that follows (of key 4 g + e, row i).
// Where a masked key or row holds an infinity, its weight 0 makes a NaN of the sums; a row with a NaN is computed again by
// itself, which takes no masked key.
constexpr int BLK = 16;
__device__ __forceinline__ f32x4 mfma16(float a, float b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x4f32(a, b, c, 0, 0, 0); }
template <int DH>
__device__ __forceinline__ void row16(const float* __restrict__ p, int g, f32x4 (&x)[DH / 16]) {
#pragma unroll
    for (int j = 0; j < DH / 16; ++j) x[j] = *reinterpret_cast<const f32x4*>(p + 16 * j + 4 * g);
}
// tiles[n] = products of rows 16 n + i (of `rows`, the last one n_rows - 1) with the lanes' row x
template <int DH>
__device__ __forceinline__ void dots16(const float* __restrict__ rows, int64_t stride, int n_rows, int i, int g, const f32x4 (&x)[DH / 16], f32x4 (&tiles)[4]) {
#pragma unroll
    for (int n = 0; n < 4; ++n) tiles[n] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int n = 0; n < 4; ++n) {
        if (16 * n >= n_rows) break;
        f32x4 y[DH / 16];
        row16<DH>(rows + min(16 * n + i, n_rows - 1) * stride, g, y);
        f32x4 part[4];                             // four short sums are closer to the exact one than a long one (and do not wait for each other)
#pragma unroll
        for (int e = 0; e < 4; ++e) part[e] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < DH / 16; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) part[e] = mfma16(y[j][e], x[j][e], part[e]);
#pragma unroll
        for (int r = 0; r < 4; ++r) tiles[n][r] = (part[0][r] + part[1][r]) + (part[2][r] + part[3][r]);
    }
}
// acc[db] += sum over rows j of p (element 4 g + e of tile n is row 16 n + 4 g + e's weight) * row j's elements 16 db + i
template <int DH>
__device__ __forceinline__ void sums16(const float* __restrict__ rows, int64_t stride, int n_rows, int i, int g, const f32x4 (&p)[4], f32x4 (&acc)[DH / 16]) {
    // a step is one row of each lane group; the next step's row is loaded ahead of this one's products
    float x[2][DH / 16];
    auto load = [&](int step, float (&y)[DH / 16]) {
        const float* const r = rows + min(16 * (step >> 2) + 4 * g + (step & 3), n_rows - 1) * stride + i;
#pragma unroll
        for (int db = 0; db < DH / 16; ++db) y[db] = r[16 * db];
    };
    load(0, x[0]);
#pragma unroll
    for (int step = 0; step < 16; ++step) {
        if ((step & 3) == 0 && 4 * step >= n_rows) break;
        if (step + 1 < 16) load(step + 1, x[(step + 1) & 1]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int db = 0; db < DH / 16; ++db) acc[db] = mfma16(x[step & 1][db], p[step >> 2][step & 3], acc[db]);
        __builtin_amdgcn_sched_barrier(0);
    }
}
__device__ __forceinline__ float max4(float x) { x = fmaxf(x, __shfl_xor(x, 16, 64)); return fmaxf(x, __shfl_xor(x, 32, 64)); }
__device__ __forceinline__ float sum4(float x) { x += __shfl_xor(x, 16, 64); return x + __shfl_xor(x, 32, 64); }
__device__ __forceinline__ bool is_nan_bits(float x) {       // by its bits: the build takes float comparisons to see no NaN
    unsigned b = __float_as_uint(x);
    asm volatile("" : "+v"(b));
    return (b & 0x7fffffffu) > 0x7f800000u;
}
// The chunks of 64 keys that any of the rows t0 .. t0 + rows - 1 sees: those of the prompt, then those of the rows' own segments from
// the first response row's first token on.
struct RowsChunks {
    int n1, n, end1, k2, end;
    __device__ __forceinline__ RowsChunks(const GroupDesc& gd, int t0, int rows) {
        end = t0 + rows;
        end1 = min(gd.Lp, end);
        n1 = (end1 + 63) / 64;
        k2 = end > gd.Lp ? seg_start(gd, max(t0, gd.Lp)) : end;
        n = n1 + (end - k2 + 63) / 64;
    }
    __device__ __forceinline__ int first(int i) const { return i < n1 ? 64 * i : k2 + 64 * (i - n1); }
    __device__ __forceinline__ int count(int i) const { return min(64, (i < n1 ? end1 : end) - first(i)); }
};
// calls f(group, first token, number) for the 16 tokens of a workgroup, group by group
template <typename F>
__device__ __forceinline__ void for_tokens(const int* tab, int64_t first, int64_t T_total, F f) {
    const int64_t end = min(first + BLK, T_total);
    for (int64_t tok = first; tok < end;) {
        const GroupDesc gd = load_group(tab, find_group_of_token(tab, tok));
        const int n = (int)min(end - tok, (int64_t)gd.tok_base + gd.Tg - tok);
        f(gd, (int)tok, n);
        tok += n;
    }
}

template <int DH>
__global__ __launch_bounds__(64 * F32_WAVES) void fwd_f32_block_kernel(TabArg table, const float* __restrict__ q, const float* __restrict__ k,
                                                                       const float* __restrict__ v, float* __restrict__ o,
                                                                       float* __restrict__ lse, int64_t T_total, int Hq, int Hkv,
                                                                       float scale, int resp_only) {
    constexpr int NB = DH / 16, PAD = DH + 4;
    __shared__ float sh_m[F32_WAVES][BLK], sh_l[F32_WAVES][BLK];
    __shared__ int sh_bad[BLK];
    __shared__ __attribute__((aligned(16))) float sh_acc[F32_WAVES][BLK][PAD];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, i = l & 15, g = l >> 4;
    const int h = (int)(blockIdx.x % (unsigned)Hq), kvh = h / (Hq / Hkv);
    for_tokens(table_of(table), (int64_t)(blockIdx.x / (unsigned)Hq) * BLK, T_total, [&](const GroupDesc& gd, int tok, int rows) {
        const int t0 = tok - gd.tok_base;
        if (resp_only && t0 + rows <= gd.Lp) return;
        const RowsChunks ch(gd, t0, rows);
        const int64_t kvs = (int64_t)Hkv * DH, qs = (int64_t)Hq * DH;
        const float* const kb = k + ((int64_t)gd.tok_base * Hkv + kvh) * DH;
        const float* const vb = v + ((int64_t)gd.tok_base * Hkv + kvh) * DH;
        const int t = t0 + min(i, rows - 1), st = seg_start(gd, t);
        f32x4 qr[NB], acc[NB];
        row16<DH>(q + (int64_t)(gd.tok_base + t) * qs + h * DH, g, qr);
#pragma unroll
        for (int db = 0; db < NB; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
        float m = -INFINITY, lsum = 0.f;
        for (int c = w; c < ch.n; c += F32_WAVES) {
            const int s0 = ch.first(c), nk = ch.count(c), lo = c < ch.n1 ? 0 : st - s0, hi = min(nk, t + 1 - s0);
            f32x4 S[4];
            dots16<DH>(kb + (int64_t)s0 * kvs, kvs, nk, i, g, qr, S);
            float mx = -INFINITY;
            bool nan = false;
#pragma unroll
            for (int n = 0; n < 4; ++n)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int key = 16 * n + 4 * g + e;
                    S[n][e] = key >= lo && key < hi ? scale * S[n][e] : -INFINITY;
                    nan |= is_nan_bits(S[n][e]);
                    mx = fmaxf(mx, S[n][e]);
                }
            const float mnew = fmaxf(m, max4(mx));
            const uint64_t nans = __builtin_amdgcn_ballot_w64(nan);
            // (nothing but masked keys and scores of -inf so far; a NaN goes on: the sums become NaN)
            const bool none = mnew == -INFINITY && ((nans >> i) & 0x0001000100010001ull) == 0;
            const float alpha = none ? 1.f : expf(m - mnew);
            if (!none) m = mnew;
            lsum *= alpha;
#pragma unroll
            for (int n = 0; n < 4; ++n)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int key = 16 * n + 4 * g + e;
                    S[n][e] = !none && key >= lo && key < hi ? expf(S[n][e] - mnew) : 0.f;
                    lsum += S[n][e];
                }
#pragma unroll
            for (int db = 0; db < NB; ++db)
#pragma unroll
                for (int e = 0; e < 4; ++e) acc[db][e] *= alpha;
            sums16<DH>(vb + (int64_t)s0 * kvs, kvs, nk, i, g, S, acc);
        }
        lsum = sum4(lsum);
        __syncthreads();                           // (the sums of the tokens of another group are read)
        if (g == 0) { sh_m[w][i] = m; sh_l[w][i] = lsum; }
        if (threadIdx.x < BLK) sh_bad[threadIdx.x] = 0;
#pragma unroll
        for (int db = 0; db < NB; ++db) *reinterpret_cast<f32x4*>(&sh_acc[w][i][16 * db + 4 * g]) = acc[db];
        __syncthreads();
        const int r = (int)threadIdx.x >> 5;
        const bool mine = r < rows && !(resp_only && t0 + r < gd.Lp);
        bool bad = false;
        if (mine) {
            float mt = sh_m[0][r];
#pragma unroll
            for (int x = 1; x < F32_WAVES; ++x) mt = fmaxf(mt, sh_m[x][r]);
            float ls = 0.f, f[F32_WAVES];
#pragma unroll
            for (int x = 0; x < F32_WAVES; ++x) {        // a wave without a key (or with scores of -inf only) has no part
                f[x] = __float_as_uint(sh_l[x][r]) == 0u ? 0.f : expf(sh_m[x][r] - mt);
                ls = __builtin_fmaf(sh_l[x][r], f[x], ls);
            }
#pragma unroll
            for (int n = 0; n < DH / 32; ++n) {
                const int d = (threadIdx.x & 31) + 32 * n;
                float x = 0.f;
#pragma unroll
                for (int u = 0; u < F32_WAVES; ++u) x = __builtin_fmaf(sh_acc[u][r][d], f[u], x);
                x /= ls;
                bad |= is_nan_bits(x);
                o[(int64_t)(tok + r) * qs + h * DH + d] = x;
            }
            if ((threadIdx.x & 31) == 0) lse[(int64_t)h * T_total + tok + r] = mt + logf(ls);
        }
        if (bad) sh_bad[r] = 1;
        if (__syncthreads_or(bad))
            for (int x = w; x < rows; x += F32_WAVES)
                if (sh_bad[x]) fwd_f32_row<DH, false>(gd, tok + x, h, w, l, q, k, v, o, lse, T_total, Hq, Hkv, scale, resp_only);
    });
}

template <int DH>
__global__ __launch_bounds__(64 * F32_WAVES) void bwd_dq_f32_block_kernel(TabArg table, const float* __restrict__ q, const float* __restrict__ k,
                                                                          const float* __restrict__ v, const float* __restrict__ d_o,
                                                                          const float* __restrict__ o, const float* __restrict__ lse,
                                                                          float* __restrict__ D, float* __restrict__ dq, uint32_t* __restrict__ tag,
                                                                          int64_t T_total, int Hq, int Hkv, float scale, int resp_only) {
    constexpr int NB = DH / 16, PAD = DH + 4, PER = DH / 64;
    __shared__ float sh_D[BLK];
    __shared__ int sh_bad[BLK];
    __shared__ __attribute__((aligned(16))) float sh_acc[F32_WAVES][BLK][PAD];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, i = l & 15, g = l >> 4;
    if (tag && blockIdx.x == 0 && w == 0) tag[l] = 0u;
    const int h = (int)(blockIdx.x % (unsigned)Hq), kvh = h / (Hq / Hkv);
    for_tokens(table_of(table), (int64_t)(blockIdx.x / (unsigned)Hq) * BLK, T_total, [&](const GroupDesc& gd, int tok, int rows) {
        const int t0 = tok - gd.tok_base;
        if (resp_only && t0 + rows <= gd.Lp) return;
        const RowsChunks ch(gd, t0, rows);
        const int64_t kvs = (int64_t)Hkv * DH, qs = (int64_t)Hq * DH, row0 = (int64_t)tok * qs + h * DH, word = (int64_t)h * T_total + tok;
        const float* const kb = k + ((int64_t)gd.tok_base * Hkv + kvh) * DH;
        const float* const vb = v + ((int64_t)gd.tok_base * Hkv + kvh) * DH;
        __syncthreads();                           // (the sums of the tokens of another group are read)
        for (int x = w; x < rows; x += F32_WAVES) {                   // D, as in dq_f32_row()
            float Dt = 0.f;
            if (o) {
#pragma unroll
                for (int e = 0; e < PER; ++e) Dt += d_o[row0 + x * qs + l + 64 * e] * o[row0 + x * qs + l + 64 * e];
                Dt = wave_sum(Dt);
                if (l == 0 && !(resp_only && t0 + x < gd.Lp)) D[word + x] = Dt;
            } else {
                Dt = D[word + x];
            }
            if (l == 0) { sh_D[x] = Dt; sh_bad[x] = 0; }
        }
        const int n0 = min(i, rows - 1), t = t0 + n0, st = seg_start(gd, t);
        const float L = lse[word + n0];
        f32x4 qr[NB], gr[NB], acc[NB];
        row16<DH>(q + row0 + n0 * qs, g, qr);
        row16<DH>(d_o + row0 + n0 * qs, g, gr);
#pragma unroll
        for (int db = 0; db < NB; ++db) acc[db] = f32x4{0.f, 0.f, 0.f, 0.f};
        __syncthreads();
        const float Dt = sh_D[n0];
        for (int c = w; c < ch.n; c += F32_WAVES) {
            const int s0 = ch.first(c), nk = ch.count(c), lo = c < ch.n1 ? 0 : st - s0, hi = min(nk, t + 1 - s0);
            f32x4 S[4], P[4];
            dots16<DH>(kb + (int64_t)s0 * kvs, kvs, nk, i, g, qr, S);
            dots16<DH>(vb + (int64_t)s0 * kvs, kvs, nk, i, g, gr, P);
#pragma unroll
            for (int n = 0; n < 4; ++n)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int key = 16 * n + 4 * g + e;
                    S[n][e] = key >= lo && key < hi ? expf(scale * S[n][e] - L) * (P[n][e] - Dt) : 0.f;
                }
            sums16<DH>(kb + (int64_t)s0 * kvs, kvs, nk, i, g, S, acc);
        }
#pragma unroll
        for (int db = 0; db < NB; ++db) *reinterpret_cast<f32x4*>(&sh_acc[w][i][16 * db + 4 * g]) = acc[db];
        __syncthreads();
        const int r = (int)threadIdx.x >> 5;
        bool bad = false;
        if (r < rows && !(resp_only && t0 + r < gd.Lp))
#pragma unroll
            for (int n = 0; n < DH / 32; ++n) {
                const int d = (threadIdx.x & 31) + 32 * n;
                float x = 0.f;
#pragma unroll
                for (int u = 0; u < F32_WAVES; ++u) x += sh_acc[u][r][d];
                bad |= is_nan_bits(x);
                dq[row0 + r * qs + d] = scale * x;
            }
        if (bad) sh_bad[r] = 1;
        if (__syncthreads_or(bad))
            for (int x = w; x < rows; x += F32_WAVES)
                if (sh_bad[x]) dq_f32_row<DH, false>(gd, tok + x, h, w, l, q, k, v, d_o, o, lse, D, dq, T_total, Hq, Hkv, scale, resp_only);
    });
}

template <int DH>
__global__ __launch_bounds__(64 * F32_WAVES) void bwd_dkdv_f32_block_kernel(TabArg table, const float* __restrict__ q, const float* __restrict__ k,
                                                                            const float* __restrict__ v, const float* __restrict__ d_o,
                                                                            const float* __restrict__ lse, const float* __restrict__ D,
                                                                            float* __restrict__ dk, float* __restrict__ dv,
                                                                            int64_t T_total, int Hq, int Hkv, float scale,
                                                                            int resp_only, int accumulate) {
    constexpr int NB = DH / 16, PAD = DH + 4;
    __shared__ int sh_bad[BLK];
    __shared__ __attribute__((aligned(16))) float sh_acc[F32_WAVES][BLK][PAD];
    const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), l = threadIdx.x & 63, i = l & 15, g = l >> 4;
    const int kvh = (int)(blockIdx.x % (unsigned)Hkv);
    for_tokens(table_of(table), (int64_t)(blockIdx.x / (unsigned)Hkv) * BLK, T_total, [&](const GroupDesc& gd, int tok, int keys) {
        const int s0 = tok - gd.tok_base, rep = Hq / Hkv;
        const int64_t kvs = (int64_t)Hkv * DH, qs = (int64_t)Hq * DH, key0 = (int64_t)tok * kvs + kvh * DH;
        // rows first .. end - 1 see the lane's key; row_lo .. row_end - 1 see one of the block's
        const int n0 = min(i, keys - 1), s = s0 + n0, last = s0 + keys - 1, first = resp_only ? max(s, gd.Lp) : s;
        const int end = i < keys ? (s < gd.Lp ? gd.Tg : seg_end(gd, s)) : 0;
        const int row_lo = resp_only ? max(s0, gd.Lp) : s0, row_end = s0 < gd.Lp ? gd.Tg : seg_end(gd, last);
        const int n = max(row_end - row_lo + 63, 0) / 64;
        f32x4 kr[NB], vr[NB], ak[NB], av[NB];
        row16<DH>(k + key0 + n0 * kvs, g, kr);
        row16<DH>(v + key0 + n0 * kvs, g, vr);
#pragma unroll
        for (int db = 0; db < NB; ++db) { ak[db] = f32x4{0.f, 0.f, 0.f, 0.f}; av[db] = f32x4{0.f, 0.f, 0.f, 0.f}; }
        for (int hr = 0, c = w; hr < rep; ++hr, c -= n) {              // chunk c of the n * rep, counted within the head
            for (; c < n; c += F32_WAVES) {
                const int h = kvh * rep + hr, r0 = row_lo + 64 * c, nr = min(64, row_end - r0), lo = first - r0, hi = min(nr, end - r0);
                const int64_t rows = (int64_t)(gd.tok_base + r0) * qs + h * DH, word = (int64_t)h * T_total + gd.tok_base + r0;
                f32x4 P[4], S[4];
                dots16<DH>(q + rows, qs, nr, i, g, kr, P);
                dots16<DH>(d_o + rows, qs, nr, i, g, vr, S);
#pragma unroll
                for (int x = 0; x < 4; ++x)
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int row = 16 * x + 4 * g + e, at = min(row, nr - 1);
                        const bool ok = row >= lo && row < hi;
                        P[x][e] = ok ? expf(scale * P[x][e] - lse[word + at]) : 0.f;
                        S[x][e] = ok ? P[x][e] * (S[x][e] - D[word + at]) : 0.f;
                    }
                sums16<DH>(d_o + rows, qs, nr, i, g, P, av);
                sums16<DH>(q + rows, qs, nr, i, g, S, ak);
            }
        }
        const int r = (int)threadIdx.x >> 5;
        float x[2][DH / 32];
        bool bad = false;
#pragma unroll
        for (int which = 0; which < 2; ++which) {
            __syncthreads();                       // (the sums before these are read)
            if (which == 0 && threadIdx.x < BLK) sh_bad[threadIdx.x] = 0;
#pragma unroll
            for (int db = 0; db < NB; ++db) *reinterpret_cast<f32x4*>(&sh_acc[w][i][16 * db + 4 * g]) = which == 0 ? ak[db] : av[db];
            __syncthreads();
#pragma unroll
            for (int u = 0; u < DH / 32; ++u) {
                x[which][u] = 0.f;
#pragma unroll
                for (int y = 0; y < F32_WAVES; ++y) x[which][u] += sh_acc[y][r][(threadIdx.x & 31) + 32 * u];
                bad |= r < keys && is_nan_bits(x[which][u]);
            }
        }
        if (bad) sh_bad[r] = 1;
        if (__syncthreads_or(bad))
            for (int y = w; y < keys; y += F32_WAVES)
                if (sh_bad[y]) dkdv_f32_key<DH, false>(gd, tok + y, kvh, w, l, q, k, v, d_o, lse, D, dk, dv, T_total, Hq, Hkv, scale, resp_only, accumulate);
        if (r >= keys || sh_bad[r]) return;
#pragma unroll
        for (int which = 0; which < 2; ++which)
#pragma unroll
            for (int u = 0; u < DH / 32; ++u) {
                float* const out = (which == 0 ? dk : dv) + key0 + r * kvs + (threadIdx.x & 31) + 32 * u;
                *out = (which == 0 ? scale * x[0][u] : x[1][u]) + (accumulate ? *out : 0.f);
            }
    });
}

inline int blocks_for_waves(int64_t waves) { return (int)((waves + 3) / 4); }

}  // namespace

// Tag block, segment table and (bf16) schedule of a call: one launch when the table fits a kernel-argument
// block, else the tag kernel, the table in pieces and the schedule kernel.
hipError_t launch_prepare(const int32_t* host_words, int n_words, int* dev_tab, uint32_t* tag_block, const ReserveTag& tag,
                          int tag_mode, bool with_schedule, int n_groups, int64_t total_tokens, int n256, int n128,
                          const Schedule& sched, int key_order, hipStream_t s) {
    TileDesc* const t256 = (TileDesc*)sched.tiles256;
    TileDesc* const t128 = (TileDesc*)sched.tiles128;
    TileDesc* const kt = (TileDesc*)sched.key_tiles;
    int* const key_lo = (int*)sched.key_lo;
    int* const row_hi = (int*)sched.row_hi;
    int64_t n = total_tokens;
    if (n128 > n) n = n128;                            // n128 >= n256
    const unsigned sched_blocks = (unsigned)((n + 255) / 256);
    if (n_words <= PREP_WORDS) {
        PrepChunk c;
        for (int i = 0; i < n_words; ++i) c.w[i] = host_words[i];
        for (int i = n_words; i < PREP_WORDS; ++i) c.w[i] = 0;
        hipLaunchKernelGGL(prepare_kernel, dim3(with_schedule ? sched_blocks : 1u), dim3(256), 0, s, c, n_words, dev_tab,
                           tag_block, tag, tag_mode, with_schedule ? 1 : 0, n_groups, total_tokens, n256, n128, t256, t128,
                           kt, key_lo, row_hi, key_order);
        return hipGetLastError();
    }
    if (tag_mode != TAG_KEEP) {
        hipLaunchKernelGGL(reserve_tag_kernel, dim3(1), dim3(64), 0, s, tag_block, tag, tag_mode);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    for (int off = 0; off < n_words; off += TAB_CHUNK_WORDS) {
        TabChunk c;
        const int nw = n_words - off < TAB_CHUNK_WORDS ? n_words - off : TAB_CHUNK_WORDS;
        for (int i = 0; i < nw; ++i) c.w[i] = host_words[off + i];
        for (int i = nw; i < TAB_CHUNK_WORDS; ++i) c.w[i] = 0;
        hipLaunchKernelGGL(upload_table_kernel, dim3(1), dim3(256), 0, s, c, dev_tab, off, nw);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    if (with_schedule)
        hipLaunchKernelGGL(schedule_kernel, dim3(sched_blocks), dim3(256), 0, s, (const int*)dev_tab, n_groups, total_tokens,
                           n256, n128, t256, t128, kt, key_lo, row_hi, key_order);
    return hipGetLastError();
}

hipError_t launch_rowsum(const Problem& p, bool f32, hipStream_t s) {
    const int grid = blocks_for_waves(p.total_tokens * p.Hq);
    if (f32)
        hipLaunchKernelGGL(rowsum_kernel<float>, dim3(grid), dim3(256), 0, s, (const float*)p.d_o,
                           (const float*)p.o, p.lse, p.Dbuf, p.total_tokens, p.Hq, p.head_dim, p.tab, p.resp_only, (const float*)nullptr);
    else if (rowsum_fast_path(p)) {
        const dim3 g((unsigned)((p.total_tokens + RS_TOK - 1) / RS_TOK));
        const size_t lds = (size_t)p.Hq * RS_TOK * sizeof(float);
        if (p.o_lo)
            hipLaunchKernelGGL(rowsum_bf16_kernel<true>, g, dim3(256), lds, s, (const __bf16*)p.d_o, (const __bf16*)p.o,
                               p.lse, p.Dbuf, p.total_tokens, p.Hq, p.tab, p.resp_only, (const __bf16*)p.o_lo, p.o_lo_flag);
        else
            hipLaunchKernelGGL(rowsum_bf16_kernel<false>, g, dim3(256), lds, s, (const __bf16*)p.d_o, (const __bf16*)p.o,
                               p.lse, p.Dbuf, p.total_tokens, p.Hq, p.tab, p.resp_only, (const __bf16*)nullptr,
                               (const uint32_t*)nullptr);
        hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        // exact D for the rows that see only a few keys (sp_edge.hpp)
        e = launch_short_rows(p, s);
        if (e != hipSuccess) return e;
    }
    else
        hipLaunchKernelGGL(rowsum_kernel<__bf16>, dim3(grid), dim3(256), 0, s, (const __bf16*)p.d_o,
                           (const __bf16*)p.o, p.lse, p.Dbuf, p.total_tokens, p.Hq, p.head_dim, p.tab, p.resp_only,
                           (const __bf16*)(p.o_lo_flag ? nullptr : p.o_lo));      // this fallback does not consult the reserve
    return hipGetLastError();
}

namespace {
// Rows (keys) times heads of a float32 kernel; the chunks of 32 keys (rows) that they walk, and the longest one's; blocks of 16 times
// heads, one for each group of which it holds tokens, and the most of them in one block.
struct F32Counts { int64_t items = 0, chunks = 0, blocks = 0; int longest = 0, spans = 1; };
// sum of ceil(i / 32) over i = 1 .. n
inline int64_t chunks_to(int64_t n) { const int64_t c = n / 32; return 16 * c * (c + 1) + (n - 32 * c) * (c + 1); }
inline F32Counts f32_counts(const Problem& p, bool keys) {
    F32Counts n;
    const int heads = keys ? p.Hkv : p.Hq, rep = keys ? p.Hq / p.Hkv : 1;
    int spans = 0, block = -1;
    for (int g = 0; g < p.n_groups; ++g) {
        const int32_t* e = p.host_table + TAB_HEADER + TAB_GROUP_WORDS * g;
        const int32_t* roff = p.host_table + e[3];
        const int Lp = e[1], Tg = e[2], lo = p.resp_only ? Tg - Lp : Tg, prompt = (Lp + 31) / 32;      // lo: rows that see prompt key 0
        if (keys) n.chunks += p.resp_only ? (int64_t)Lp * ((lo + 31) / 32) : chunks_to(Tg) - chunks_to(Tg - Lp);
        else if (!p.resp_only) n.chunks += chunks_to(Lp);
        int most = keys ? (Lp > 0 ? (lo + 31) / 32 : 0) : (p.resp_only ? 0 : prompt);
        for (int i = 0; i < e[4]; ++i) {
            const int len = roff[i + 1] - roff[i];
            n.chunks += chunks_to(len) + (keys ? 0 : (int64_t)len * prompt);
            most = std::max(most, (len + 31) / 32 + (keys || len == 0 ? 0 : prompt));
        }
        n.longest = std::max(n.longest, most * rep);
        n.blocks += e[0] % BLK != 0;
        spans = e[0] / BLK == block ? spans + 1 : 1 + (e[0] % BLK != 0);      // groups that begin in the block so far, and one that reaches into it
        block = e[0] / BLK;
        n.spans = std::max(n.spans, spans);
    }
    n.chunks *= p.Hq;
    n.items = p.total_tokens * heads;
    n.blocks = (n.blocks + (p.total_tokens + BLK - 1) / BLK) * heads;
    return n;
}
// The shape with the least time by its counts: a launch takes `fixed` us, and behind that as long as its longest workgroup (`step` per round of
// chunks, one of a lone wave, eight of eight waves, 16 in a block, and `span` for each further group of a block) or as all of them
// together (`item` per row or block, `chunk` per chunk of a row or a block).  Fitted to 500 packings of 20 to 12000 tokens, one to 150 groups, 2 / 1 to
// 16 / 4 heads, each timed in all three shapes: rms of an estimate 6 to 19 %; the shape taken costs 0.8 % over the best one on average.
// By rows times heads alone (blocks from 760, 550 and 700 on, and no row by a wave) what takes few chunks, or holds many groups, had lost to
// a wave or a workgroup per row; us, by rows times heads -> by counts: 8 + 100 x 30 tokens, 4 / 2 heads of 64, dkdv 210 -> 133; 32 + 40 x 20, 4 / 2
// of 128, dkdv 115 -> 69; 25 x (3 x 3), 4 / 2 of 128, forward 20.5 -> 13.7; 3 x (5 + 3 x 20), 4 / 4 of 64, 45 -> 29 in all; 500 packings 0.94
// of the time on average.
enum F32Shape { BY_WAVE, BY_WORKGROUP, BY_BLOCK };       // rows (keys) per workgroup: 4, 1, 16
struct F32Time { float fixed, step, item, chunk, span; };
constexpr F32Time F32_TIMES[3][2][3] = {       // [forward, dq, dkdv][heads of 64, 128][F32Shape]
    {{{4.8f, 1.7f, .0006f, .0010f, 0.f}, {3.8f, 2.4f, .0047f, .0012f, 0.f}, {4.5f, 5.5f, .028f, .0024f, 3.7f}},
     {{5.4f, 2.9f, 0.f, .0026f, 0.f}, {3.5f, 6.2f, .0099f, .0027f, 0.f}, {5.3f, 6.9f, .033f, .0061f, 4.0f}}},
    {{{6.3f, 2.0f, .0007f, .0016f, 0.f}, {3.9f, 2.6f, .0032f, .0023f, 0.f}, {5.5f, 6.1f, .024f, .0045f, 2.0f}},
     {{7.2f, 3.8f, 0.f, .0042f, 0.f}, {4.4f, 6.1f, .0077f, .0044f, 0.f}, {6.9f, 7.7f, .027f, .011f, 3.1f}}},
    {{{6.5f, 3.4f, 0.f, .0036f, 0.f}, {2.4f, 5.4f, .0050f, .0029f, 0.f}, {5.0f, 14.f, .041f, .0078f, 3.8f}},
     {{5.3f, 6.3f, 0.f, .0057f, 0.f}, {1.0f, 9.5f, .013f, .0052f, 0.f}, {1.9f, 28.f, .085f, .014f, 6.5f}}}};
F32Shape f32_shape(const F32Counts& n, int kernel, int head_dim) {
    const F32Time* const t = F32_TIMES[kernel][head_dim == 64 ? 0 : 1];
    auto time = [&](F32Shape s, int per_step, int64_t items, int per_chunk, int spans) {
        return t[s].fixed + std::max(t[s].step * (float)((n.longest + per_step - 1) / per_step) + t[s].span * (float)(spans - 1),
                                     t[s].item * (float)items + t[s].chunk * (float)n.chunks / (float)per_chunk);
    };
    const float wave = time(BY_WAVE, 1, n.items, 1, 1), group = time(BY_WORKGROUP, F32_WAVES, n.items, 1, 1);
    const float block = time(BY_BLOCK, 2 * F32_WAVES, n.blocks, BLK, n.spans);
    return block <= std::min(wave, group) ? BY_BLOCK : group <= wave ? BY_WORKGROUP : BY_WAVE;
}
}  // namespace

int f32_rows(const Problem& p, int kernel) {
    constexpr int ROWS[3] = {4, 1, BLK};
    return ROWS[f32_shape(f32_counts(p, kernel == 2), kernel, p.head_dim)];
}

// Calls row(head dimension, WIDE, grid, workgroup) or block(head dimension, grid, workgroup).
template <typename F, typename G>
void with_f32_shape(const Problem& p, int kernel, F row, G block) {
    const int heads = kernel == 2 ? p.Hkv : p.Hq, rows = f32_rows(p, kernel);
    const dim3 grid((unsigned)(rows == BLK ? (p.total_tokens + BLK - 1) / BLK * heads : (p.total_tokens * heads + rows - 1) / rows));
    auto sized = [&](auto dh) {
        if (rows == 4) row(dh, std::false_type{}, grid, dim3(F32_BLOCK<false>));
        else if (rows == 1) row(dh, std::true_type{}, grid, dim3(F32_BLOCK<true>));
        else block(dh, grid, dim3(64 * F32_WAVES));
    };
    if (p.head_dim == 64) sized(std::integral_constant<int, 64>{}); else sized(std::integral_constant<int, 128>{});
}
inline TabArg f32_table(const Problem& p) {
    return make_tab_arg(p.host_table, p.small.on ? (size_t)p.host_table[2] : (size_t)ARG_WORDS + 1, p.tab);
}

hipError_t launch_fwd_f32(const Problem& p, hipStream_t s) {
    auto go = [&](auto kernel, dim3 grid, dim3 block) {
        hipLaunchKernelGGL(kernel, grid, block, 0, s, f32_table(p), (const float*)p.q, (const float*)p.k, (const float*)p.v,
                           (float*)p.o_out, p.lse_out, p.total_tokens, p.Hq, p.Hkv, p.scale, p.resp_only);
    };
    with_f32_shape(p, 0,
        [&](auto dh, auto wide, dim3 grid, dim3 block) { go(fwd_f32_kernel<decltype(dh)::value, decltype(wide)::value>, grid, block); },
        [&](auto dh, dim3 grid, dim3 block) { go(fwd_f32_block_kernel<decltype(dh)::value>, grid, block); });
    return hipGetLastError();
}

hipError_t launch_bwd_f32(const Problem& p, hipStream_t s) {
    const bool fused = (p.stages & STAGE_ROWSUM) && (p.stages & STAGE_DQ);      // rowsum within the dq kernel
    if ((p.stages & STAGE_ROWSUM) && !fused) {
        hipError_t e = launch_rowsum(p, true, s);
        if (e != hipSuccess) return e;
    }
    if (p.stages & STAGE_DQ) {
        auto go = [&](auto kernel, dim3 grid, dim3 block) {
            hipLaunchKernelGGL(kernel, grid, block, 0, s, f32_table(p), (const float*)p.q, (const float*)p.k, (const float*)p.v,
                               (const float*)p.d_o, fused ? (const float*)p.o : nullptr, p.lse, p.Dbuf, (float*)p.dq,
                               p.small.on ? p.small.tag : nullptr, p.total_tokens, p.Hq, p.Hkv, p.scale, p.resp_only);
        };
        with_f32_shape(p, 1,
            [&](auto dh, auto wide, dim3 grid, dim3 block) { go(bwd_dq_f32_kernel<decltype(dh)::value, decltype(wide)::value>, grid, block); },
            [&](auto dh, dim3 grid, dim3 block) { go(bwd_dq_f32_block_kernel<decltype(dh)::value>, grid, block); });
    }
    if (p.stages & STAGE_DKDV) {
        auto go = [&](auto kernel, dim3 grid, dim3 block) {
            hipLaunchKernelGGL(kernel, grid, block, 0, s, f32_table(p), (const float*)p.q, (const float*)p.k, (const float*)p.v,
                               (const float*)p.d_o, p.lse, p.Dbuf, (float*)p.dk, (float*)p.dv, p.total_tokens, p.Hq, p.Hkv, p.scale,
                               p.resp_only, p.accumulate);
        };
        with_f32_shape(p, 2,
            [&](auto dh, auto wide, dim3 grid, dim3 block) { go(bwd_dkdv_f32_kernel<decltype(dh)::value, decltype(wide)::value>, grid, block); },
            [&](auto dh, dim3 grid, dim3 block) { go(bwd_dkdv_f32_block_kernel<decltype(dh)::value>, grid, block); });
    }
    return hipGetLastError();
}

}  // namespace sp
