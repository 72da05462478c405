// float32 plain-ALU debug path of shared-prompt attention, the segment-table upload
// and the backward preprocess D = rowsum(dO * O).
//
// The debug kernels give one wavefront a single (row, head) or (key, kv head) and walk
// the allowed keys / rows of the Section 4.3 mask in chunks of 64, one per lane.  No
// MFMA, no LDS: they exist to cross-check the MFMA path and to serve float32 callers.
#include "sp_common.hpp"
#include "sp_launch.hpp"
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

// The float32 kernels are bound by latency, not by arithmetic: a wave walks its keys (rows) in chunks of 64, and per chunk
// each lane first needs a whole row of its own (dot_row: all loads ahead of the sums; the wave's own row x is uniform) and
// then the wave a row per key, ROWS of them in flight (add_rows; with one in flight a chunk took 5 us).
// Order of every sum as in the plain loops.  One box, a group of 64 + 4 x 32 tokens, 2 heads of 64, us before -> after:
// forward 19.6 -> 10.8, dq 23.0 -> 13.0, dkdv 37.1 -> 24.0; backward of 1500 + 5 x 200 tokens, 4 heads of 128,
// 4.30 -> 3.29 ms (ROWS = 16: 3.56).
constexpr int ROWS = 32;
template <int DH>
__device__ __forceinline__ float dot_row(const float* __restrict__ x, const float* __restrict__ y) {
    f32x4 v[DH / 4];
#pragma unroll
    for (int i = 0; i < DH / 4; ++i) v[i] = *reinterpret_cast<const f32x4*>(y + 4 * i);
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < DH; ++i) acc = __builtin_fmaf(x[i], v[i >> 2][i & 3], acc);
    return acc;
}
__device__ __forceinline__ float lane_value(float x, int lane) {      // of a wave-uniform lane
    return __uint_as_float((unsigned)__builtin_amdgcn_readlane((int)__float_as_uint(x), lane));
}
// acc[e] += sum over j < n of lane j's p * row j's element l + 64 e; p is 0 in the lanes from n on.  Row j at base + j * stride.
// The last ROWS rows may run past n: they repeat row n - 1 with weight 0, which is nothing unless that row holds an
// infinity (0 * inf).  A sum that became NaN is therefore taken once more over the n rows alone, one by one; excluding the
// repeated rows with a select per row instead cost the tiny group above 52.8 -> 60.3 us a training pass.
template <int PER>
__device__ __forceinline__ void add_rows(float (&acc)[PER], float p, const float* __restrict__ base, int64_t stride, int n, int l) {
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

template <int DH>
__global__ __launch_bounds__(256) void fwd_f32_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                      const float* __restrict__ v, float* __restrict__ o,
                                                      float* __restrict__ lse, const int* __restrict__ tab,
                                                      int Hq, int Hkv, float scale, int resp_only) {
    constexpr int PER = DH / 64;
    const int64_t T_total = tab[1];
    const int64_t gw = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = threadIdx.x & 63;
    if (gw >= T_total * Hq) return;
    const int tok = (int)(gw / Hq), h = (int)(gw % Hq);
    const GroupDesc gd = load_group(tab, find_group_of_token(tab, tok));
    const int t = tok - gd.tok_base;
    if (resp_only && t < gd.Lp) return;
    const int st = seg_start(gd, t);
    const int kvh = h / (Hq / Hkv);
    const float* qrow = q + ((int64_t)tok * Hq + h) * DH;
    const float* kb = k + ((int64_t)gd.tok_base * Hkv + kvh) * DH;
    const float* vb = v + ((int64_t)gd.tok_base * Hkv + kvh) * DH;
    const int64_t kvs = (int64_t)Hkv * DH;

    float m = -INFINITY, lsum = 0.f, acc[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] = 0.f;
    for (int s0 = 0; s0 <= t; s0 += 64) {
        if (s0 >= gd.Lp && s0 + 64 <= st) continue;        // wholly inside other responses
        const int s = s0 + l;
        const bool ok = s <= t && (s < gd.Lp || s >= st);
        const float sc = ok ? scale * dot_row<DH>(qrow, kb + (int64_t)s * kvs) : -INFINITY;
        const float mnew = fmaxf(m, wave_max(sc));
        if (mnew == -INFINITY) continue;
        const float alpha = expf(m - mnew);
        const float p = ok ? expf(sc - mnew) : 0.f;
        lsum = lsum * alpha + wave_sum(p);
        m = mnew;
        const int nk = min(64, t + 1 - s0);
#pragma unroll
        for (int e = 0; e < PER; ++e) acc[e] *= alpha;
        add_rows<PER>(acc, p, vb + (int64_t)s0 * kvs, kvs, nk, l);
    }
    float* orow = o + ((int64_t)tok * Hq + h) * DH;
#pragma unroll
    for (int e = 0; e < PER; ++e) orow[l + 64 * e] = acc[e] / lsum;
    if (l == 0) lse[(int64_t)h * T_total + tok] = m + logf(lsum);
}

// dQ[t,h] = scale * sum_s dS[t,s] K[s],  dS = P * (dP - D)
template <int DH>
__global__ __launch_bounds__(256) void bwd_dq_f32_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                         const float* __restrict__ v, const float* __restrict__ d_o,
                                                         const float* __restrict__ lse, const float* __restrict__ D,
                                                         float* __restrict__ dq, const int* __restrict__ tab,
                                                         int Hq, int Hkv, float scale, int resp_only) {
    constexpr int PER = DH / 64;
    const int64_t T_total = tab[1];
    const int64_t gw = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = threadIdx.x & 63;
    if (gw >= T_total * Hq) return;
    const int tok = (int)(gw / Hq), h = (int)(gw % Hq);
    const GroupDesc gd = load_group(tab, find_group_of_token(tab, tok));
    const int t = tok - gd.tok_base;
    if (resp_only && t < gd.Lp) return;
    const int st = seg_start(gd, t);
    const int kvh = h / (Hq / Hkv);
    const float* qrow = q + ((int64_t)tok * Hq + h) * DH;
    const float* gorow = d_o + ((int64_t)tok * Hq + h) * DH;
    const float* kb = k + ((int64_t)gd.tok_base * Hkv + kvh) * DH;
    const float* vb = v + ((int64_t)gd.tok_base * Hkv + kvh) * DH;
    const int64_t kvs = (int64_t)Hkv * DH;
    const float L = lse[(int64_t)h * T_total + tok];
    const float Dt = D[(int64_t)h * T_total + tok];

    float acc[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) acc[e] = 0.f;
    for (int s0 = 0; s0 <= t; s0 += 64) {
        if (s0 >= gd.Lp && s0 + 64 <= st) continue;
        const int s = s0 + l;
        const bool ok = s <= t && (s < gd.Lp || s >= st);
        float ds = 0.f;
        if (ok) {
            const float p = expf(scale * dot_row<DH>(qrow, kb + (int64_t)s * kvs) - L);
            ds = p * (dot_row<DH>(gorow, vb + (int64_t)s * kvs) - Dt);
        }
        const int nk = min(64, t + 1 - s0);
        add_rows<PER>(acc, ds, kb + (int64_t)s0 * kvs, kvs, nk, l);
    }
    float* out = dq + ((int64_t)tok * Hq + h) * DH;
#pragma unroll
    for (int e = 0; e < PER; ++e) out[l + 64 * e] = scale * acc[e];
}

// dK[s,g] = scale * sum_{h in g} sum_t dS[t,s] Q[t,h];  dV[s,g] = sum_{h in g} sum_t P[t,s] dO[t,h].
// The rows that see key s are contiguous: [s, Tg) for a prompt key (later prompt rows and
// every row of every response), [s, end of its response) otherwise.
template <int DH>
__global__ __launch_bounds__(256) void bwd_dkdv_f32_kernel(const float* __restrict__ q, const float* __restrict__ k,
                                                           const float* __restrict__ v, const float* __restrict__ d_o,
                                                           const float* __restrict__ lse, const float* __restrict__ D,
                                                           float* __restrict__ dk, float* __restrict__ dv,
                                                           const int* __restrict__ tab, int Hq, int Hkv, float scale,
                                                           int resp_only, int accumulate) {
    constexpr int PER = DH / 64;
    const int64_t T_total = tab[1];
    const int64_t gw = (int64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int l = threadIdx.x & 63;
    if (gw >= T_total * Hkv) return;
    const int tok = (int)(gw / Hkv), kvh = (int)(gw % Hkv);
    const GroupDesc gd = load_group(tab, find_group_of_token(tab, tok));
    const int s = tok - gd.tok_base;
    const int row_end = s < gd.Lp ? gd.Tg : seg_end(gd, s);
    const int rep = Hq / Hkv;
    const float* krow = k + ((int64_t)tok * Hkv + kvh) * DH;
    const float* vrow = v + ((int64_t)tok * Hkv + kvh) * DH;

    float ak[PER], av[PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) { ak[e] = 0.f; av[e] = 0.f; }
    for (int hr = 0; hr < rep; ++hr) {
        const int h = kvh * rep + hr;
        for (int r0 = resp_only ? max(s, gd.Lp) : s; r0 < row_end; r0 += 64) {
            const int t = r0 + l;
            float p = 0.f, ds = 0.f;
            if (t < row_end) {
                const int64_t row = ((int64_t)(gd.tok_base + t) * Hq + h) * DH;
                const int64_t sidx = (int64_t)h * T_total + gd.tok_base + t;
                p = expf(scale * dot_row<DH>(q + row, krow) - lse[sidx]);
                ds = p * (dot_row<DH>(d_o + row, vrow) - D[sidx]);
            }
            const int nr = min(64, row_end - r0);
            const int64_t row0 = ((int64_t)(gd.tok_base + r0) * Hq + h) * DH;
            add_rows<PER>(av, p, d_o + row0, (int64_t)Hq * DH, nr, l);
            add_rows<PER>(ak, ds, q + row0, (int64_t)Hq * DH, nr, l);
        }
    }
    float* okr = dk + ((int64_t)tok * Hkv + kvh) * DH;
    float* ovr = dv + ((int64_t)tok * Hkv + kvh) * DH;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        okr[l + 64 * e] = scale * ak[e] + (accumulate ? okr[l + 64 * e] : 0.f);
        ovr[l + 64 * e] = av[e] + (accumulate ? ovr[l + 64 * e] : 0.f);
    }
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

hipError_t launch_fwd_f32(const Problem& p, hipStream_t s) {
    const int grid = blocks_for_waves(p.total_tokens * p.Hq);
    if (p.head_dim == 64)
        hipLaunchKernelGGL(fwd_f32_kernel<64>, dim3(grid), dim3(256), 0, s, (const float*)p.q, (const float*)p.k,
                           (const float*)p.v, (float*)p.o_out, p.lse_out, p.tab, p.Hq, p.Hkv, p.scale, p.resp_only);
    else
        hipLaunchKernelGGL(fwd_f32_kernel<128>, dim3(grid), dim3(256), 0, s, (const float*)p.q, (const float*)p.k,
                           (const float*)p.v, (float*)p.o_out, p.lse_out, p.tab, p.Hq, p.Hkv, p.scale, p.resp_only);
    return hipGetLastError();
}

hipError_t launch_bwd_f32(const Problem& p, hipStream_t s) {
    if (p.stages & STAGE_ROWSUM) {
        hipError_t e = launch_rowsum(p, true, s);
        if (e != hipSuccess) return e;
    }
    const int gq = blocks_for_waves(p.total_tokens * p.Hq);
    const int gk = blocks_for_waves(p.total_tokens * p.Hkv);
#define SP_F32_BWD(DH)                                                                                      \
    if (p.stages & STAGE_DQ)                                                                               \
    hipLaunchKernelGGL(bwd_dq_f32_kernel<DH>, dim3(gq), dim3(256), 0, s, (const float*)p.q, (const float*)p.k, \
                       (const float*)p.v, (const float*)p.d_o, p.lse, p.Dbuf, (float*)p.dq, p.tab, p.Hq,   \
                       p.Hkv, p.scale, p.resp_only);                                                       \
    if (p.stages & STAGE_DKDV)                                                                             \
    hipLaunchKernelGGL(bwd_dkdv_f32_kernel<DH>, dim3(gk), dim3(256), 0, s, (const float*)p.q,              \
                       (const float*)p.k, (const float*)p.v, (const float*)p.d_o, p.lse, p.Dbuf,           \
                       (float*)p.dk, (float*)p.dv, p.tab, p.Hq, p.Hkv, p.scale, p.resp_only, p.accumulate);
    if (p.head_dim == 64) { SP_F32_BWD(64) } else { SP_F32_BWD(128) }
#undef SP_F32_BWD
    return hipGetLastError();
}

}  // namespace sp
