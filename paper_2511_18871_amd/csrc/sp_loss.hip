// Response-token loss on the packed sequence (Section 4.3, modification 4: the loss is taken over
// the response tokens only, prompt rows are discarded; Section 2: the GRPO objective
// J = 1/(NG) sum_k (L_k - beta D_KL^k)).
//
//  logprob_fwd  logp[t] = z[t, y_t] - log sum_v exp z[t, v]  for response rows t; prompt rows are
//               neither read nor written.  One workgroup per row, one pass over the row with a
//               running (max, sum) per thread: a pure HBM read of T_resp * V elements.
//  logprob_bwd  dz[t, v] = g_t (1[v = y_t] - exp(z[t, v] - lse_t)); reads z, writes dz.
//  grpo         per response k (one wave): J_k = 1/|o_k| sum_t (min(r A, clip(r) A) - beta kl),
//               r = exp(logp - logp_old), kl = exp(u) - u - 1 with u = logp_ref - logp; writes
//               g[t] = dloss/dlogp[t] and J_k; a single workgroup then sums the J_k in a fixed
//               order (bitwise repeatable) into loss = -1/R sum_k J_k.
#include "sp_common.hpp"
#include "sp_launch.hpp"
#include <type_traits>

namespace sp {
namespace {

template <typename T> struct Ld;
template <> struct Ld<__bf16> { typedef bf16x8 vec; static constexpr int N = 8; };
template <> struct Ld<float> { typedef f32x4 vec; static constexpr int N = 4; };

// Both passes over the logits stream one row per workgroup and are bound by HBM.  A row is cut into the elements ahead
// of its first 16-byte boundary (rows of an odd vocabulary start anywhere), 16-byte vectors, and a tail; a thread has UNROLL
// vectors in flight.  A workgroup has LT threads: 1024 (few rows open at a time) for rows that fill them eight
// times, else 256 or 64.  One box, 2048 rows of 151936 bf16 logits under 1024 prompt rows, forward + backward: 256
// threads 165 + 268 us, 1024 threads 172 + 260, with stores that bypass the caches 98 + 270 (the forward no longer waits
// for the write-back of the gradient before it), with exponents of differences (below) 100 + 270 (6.2 and 5.8 TB/s).  Before: 147 + 396, the gradient filled with zeros first.
constexpr int UNROLL = 2;
template <typename T>
struct RowSplit {
    int head;                   // elements ahead of the first vector
    int64_t vecs, tail0;        // vectors; first element behind them
    __device__ __forceinline__ RowSplit(const T* row, int64_t V) {
        constexpr int N = Ld<T>::N;
        head = (int)(((16 - ((uintptr_t)row & 15)) & 15) / sizeof(T));
        if (head > V) head = (int)V;
        vecs = (V - head) / N;
        tail0 = head + vecs * N;
    }
};

// Running (m, s): the sum of exponentials is s e^m, m the largest element so far.  Differences are taken before they are
// scaled, so that they are exact at any magnitude: scaled apart, the roundings of two products of 1e10 differ by powers of
// two that overflow.  The lowest finite value instead of -inf as the start, so that elements of -inf contribute 0.
constexpr float M_LOWEST = -3.402823466e38f;
__device__ __forceinline__ void ms_merge(float& m, float& s, float m2, float s2) {
    const float mn = fmaxf(m, m2);
    s = s * __expf(m - mn) + s2 * __expf(m2 - mn);
    m = mn;
}

__device__ __forceinline__ void block_lse(float& m, float& s, float* sh) {
    for (int o = 32; o >= 1; o >>= 1) {
        const float m2 = __shfl_xor(m, o, 64), s2 = __shfl_xor(s, o, 64);
        ms_merge(m, s, m2, s2);
    }
    const int w = threadIdx.x >> 6, l = threadIdx.x & 63;
    if (l == 0) { sh[2 * w] = m; sh[2 * w + 1] = s; }
    __syncthreads();
    m = sh[0]; s = sh[1];
    for (int i = 1; i < (int)(blockDim.x >> 6); ++i) ms_merge(m, s, sh[2 * i], sh[2 * i + 1]);
}

template <typename T, int LT>
__global__ __launch_bounds__(LT) void logprob_fwd_kernel(TabArg table, const T* __restrict__ z, const int* __restrict__ y,
                                                         float* __restrict__ logp, float* __restrict__ lse, int64_t V) {
    const int* const tab = table_of(table);
    __shared__ float sh[2 * LT / 64];
    const int64_t tok = blockIdx.x;
    const GroupDesc gd = load_group(tab, find_group_of_token(tab, tok));
    if (tok - gd.tok_base < gd.Lp) return;              // prompt row: discarded
    const T* row = z + tok * V;
    float m = M_LOWEST, s = 0.f;
    constexpr int N = Ld<T>::N;
    typedef typename Ld<T>::vec Vec;
    const RowSplit<T> rs(row, V);
    const Vec* rv = reinterpret_cast<const Vec*>(row + rs.head);
    auto add = [&](auto n_tag, const auto& x) {         // n vectors
        constexpr int n = decltype(n_tag)::value;
        float mx = (float)x[0][0];
#pragma unroll
        for (int u = 0; u < n; ++u)
#pragma unroll
            for (int e = 0; e < N; ++e) mx = fmaxf(mx, (float)x[u][e]);
        const float mn = fmaxf(m, mx);
        float acc = 0.f;
#pragma unroll
        for (int u = 0; u < n; ++u) {
            float part = 0.f;
#pragma unroll
            for (int e = 0; e < N; ++e) part += __expf((float)x[u][e] - mn);
            acc += part;
        }
        s = s * __expf(m - mn) + acc;
        m = mn;
    };
    int64_t i = threadIdx.x;
    for (; i + (UNROLL - 1) * LT < rs.vecs; i += UNROLL * LT) {
        Vec x[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) x[u] = rv[i + u * LT];
        add(std::integral_constant<int, UNROLL>{}, x);
    }
    for (; i < rs.vecs; i += LT) {
        const Vec x[1] = {rv[i]};
        add(std::integral_constant<int, 1>{}, x);
    }
    const int n_loose = rs.head + (int)(V - rs.tail0);       // fewer than 2 N, so one per thread
    if ((int)threadIdx.x < n_loose) {
        const int64_t k = (int)threadIdx.x < rs.head ? threadIdx.x : rs.tail0 + threadIdx.x - rs.head;
        Vec x[1];
        x[0][0] = row[k];
#pragma unroll
        for (int e = 1; e < N; ++e) x[0][e] = (T)-INFINITY;
        add(std::integral_constant<int, 1>{}, x);
    }
    block_lse(m, s, sh);
    if (threadIdx.x == 0) {
        const float L = m + __logf(s);
        const int label = y[tok];
        lse[tok] = L;
        logp[tok] = (label >= 0 && label < V) ? (float)row[label] - L : -INFINITY;
    }
}

// zero_prompt: prompt rows of dz are set to zero (otherwise they are not touched).  Rows are taken last first and each
// from its end: the last 256 MB that the forward read are what the Infinity Cache still holds.
template <typename T, int LT, bool LAST, bool BYPASS>       // LAST: the logits are read past the caches, BYPASS: the gradient is stored past them
__global__ __launch_bounds__(LT) void logprob_bwd_kernel(TabArg table, const T* __restrict__ z, const int* __restrict__ y,
                                                         const float* __restrict__ lse, const float* __restrict__ g,
                                                         T* __restrict__ dz, int64_t V, int zero_prompt) {
    const int* const tab = table_of(table);
    const int64_t tok = (int64_t)gridDim.x - 1 - blockIdx.x;
    const GroupDesc gd = load_group(tab, find_group_of_token(tab, tok));
    constexpr int N = Ld<T>::N;
    typedef typename Ld<T>::vec Vec;
    T* const out = dz + tok * V;
    const RowSplit<T> rs(out, V);
    Vec* const ov = reinterpret_cast<Vec*>(out + rs.head);
    const int n_loose = rs.head + (int)(V - rs.tail0);
    const int64_t loose = (int)threadIdx.x < rs.head ? threadIdx.x : rs.tail0 + threadIdx.x - rs.head;
    auto store = [&](int64_t i, const Vec& d) {
        if constexpr (BYPASS) __builtin_nontemporal_store(d, &ov[i]);
        else ov[i] = d;
    };
    if (tok - gd.tok_base < gd.Lp) {
        if (!zero_prompt) return;
        Vec d;
#pragma unroll
        for (int e = 0; e < N; ++e) d[e] = (T)0.f;
        for (int64_t i = threadIdx.x; i < rs.vecs; i += LT) store(i, d);
        if ((int)threadIdx.x < n_loose) out[loose] = (T)0.f;
        return;
    }
    const T* const row = z + tok * V;                    // starts at the same offset from a 16-byte boundary as `out`
    const Vec* const rv = reinterpret_cast<const Vec*>(row + rs.head);
    const float L = lse[tok], gt = g[tok];
    const int64_t label = y[tok];
    auto vec = [&](int64_t i) -> Vec {
        if constexpr (LAST) return __builtin_nontemporal_load(&rv[i]);
        else return rv[i];
    };
    auto value = [&](T x, int64_t k) { return (T)(gt * ((k == label ? 1.f : 0.f) - __expf((float)x - L))); };
    auto put = [&](const Vec& x, int64_t i) {
        Vec d;
#pragma unroll
        for (int e = 0; e < N; ++e) d[e] = value(x[e], rs.head + i * N + e);
        store(i, d);
    };
    int64_t i = rs.vecs - 1 - threadIdx.x;
    for (; i - (UNROLL - 1) * LT >= 0; i -= UNROLL * LT) {
        Vec x[UNROLL];
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) x[u] = vec(i - u * LT);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) put(x[u], i - u * LT);
    }
    for (; i >= 0; i -= LT) put(vec(i), i);
    if ((int)threadIdx.x < n_loose) out[loose] = value(row[loose], loose);
}

// objective of response k (global index over all groups), one wave; returns J_k in every lane and writes g of its rows
__device__ __forceinline__ float grpo_response(const int* tab, int k, int l, const float* __restrict__ logp, const float* __restrict__ old,
                                               const float* __restrict__ ref, const float* __restrict__ adv,
                                               float* __restrict__ g, float eps_low, float eps_high, float beta, float inv_R) {
    // Group that holds response k.  Group g's response offsets start at table word e[3] = base + R_g + g,
    // with base the first offset word and R_g the responses in earlier groups, so R_g is read off the
    // group entries and the group is the last one with R_g <= k: a bisection (responses of empty groups
    // never match, since R_g of the next group is the same).
    const int ng = tab[0];
    const int base = TAB_HEADER + TAB_GROUP_WORDS * ng;
    int lo = 0, hi = ng;                                 // invariant: R_lo <= k, (hi == ng or R_hi > k)
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (tab[TAB_HEADER + TAB_GROUP_WORDS * mid + 3] - base - mid <= k) lo = mid; else hi = mid;
    }
    const GroupDesc gd = load_group(tab, lo);
    const int i = k - (tab[TAB_HEADER + TAB_GROUP_WORDS * lo + 3] - base - lo);
    const int b = gd.roff[i], e = gd.roff[i + 1];       // group-local token range of the response
    const float a = adv[k];
    const float inv_len = e > b ? 1.0f / (float)(e - b) : 0.f;
    float acc = 0.f;
    for (int t = b + l; t < e; t += 64) {
        const int64_t tok = (int64_t)gd.tok_base + t;
        const float lp = logp[tok];
        const float r = __expf(lp - old[tok]);
        const float un = r * a, cl = fminf(fmaxf(r, 1.0f - eps_low), 1.0f + eps_high) * a;
        const bool inside = r > 1.0f - eps_low && r < 1.0f + eps_high;
        const float surr = fminf(un, cl);
        const float d_surr = (un <= cl || inside) ? un : 0.f;      // d(r a)/dlogp = r a
        const float u = ref[tok] - lp;
        const float eu = __expf(u);
        acc += surr - beta * (eu - u - 1.0f);
        g[tok] = -inv_len * inv_R * (d_surr - beta * (1.0f - eu));
    }
    for (int o = 32; o >= 1; o >>= 1) acc += __shfl_xor(acc, o, 64);
    return acc * inv_len;
}

// One wave per response.  J lies in the workspace, whose tag block is cleared as by every call that writes there.
__global__ __launch_bounds__(256) void grpo_kernel(TabArg table, const float* __restrict__ logp, const float* __restrict__ old,
                                                   const float* __restrict__ ref, const float* __restrict__ adv,
                                                   float* __restrict__ g, float* __restrict__ J, uint32_t* __restrict__ tag,
                                                   int n_resp, float eps_low, float eps_high, float beta, float inv_R) {
    const int k = blockIdx.x * 4 + (threadIdx.x >> 6), l = threadIdx.x & 63;
    if (blockIdx.x == 0 && threadIdx.x < 64) tag[l] = 0u;
    if (k >= n_resp) return;
    const float j = grpo_response(table_of(table), k, l, logp, old, ref, adv, g, eps_low, eps_high, beta, inv_R);
    if (l == 0) J[k] = j;
}

// The same for up to ONE_BLOCK responses, with the sum of grpo_reduce_kernel, in one launch
constexpr int ONE_BLOCK = 16;
__global__ __launch_bounds__(64 * ONE_BLOCK) void grpo_small_kernel(TabArg table, const float* __restrict__ logp, const float* __restrict__ old,
                                                                    const float* __restrict__ ref, const float* __restrict__ adv,
                                                                    float* __restrict__ g, float* __restrict__ loss, int n_resp,
                                                                    float eps_low, float eps_high, float beta, float inv_R) {
    __shared__ float sh[ONE_BLOCK];
    const int k = threadIdx.x >> 6, l = threadIdx.x & 63;
    const float j = k < n_resp ? grpo_response(table_of(table), k, l, logp, old, ref, adv, g, eps_low, eps_high, beta, inv_R) : 0.f;
    if (l == 0) sh[k] = j;
    __syncthreads();
    if (threadIdx.x == 0) {          // the tree of grpo_reduce_kernel over the first ONE_BLOCK elements (the others are zero)
        float x[ONE_BLOCK];
#pragma unroll
        for (int i = 0; i < ONE_BLOCK; ++i) x[i] = sh[i];
#pragma unroll
        for (int o = ONE_BLOCK / 2; o >= 1; o >>= 1)
#pragma unroll
            for (int i = 0; i < o; ++i) x[i] += x[i + o];
        loss[0] = -x[0] * inv_R;
    }
}

// fixed-order sum of J[0..n) by one workgroup: thread i adds J[i], J[i+256], ... then a tree
__global__ __launch_bounds__(256) void grpo_reduce_kernel(const float* __restrict__ J, int n, float inv_R,
                                                          float* __restrict__ loss) {
    __shared__ float sh[256];
    float acc = 0.f;
    for (int i = threadIdx.x; i < n; i += 256) acc += J[i];
    sh[threadIdx.x] = acc;
    __syncthreads();
    for (int o = 128; o >= 1; o >>= 1) {
        if ((int)threadIdx.x < o) sh[threadIdx.x] += sh[threadIdx.x + o];
        __syncthreads();
    }
    if (threadIdx.x == 0) loss[0] = -sh[0] * inv_R;
}

}  // namespace

// calls f(type, workgroup size) for rows of V elements
template <typename F>
void with_row_kernel(int64_t V, bool f32, F f) {
    auto sized = [&](auto elem) {
        const int64_t vecs = V / Ld<decltype(elem)>::N;
        if (vecs >= 4 * UNROLL * 1024) f(elem, std::integral_constant<int, 1024>{});
        else if (vecs >= UNROLL * 256) f(elem, std::integral_constant<int, 256>{});
        else f(elem, std::integral_constant<int, 64>{});
    };
    if (f32) sized(float{}); else sized(__bf16{});
}

hipError_t launch_logprob_fwd(const void* z, const int* y, float* logp, float* lse, const TabArg& tab,
                              int64_t total_tokens, int64_t V, bool f32, hipStream_t s) {
    with_row_kernel(V, f32, [&](auto elem, auto lt) {
        typedef decltype(elem) T;
        hipLaunchKernelGGL((logprob_fwd_kernel<T, decltype(lt)::value>), dim3((unsigned)total_tokens),
                           dim3(decltype(lt)::value), 0, s, tab, (const T*)z, y, logp, lse, V);
    });
    return hipGetLastError();
}

hipError_t launch_logprob_bwd(const void* z, const int* y, const float* lse, const float* g, void* dz,
                              const TabArg& tab, int64_t total_tokens, int64_t V, bool f32, bool zero_prompt, hipStream_t s) {
    // A gradient that the Infinity Cache (256 MB) cannot hold for its reader is stored past the caches, and then the logits, which nothing
    // after this pass reads, are read past them too: what they would displace is the part of them that the forward left.  Not where
    // rows are short and share cache lines, which would be read twice.  Forward, objective and gradient on new buffers, us, cached reads ->
    // not: 275 MB 142 -> 136, 351 MB 196 -> 183, 933 MB 392 -> 385; smaller ones either way: 93 MB 75.3 -> 72.8, 130 MB 99 -> 102, 184 MB
    // 137 -> 143, 249 MB 186 -> 183; 201 MB in rows of 1003 112.5 -> 114.5.
    const int64_t row = V * (f32 ? 4 : 2), bytes = total_tokens * row, cache = (int64_t)256 << 20;
    with_row_kernel(V, f32, [&](auto elem, auto lt) {
        typedef decltype(elem) T;
        constexpr int LT = decltype(lt)::value;
        auto launch = [&](auto last, auto bypass) {
            hipLaunchKernelGGL((logprob_bwd_kernel<T, LT, decltype(last)::value, decltype(bypass)::value>), dim3((unsigned)total_tokens),
                               dim3(LT), 0, s, tab, (const T*)z, y, lse, g, (T*)dz, V, (int)zero_prompt);
        };
        if (bytes <= cache) launch(std::false_type{}, std::false_type{});
        else if (row >= 8192 || row % 128 == 0) launch(std::true_type{}, std::true_type{});
        else launch(std::false_type{}, std::true_type{});
    });
    return hipGetLastError();
}

hipError_t launch_grpo(const float* logp, const float* old, const float* ref, const float* adv, float* g,
                       float* J, float* loss, const TabArg& tab, uint32_t* tag, int n_resp, int n_nonempty,
                       float eps_low, float eps_high, float beta, hipStream_t s) {
    const float inv_R = n_nonempty > 0 ? 1.0f / (float)n_nonempty : 0.f;
    if (n_resp <= ONE_BLOCK) {
        hipLaunchKernelGGL(grpo_small_kernel, dim3(1), dim3(64 * ONE_BLOCK), 0, s, tab, logp, old, ref, adv, g, loss, n_resp,
                           eps_low, eps_high, beta, inv_R);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(grpo_kernel, dim3((n_resp + 3) / 4), dim3(256), 0, s, tab, logp, old, ref, adv, g, J, tag, n_resp,
                       eps_low, eps_high, beta, inv_R);
    hipLaunchKernelGGL(grpo_reduce_kernel, dim3(1), dim3(256), 0, s, J, n_resp, inv_R, loss);
    return hipGetLastError();
}

}  // namespace sp
