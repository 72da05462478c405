// Rotary position embedding with the shared-prompt position indices (Section 4.3,
// modification 2): the prompt keeps positions 0 .. Lp-1 and every response starts again at Lp,
// so a response token is rotated as it would be if [prompt | resp_i] were a sample of its own.
// Half-split form: with theta_i = base^(-2i/d), pair (x_i, x_{i+d/2}) at position p turns by the
// angle p * theta_i.  The rotation is orthogonal; `inverse` turns by the negative angle, which
// maps gradients with respect to rotated q / k back to gradients with respect to q / k.
//
// The kernel is a pure HBM pass (read x, write y).  The frequencies theta_i come from the host in double precision (a
// kernel argument), the product p * theta_i is formed and reduced to [-pi, pi] in double (positions reach tens of thousands
// of radians, where an fp32 product is already off by 1e-3), and only the reduced angle goes through the fp32 sine and
// cosine.  The same angles then serve every head of the token -- of one tensor, or of q AND k in one
// launch (sp_attn_rope_qk): one table lookup, one position and one set of angles for both.
#include "sp_common.hpp"
#include "sp_launch.hpp"
#include <cmath>
#include <type_traits>

namespace sp {
namespace {

template <typename T> struct Vec8;
template <> struct Vec8<__bf16> { typedef bf16x8 type; };
template <> struct Vec8<float> { typedef float type __attribute__((ext_vector_type(8))); };

struct RopeFreq { double theta[64]; };      // theta_i = base^(-2 i / d), i < d / 2 <= 64

// Bound: HBM.  A workgroup takes 512 / D tokens, so that each of its 256 threads evaluates one angle (they are exchanged
// through LDS).  D / 16 lanes hold a head's pairs, 8 of each half as 16-byte pieces (bf16), and the next lanes the next heads:
// a wave's two loads cover whole heads that lie in one piece.  The rows do not wait for the positions: the first
// UNROLL of them per lane are loaded ahead of the lookups, past the caches (each is read once).  One thread per eight
// pairs of a token, a head at a time, left most of the chip waiting for single loads: 16K prompt and 32 answers, 40 + 8 heads (528 MB),
// 109.4 -> 98.1 us (4.8 -> 5.4 TB/s), with six rows in flight instead of three 96.0, with loads past the caches 93.0, stores too 86.6
// (6.1 TB/s); 2048 tokens of 32 + 8 heads 24.5 -> 11.4.
template <typename T, int D, bool BYPASS>
__global__ __launch_bounds__(256) void rope_kernel(TabArg table, const T* __restrict__ x, T* __restrict__ y, int H,
                                                   const T* __restrict__ x2, T* __restrict__ y2, int H2,
                                                   RopeFreq f, int inverse) {
    const int* const tab = table_of(table);
    typedef typename Vec8<T>::type V8;
    constexpr int HALF = D / 2, TOKENS = 256 / HALF, LANES = D / 16, UNROLL = 6;
    __shared__ float cs[TOKENS][HALF], sn[TOKENS][HALF];
    const int64_t T_total = tab[1];
    const int i0 = 8 * ((int)threadIdx.x % LANES), hg = (int)threadIdx.x / LANES % 8, tb = (int)threadIdx.x / HALF;
    static_assert(LANES * 8 == HALF, "a token's threads are those that evaluate its angles");
    const int64_t tok = (int64_t)blockIdx.x * TOKENS + (HALF == 64 ? __builtin_amdgcn_readfirstlane(tb) : tb);
    const bool valid = tok < T_total;
    const int64_t row1 = tok * H * D + i0, row2 = tok * H2 * D + i0;
    auto at = [&](int h) { return h < H ? row1 + (int64_t)h * D : row2 + (int64_t)(h - H) * D; };
    V8 lo[UNROLL], hi[UNROLL];
    auto load = [&](int h0) {
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int h = h0 + 8 * u;
            if (!valid || h >= H + H2) continue;
            const T* const p = (h < H ? x : x2) + at(h);
            lo[u] = __builtin_nontemporal_load(reinterpret_cast<const V8*>(p));
            hi[u] = __builtin_nontemporal_load(reinterpret_cast<const V8*>(p + HALF));
        }
    };
    load(hg);
    if (valid) {       // the angle of this thread: pair i of its token
        const int i = (int)threadIdx.x % HALF;
        const GroupDesc gd = load_group(tab, find_group_of_token(tab, tok));
        const int t = (int)(tok - gd.tok_base);
        const int pos = t < gd.Lp ? t : gd.Lp + (t - seg_start(gd, t));
        const double ang = (double)pos * f.theta[i];
        const double red = ang - 6.283185307179586476925 * rint(ang * 0.15915494309189533577);   // into [-pi, pi]
        float sv, cv;
        sincosf((float)red, &sv, &cv);
        cs[tb][i] = cv;
        sn[tb][i] = inverse ? -sv : sv;
    }
    __syncthreads();
    if (!valid) return;
    float c[8], s[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) { c[e] = cs[tb][i0 + e]; s[e] = sn[tb][i0 + e]; }
    for (int h0 = hg; h0 < H + H2; h0 += 8 * UNROLL) {
        if (h0 != hg) load(h0);
#pragma unroll
        for (int u = 0; u < UNROLL; ++u) {
            const int h = h0 + 8 * u;
            if (h >= H + H2) continue;
            V8 ylo, yhi;
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float a = (float)lo[u][e], b = (float)hi[u][e];
                ylo[e] = (T)(a * c[e] - b * s[e]);
                yhi[e] = (T)(a * s[e] + b * c[e]);
            }
            T* const p = (h < H ? y : y2) + at(h);
            if constexpr (BYPASS) {
                __builtin_nontemporal_store(ylo, reinterpret_cast<V8*>(p));
                __builtin_nontemporal_store(yhi, reinterpret_cast<V8*>(p + HALF));
            } else {
                *reinterpret_cast<V8*>(p) = ylo;
                *reinterpret_cast<V8*>(p + HALF) = yhi;
            }
        }
    }
}

}  // namespace

hipError_t launch_rope(const void* x, void* y, int H, const void* x2, void* y2, int H2, const TabArg& tab,
                       int64_t total_tokens, int d, double base, bool inverse, bool f32, hipStream_t s) {
    RopeFreq f{};
    for (int i = 0; i < d / 2; ++i) f.theta[i] = pow(base, -2.0 * (double)i / (double)d);
    const unsigned grid = (unsigned)((total_tokens + 512 / d - 1) / (512 / d));
    // Outputs that (nearly) fill the Infinity Cache (256 MB) are stored past the caches.  us, cached -> not, 40 heads.  Outputs in
    // four buffers in turn, as those of a model's layers: 210 MB 73.9 -> 70.7, 252 MB 88.0 -> 84.0, 336 MB 118 -> 111; with a forward of short groups
    // behind, which reads them, 219 -> 221, 261 -> 262, 338 -> 335.  The line is where the pass gains more than its reader loses; a
    // buffer that is written again and again stays in the cache and would have it at 300 MB (210 MB 63 -> 70, 252 MB 75 -> 84, 336 MB 117 -> 111).
    const bool bypass = total_tokens * (H + (x2 ? H2 : 0)) * d * (f32 ? 4 : 2) > (int64_t)240 << 20;
    auto launch = [&](auto elem, auto dim, auto past) {
        typedef decltype(elem) T;
        hipLaunchKernelGGL((rope_kernel<T, decltype(dim)::value, decltype(past)::value>), dim3(grid), dim3(256), 0, s, tab,
                           (const T*)x, (T*)y, H, (const T*)x2, (T*)y2, x2 ? H2 : 0, f, (int)inverse);
    };
    auto with_d = [&](auto elem, auto past) {
        if (d == 64) launch(elem, std::integral_constant<int, 64>{}, past);
        else launch(elem, std::integral_constant<int, 128>{}, past);
    };
    auto with_t = [&](auto past) { if (f32) with_d(float{}, past); else with_d(__bf16{}, past); };
    if (bypass) with_t(std::true_type{}); else with_t(std::false_type{});
    return hipGetLastError();
}

}  // namespace sp
