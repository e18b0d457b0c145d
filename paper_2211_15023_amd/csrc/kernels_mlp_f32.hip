// fp32 MLP teacher (dense chain + heads + sampler) in one kernel on v_mfma_f32_16x16x4_f32.
//
// A workgroup of four wavefronts owns 16 * ST states for the whole network.  Output units are the MFMA rows, states the
// columns: a lane's accumulator is four consecutive units of one state, which is one 16-byte chunk of the next layer's
// operand, so activations go through LDS as whole chunks [unit tile of 16][state tile][lane][16 B] (no bank conflicts,
// written and read at consecutive addresses).  Unit tile t of a layer belongs to wavefront t % 4; weights come straight
// from memory (the second-level cache: all workgroups read the same ones) in fragments [K block of 16][unit tile][lane]
// [16 B], each of which feeds 4 * ST MFMAs.  The K order inside a block is (lane group, element) on both operands.
// The heads multiply the last layer's accumulators where they are (a wavefront's own units are a slice of K) and the four
// partial sums meet in LDS.
//
// What bounds it: the fp32 matrix rate (157 TFLOP/s nominal).  The layer-by-layer kernel issued one vector multiply-add
// per product (half that rate at best), read LDS once per eight products and needed four launches: 24-256-256-4 at 8192
// states 84.5 -> 15.5 us per call (77 TFLOP/s; 7.6 us at the matrix rate, the rest is launch, the first weights and the
// heads); error against float64 3.0e-7 -> 2.3e-7 (2-norm).
#include <algorithm>

#include "accerl_internal.h"

namespace accerl {

namespace {

// NT = unit tiles per wavefront (layers of at most 64 * NT units), ST = state tiles per workgroup
template <int NT, int ST>
__global__ __launch_bounds__(256, 2) void mlp_f32_kernel(const MlpF32Params p) {
    constexpr int UT = 4 * NT;                                 // unit tiles of a hidden layer
    __shared__ __attribute__((aligned(16))) v4f s_act[UT * ST * 64];
    __shared__ float s_head[4][16 * ST][17];                   // one head tile: partial sums of the four wavefronts
    __shared__ float s_logit[16 * ST][65];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    const int64_t b0 = (int64_t)blockIdx.x * (16 * ST);

    v4f acc[NT][ST], w[4][NT];
    const v4f* wp = p.wfrag + wave * 64 + lane;                // fragment (block, tile i) of this wavefront: wp[(block * UT + 4 * i) * 64]
    auto load_w = [&](int slot, const v4f* at) {
#pragma unroll
        for (int i = 0; i < NT; ++i) w[slot][i] = at[4 * i * 64];
    };
    auto mul = [&](int slot, int kb) {
        v4f x[ST];
#pragma unroll
        for (int s = 0; s < ST; ++s) x[s] = s_act[(kb * ST + s) * 64 + lane];
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int i = 0; i < NT; ++i)
#pragma unroll
                for (int s = 0; s < ST; ++s) acc[i][s] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[slot][i][e], x[s][e], acc[i][s], 0, 0, 0);
    };
    auto clear = [&]() {
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int s = 0; s < ST; ++s) acc[i][s] = (v4f){0.f, 0.f, 0.f, 0.f};
    };
    // bias and ReLU; units past the layer's width become zeros whatever the inputs were (0 * inf)
    auto finish = [&](int l) {
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const int n0 = 16 * (wave + 4 * i) + 4 * g;
            const v4f b = *(const v4f*)(p.bias + l * 64 * NT + n0);
#pragma unroll
            for (int s = 0; s < ST; ++s)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    float v = acc[i][s][r] + b[r];
                    if (p.relu[l]) v = fmaxf(v, 0.0f);
                    acc[i][s][r] = n0 + r < p.N[l] ? v : 0.0f;
                }
        }
    };

    // ---- observations to LDS, zero past their width and past the batch; an even number of K blocks
    const int kb0 = p.kb0;
    load_w(0, wp);
    load_w(1, wp + UT * 64);
    for (int u = tid; u < kb0 * ST * 64; u += 256) {
        const int t = u >> 6, ln = u & 63;
        const int kb = t / ST, s = t - kb * ST;
        const int64_t b = b0 + 16 * s + (ln & 15);
        const int k0 = 16 * kb + 4 * (ln >> 4);
        const float* src = p.obs + (b < p.B ? b : p.B - 1) * p.D;
        v4f v;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float t4 = src[k0 + e < p.D ? k0 + e : p.D - 1];
            v[e] = (b < p.B && k0 + e < p.D) ? t4 : 0.0f;
        }
        s_act[u] = v;
    }
    clear();
    __syncthreads();
    for (int kb = 0; kb < kb0; kb += 2) {
        const bool more = kb + 2 < kb0;
        wp += 2 * UT * 64;
        mul(0, kb);
        if (more) load_w(0, wp);
        mul(1, kb + 1);
        if (more) load_w(1, wp + UT * 64);
    }
    // ---- further hidden layers: 64 * NT inputs each, four blocks in flight across the layers (the planner pads the end)
#pragma unroll
    for (int q = 0; q < 4; ++q) load_w(q, wp + q * UT * 64);
    for (int l = 1; l < p.n_hidden; ++l) {
        finish(l - 1);
        __syncthreads();                                       // every wavefront has read the layer's inputs
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int s = 0; s < ST; ++s) s_act[((wave + 4 * i) * ST + s) * 64 + lane] = acc[i][s];
        clear();
        __syncthreads();
        for (int kb = 0; kb < UT; kb += 4) {
            wp += 4 * UT * 64;
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                mul(q, kb + q);
                load_w(q, wp + q * UT * 64);
            }
        }
    }
    finish(p.n_hidden - 1);

    // ---- heads, one tile of 16 outputs at a time; this wavefront's slice of K is its own units
    const int n_out = p.A + 1;
    for (int h = 0; 16 * h < n_out; ++h) {
        v4f hw[NT], part[ST];
#pragma unroll
        for (int i = 0; i < NT; ++i) hw[i] = p.whead[(h * UT + wave + 4 * i) * 64 + lane];
#pragma unroll
        for (int s = 0; s < ST; ++s) part[s] = (v4f){0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int i = 0; i < NT; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int s = 0; s < ST; ++s) part[s] = __builtin_amdgcn_mfma_f32_16x16x4f32(hw[i][e], acc[i][s][e], part[s], 0, 0, 0);
        if (h) __syncthreads();                                // the tile before has been folded
#pragma unroll
        for (int s = 0; s < ST; ++s)
#pragma unroll
            for (int r = 0; r < 4; ++r) s_head[wave][16 * s + j][4 * g + r] = part[s][r];
        __syncthreads();
        for (int u = tid; u < 256 * ST; u += 256) {
            const int st = u >> 4, o = u & 15, n = 16 * h + o;
            if (n >= n_out) continue;
            const float v = ((s_head[0][st][o] + s_head[1][st][o]) + (s_head[2][st][o] + s_head[3][st][o])) + p.bhead[n];
            s_logit[st][n] = v;
            if (b0 + st < p.B) { if (n < p.A) p.logits[(b0 + st) * p.A + n] = v; else p.value[b0 + st] = v; }
        }
    }
    __syncthreads();
    // ---- sampler: one lane per state, the arithmetic of sample_kernel
    if (tid < 16 * ST && b0 + tid < p.B) {
        const float* lg = s_logit[tid];
        float m = lg[0];
        for (int a = 1; a < p.A; ++a) m = fmaxf(m, lg[a]);
        float Z = 0.0f;
        for (int a = 0; a < p.A; ++a) Z += expf(lg[a] - m);
        const float thr = p.uniforms[b0 + tid] * Z;
        float cum = 0.0f;
        int act = p.A - 1;
        for (int a = 0; a < p.A; ++a) {
            cum += expf(lg[a] - m);
            if (cum > thr) { act = a; break; }
        }
        p.action[b0 + tid] = act;
    }
}

// one launch takes 2^28 or 2^29 states less a workgroup's; a larger batch goes out in pieces
template <int NT, int ST>
hipError_t go(MlpF32Params p, hipStream_t s) {
    constexpr int64_t most = MAX_LAUNCH_ITEMS / 256 * (16 * ST);
    for (int64_t left = p.B; left > 0; left -= most) {
        p.B = std::min(left, most);
        mlp_f32_kernel<NT, ST><<<dim3((unsigned)((p.B + 16 * ST - 1) / (16 * ST))), dim3(256), 0, s>>>(p);
        if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
        p.obs += p.B * p.D; p.uniforms += p.B;
        p.logits += p.B * p.A; p.value += p.B; p.action += p.B;
    }
    return hipSuccess;
}

}  // namespace

hipError_t launch_mlp_f32(const MlpF32Params& p, hipStream_t s) {
    if (p.B <= 0) return hipSuccess;
    if (p.n_hidden < 1 || p.n_hidden > MLP_F32_MAX_LAYERS || p.kb0 < 2 || (p.kb0 & 1) || p.kb0 > 4 * p.nt) return hipErrorInvalidValue;
    // 32 states per workgroup halve the weight traffic, but leave compute units empty or with one workgroup where 16 would give
    // each of them more.  us with 16 / 32: 24-256-256-4 at 4096 states 11.4 / 15.6, 4100 15.8 / 15.5, 8192 17.0 / 16.0, 65536
    // 104 / 90; two layers of 128 at 8192 8.4 / 8.8, four of them 13.8 / 14.3, 16384 12.4 / 12.2 and 22.8 / 21.8, 65536 37.4 / 35.1
    // and 76.8 / 69.6; two layers of 64 at 8192 6.0 / 6.4, 16384 7.7 / 7.6, 65536 18.2 / 19.3.
    switch (p.nt) {
        case 1: return go<1, 1>(p, s);
        case 2: return p.B > 8192 ? go<2, 2>(p, s) : go<2, 1>(p, s);
        case 4: return p.B > 4096 ? go<4, 2>(p, s) : go<4, 1>(p, s);
    }
    return hipErrorInvalidValue;
}

}  // namespace accerl
