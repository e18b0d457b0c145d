// What the dense kernels share: operand fix-ups and the epilogues.
#pragma once
#include "accerl_internal.h"

namespace accerl {

// bf16 dense layers of this many MFMA steps or more sum K in this many parts: part i is the steps i * k_steps / PARTS up to
// (i + 1) * k_steps / PARTS in order from zero, and the parts are added to the bias in order
constexpr int KSPLIT_PARTS = 8;

__device__ __forceinline__ uint32_t g_relu_i8x4(uint32_t x) {
    const uint32_t neg = (x & 0x80808080u) >> 7;
    return x & ~(neg * 0xffu);
}
__device__ __forceinline__ uint32_t g_relu_bf16x2(uint32_t x) {
    const uint32_t neg = (x & 0x80008000u) >> 15;
    return x & ~(neg * 0xffffu);
}
__device__ __forceinline__ uint32_t g_f2bf(float x) {
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7fffffffu) > 0x7f800000u) return u >> 16;
    u += 0x7fffu + ((u >> 16) & 1u);
    return u >> 16;
}
__device__ __forceinline__ float g_sigmoid(float x) { return 1.0f / (1.0f + expf(-x)); }


// The tile of a workgroup: x of the states, y of the features.  Workgroup n runs on XCD n mod 8.  by_xcd: every XCD takes consecutive
// tiles, all features of one group of states before the next group, so that a group's states come into one second-level cache
// (the kernels' launch functions say when).
struct GemmTile { unsigned x, y; };
// BRANCH: a branch around the division (kernels that divide by the grid's height anyway share its reciprocal instead: with the branch they
// waited for two scalar loads and two reciprocals in a row, 0.25 us).
template <bool BRANCH>
__device__ __forceinline__ GemmTile gemm_tile(int by_xcd) {
    if (BRANCH && !by_xcd) return {blockIdx.x, blockIdx.y};
    const unsigned n = gridDim.x * gridDim.y, id = blockIdx.y * gridDim.x + blockIdx.x, xcd = id & 7;
    const unsigned t = xcd * (n >> 3) + min(xcd, n & 7) + (id >> 3);     // the first n mod 8 XCDs have one tile more
    const unsigned x = t / gridDim.y, y = t - x * gridDim.y;
    return {by_xcd ? x : blockIdx.x, by_xcd ? y : blockIdx.y};
}

// 16-byte piece of inputs k .. k + 7 (k a multiple of 8) of state b in the LSTM operand's fragment order
__device__ __forceinline__ char* lstm_piece(const GemmParams& p, int64_t b, int k) {
    return (char*)p.xh + ((((b >> 4) * p.xh_ks + (k >> 5)) << 6) + ((k >> 3) & 3) * 16 + (b & 15)) * 16;
}
typedef int v2i __attribute__((ext_vector_type(2)));
__device__ __forceinline__ v2i lstm_pack4(const float (&v)[4]) {
    return (v2i){(int)(g_f2bf(v[0]) | (g_f2bf(v[1]) << 16)), (int)(g_f2bf(v[2]) | (g_f2bf(v[3]) << 16))};
}

// Results of features n0 .. n0 + 3 of state b (sums with the bias): requantized int8, bf16, head outputs or the LSTM cell.
// XH: to the LSTM's operand instead (the values lstm_pack_frag_kernel makes of the stored ones).
template <int EPI, bool XH = false, typename ACC>
__device__ __forceinline__ void gemm_finish(const GemmParams& p, const ACC& acc, int64_t b, int n0) {
    if constexpr (EPI == EPI_REQUANT) {
        const v4f ml = *(const v4f*)(p.mult + n0);
        uint32_t pk = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int v = acc[r];
            if (p.tap_acc && n0 + r < p.N) p.tap_acc[b * p.N + n0 + r] = v;
            if (p.relu) {   // clamp(rint(y), 0, 127): the pack instruction rounds to nearest even, saturates at 0
                pk = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_fmed3f((float)v * ml[r], 0.0f, 127.0f), r, pk);
            } else {
                const float y = __builtin_amdgcn_fmed3f(rintf((float)v * ml[r]), -127.0f, 127.0f);
                pk |= ((uint32_t)(int)y & 0xffu) << (8 * r);
            }
        }
        if constexpr (XH) {
            float v[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int q = (int)(int8_t)(pk >> (8 * r));
                v[r] = (float)(p.xh_relu ? max(q, 0) : q) * p.xh_scale;
            }
            *(v2i*)(lstm_piece(p, b, n0) + 2 * (n0 & 4)) = lstm_pack4(v);
        } else {
            *(uint32_t*)((int8_t*)p.out + b * p.Np + n0) = pk;
        }
    } else if constexpr (EPI == EPI_HEADS_I8) {
        const v4f ml = *(const v4f*)(p.mult + n0);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int n = n0 + r;
            if (n > p.A) continue;
            const int v = acc[r];
            if (p.tap_acc) p.tap_acc[b * (p.A + 1) + n] = v;
            const float o = (float)v * ml[r];
            if (p.logits) { if (n < p.A) p.logits[b * p.A + n] = o; else p.value[b] = o; }
        }
    } else if constexpr (EPI == EPI_BF16) {
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            v[r] = acc[r];
            if (p.relu) v[r] = fmaxf(v[r], 0.0f);
        }
        if constexpr (XH) {
            if (p.xh_relu) {
#pragma unroll
                for (int r = 0; r < 4; ++r) v[r] = fmaxf(__uint_as_float(g_f2bf(v[r]) << 16), 0.0f);
            }
            *(v2i*)(lstm_piece(p, b, n0) + 2 * (n0 & 4)) = lstm_pack4(v);
            return;
        }
        uint32_t* d = (uint32_t*)((uint16_t*)p.out + b * p.Np + n0);
        d[0] = g_f2bf(v[0]) | (g_f2bf(v[1]) << 16);
        d[1] = g_f2bf(v[2]) | (g_f2bf(v[3]) << 16);
    } else if constexpr (EPI == EPI_HEADS_F32ACC) {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int n = n0 + r;
            if (n > p.A) continue;
            const float o = acc[r];
            if (p.logits) { if (n < p.A) p.logits[b * p.A + n] = o; else p.value[b] = o; }
        }
    } else {   // EPI_LSTM: rows 4*unit + {i,f,g,o}
        const int unit = n0 >> 2;
        const float pi = acc[0], pf = acc[1];
        const float pg = acc[2], po = acc[3];
        const float si = g_sigmoid(pi), sf = g_sigmoid(pf), tg = tanhf(pg), so = g_sigmoid(po);
        const float c_old = p.c[b * p.Hd + unit];
        const float t1 = sf * c_old;
        const float t2 = si * tg;
        const float cn = t1 + t2;
        const float hn = so * tanhf(cn);
        p.c[b * p.Hd + unit] = cn;
        p.h[b * p.Hd + unit] = hn;
        ((uint16_t*)p.out)[b * p.Np + unit] = (uint16_t)g_f2bf(hn);   // bf16 copy for the heads
    }
}

}  // namespace accerl
