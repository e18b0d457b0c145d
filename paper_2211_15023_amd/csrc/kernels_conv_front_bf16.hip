// The first two convolutions of the paper's original network (32 filters of 8x8 stride 4, 64 of 4x4 stride 2, no padding,
// on a 4x84x84 uint8 observation) for the bf16 teacher, as one pipelined kernel with every size known at compile time.
//
// A workgroup of eight wavefronts (one per compute unit, two per SIMD) walks over observations.  In one tick wavefronts
// 4..7 compute the first convolution of observation n+1 from its bf16 copy in LDS and write the 20x20x32 image to LDS,
// wavefronts 0..3 compute the second convolution of observation n from the image written in the tick before, and the bytes
// of observation n+2 are in flight; then the first-layer wavefronts convert those bytes to bf16 (v / 255) into LDS while the
// second-layer wavefronts finish their last two tiles.  The first layer's output never leaves the chip.
//
//  * Weights stay in registers: 8 K steps x 2 channel tiles for the first layer (64), 16 x 2 for one half of the second
//    layer's filters (128).
//  * Observation copy.  A unit is 4 horizontally adjacent pixels of all four planes; its 16 values are two chunks, channels
//    0, 1 and channels 2, 3, each [channel][pixel] as the plane's bytes arrive, and the two kinds of chunk lie in planes of
//    their own.  A K step of the first layer is one kernel row: lane group g reads chunk kind g & 1 of unit ox + g / 2, so 16
//    pixels of an output row are 256 consecutive bytes.  The weight fragments are brought to that order once.
//  * The first 16 output columns are tiled by output rows, five in a row per wavefront: rows 4..7 of a window are rows 0..3
//    of the window below, so a tile fetches four of its eight fragments; the other 4 columns are five 4 x 4 tiles.
//  * First-layer image: [8 channels][column parity][row][column / 2][16 B], rows of 12 columns: the stride-2 second layer
//    reads consecutive chunks, and the second of two output rows starts 128 bytes further round the banks.
//  * The second layer's 81 pixels are the tiles 0..47 and 33..80; the overlap is stored twice with the same bytes.
//
// What bounds it: LDS (410 KB per observation) and the matrix cores (784 MFMAs per observation, 3 136 clocks per SIMD) about
// equally.
#include "conv_kernel.h"

namespace accerl {

namespace {

constexpr int FB_THREADS = 512, FB_STAGERS = 256;
constexpr int FB_PLANE_IN = 84 * 84;                     // bytes of a channel plane of the observation
constexpr int FB_UNITS = FB_PLANE_IN / 4;                // 1764
constexpr int FB_PF = (FB_UNITS + FB_STAGERS - 1) / FB_STAGERS;   // 7
constexpr int FB_ROW_A = 21 * 16, FB_KIND_A = FB_UNITS * 16, FB_TILE_A = 2 * FB_KIND_A;
constexpr int FB_ROW_B = 12 * 16, FB_PAR_B = 20 * FB_ROW_B + 128, FB_CH_B = 2 * FB_PAR_B, FB_TILE_B = 4 * FB_CH_B;
constexpr int FB_LDS = FB_TILE_A + 2 * FB_TILE_B;
constexpr int FB_NPIX2 = 81, FB_PIX2_BYTES = 128;

struct FrontBParams {
    const uint8_t* obs;      // [B, 4, 84, 84]
    char* out;               // bf16 [B, 9, 9, 64]
    const v4i* wA; const float* biasA;
    const v4i* wB; const float* biasB;
    int64_t B;
};

__device__ __forceinline__ v4f fb_mfma(v4i a, v4i b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}
__device__ __forceinline__ int fb_pack2(float a, float b) {
    typedef float v2f __attribute__((ext_vector_type(2)));
    typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(int, __builtin_convertvector((v2f){a, b}, v2bf));
}
// ReLU of eight accumulators (consecutive channels) as bf16: a negative bf16 is a negative 16-bit integer
__device__ __forceinline__ v4i fb_relu_pack(v4f a, v4f b) {
    typedef short v8s __attribute__((ext_vector_type(8)));
    const v8s z = {0, 0, 0, 0, 0, 0, 0, 0};
    const v4i v = {fb_pack2(a[0], a[1]), fb_pack2(a[2], a[3]), fb_pack2(b[0], b[1]), fb_pack2(b[2], b[3])};
    return __builtin_bit_cast(v4i, __builtin_elementwise_max(__builtin_bit_cast(v8s, v), z));
}
// bf16(v / 255) of two bytes of a dword
template <int LO>
__device__ __forceinline__ int fb_obs2(uint32_t d) {
    constexpr float k = 1.0f / 255.0f;
    return fb_pack2((float)((d >> (8 * LO)) & 0xffu) * k, (float)((d >> (8 * LO + 8)) & 0xffu) * k);
}

__global__ __launch_bounds__(FB_THREADS, 2) void conv_front_bf16_kernel(const FrontBParams p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    char* tileA = smem;
    char* tilesB = smem + FB_TILE_A;
    const int64_t stride = gridDim.x;
    int64_t img = blockIdx.x;                            // the observation whose second convolution runs this tick
    if (img >= p.B) return;

    if (wave >= 4) {
        const int aw = wave - 4, stid = tid - FB_STAGERS;
        uint32_t pre[FB_PF][4];
        auto obs_of = [&](int64_t im) { return p.obs + min(im, p.B - 1) * (int64_t)(4 * FB_PLANE_IN); };   // past the batch: the last observation, never used
        auto stage_load_part = [&](const uint8_t* src, int k) {
            const int u = min(stid + k * FB_STAGERS, FB_UNITS - 1);
#pragma unroll
            for (int c = 0; c < 4; ++c) pre[k][c] = *(const uint32_t*)(src + c * FB_PLANE_IN + 4 * u);
        };
        auto stage_commit = [&]() {
#pragma unroll
            for (int k = 0; k < FB_PF; ++k) {
                const int u = stid + k * FB_STAGERS;
                if (u < FB_UNITS) {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        *(v4i*)(tileA + h * FB_KIND_A + 16 * u) = (v4i){fb_obs2<0>(pre[k][2 * h]), fb_obs2<2>(pre[k][2 * h]),
                                                                         fb_obs2<0>(pre[k][2 * h + 1]), fb_obs2<2>(pre[k][2 * h + 1])};
                }
            }
        };
#pragma unroll
        for (int k = 0; k < FB_PF; ++k) stage_load_part(obs_of(img), k);
        // The planner's chunk q of a kernel row is pixels 2q, 2q+1 x channels 0..3.  Lane group g needs channels 2 (g & 1) and
        // + 1 of pixels 4 (g / 2) .. + 3: dwords (g & 1), 2 + (g & 1) of chunks 2 (g / 2) and + 1, low halves then high halves.
        v4i wA[8][2];
#pragma unroll
        for (int st = 0; st < 8; ++st)
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                const v4i* src = p.wA + (st * 2 + t) * 64 + j + 32 * (g >> 1);
                const v4i a = src[0], b = src[16];
                const uint32_t a0 = (uint32_t)(g & 1 ? a[1] : a[0]), a1 = (uint32_t)(g & 1 ? a[3] : a[2]);
                const uint32_t b0 = (uint32_t)(g & 1 ? b[1] : b[0]), b1 = (uint32_t)(g & 1 ? b[3] : b[2]);
                wA[st][t] = (v4i){(int)__builtin_amdgcn_perm(a1, a0, 0x05040100u), (int)__builtin_amdgcn_perm(b1, b0, 0x05040100u),
                                  (int)__builtin_amdgcn_perm(a1, a0, 0x07060302u), (int)__builtin_amdgcn_perm(b1, b0, 0x07060302u)};
            }
        const v4f bi0 = *(const v4f*)(p.biasA + 8 * g), bi1 = *(const v4f*)(p.biasA + 8 * g + 4);

        // chain tiles: output row 5 aw + r, column j; then the 4 x 4 tiles aw and (first wavefront only) 4
        const int lane_in = (g >> 1) * 16 + (g & 1) * FB_KIND_A;
        const int rb_chain = (5 * aw) * (4 * FB_ROW_A) + j * 16 + lane_in;
        const int wb_chain = g * FB_CH_B + (j & 1) * FB_PAR_B + (5 * aw) * FB_ROW_B + (j >> 1) * 16;
        int rb_blk[2], wb_blk[2];
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int b = k == 0 ? aw : 4, oy = 4 * b + (j >> 2), ox = 16 + (j & 3);
            rb_blk[k] = oy * (4 * FB_ROW_A) + ox * 16 + lane_in;
            wb_blk[k] = g * FB_CH_B + (ox & 1) * FB_PAR_B + oy * FB_ROW_B + (ox >> 1) * 16;
        }
        auto frag_a = [&](int r, int st) {
            const int base = r < 5 ? rb_chain + r * (4 * FB_ROW_A) : rb_blk[r - 5];
            return *(const v4i*)(tileA + base + st * FB_ROW_A);
        };
        auto store_a = [&](char* dstB, int r, v4f a, v4f b) {
            *(v4i*)(dstB + (r < 5 ? wb_chain + r * FB_ROW_B : wb_blk[r - 5])) = fb_relu_pack(a, b);
        };
        // One tile = 16 MFMAs; the fragments of the next tile are requested and the tile before is packed and stored meanwhile,
        // and the bytes of observation `next` are requested, one unit per tile.
        auto conv_a = [&](char* dstB, const uint8_t* next) {
            v4i f[8];
#pragma unroll
            for (int st = 0; st < 8; ++st) f[st] = frag_a(0, st);
            v4f o0 = bi0, o1 = bi1;
#pragma unroll
            for (int r = 0; r < 7; ++r) {
                if (r == 6 && aw != 0) break;            // the fifth 4 x 4 tile
                v4f n0 = bi0, n1 = bi1;
                v4i fn[8];
                stage_load_part(next, r);
#pragma unroll
                for (int st = 0; st < 8; ++st) {
                    n0 = fb_mfma(wA[st][0], f[st], n0);
                    n1 = fb_mfma(wA[st][1], f[st], n1);
                    if (r + 1 < 5) fn[st] = st < 4 ? f[st + 4] : frag_a(r + 1, st);
                    else if (r + 1 < 7) fn[st] = frag_a(r + 1, st);     // (tile 6 is read by every wavefront: one copy of the code)
                }
                if (r > 0) store_a(dstB, r - 1, o0, o1);
                o0 = n0; o1 = n1;
#pragma unroll
                for (int st = 0; st < 8; ++st) f[st] = fn[st];
            }
            if (aw != 0) stage_load_part(next, 6);
            store_a(dstB, aw == 0 ? 6 : 5, o0, o1);
        };

        stage_commit();
        __syncthreads();                                 // observation copy complete
        conv_a(tilesB, obs_of(img + stride));
        __syncthreads();                                 // first image complete, observation copy free
        if (img + stride < p.B) stage_commit();
        __syncthreads();
        for (int n = 0;; ++n, img += stride) {
            if (!(img + stride < p.B)) break;            // the workgroup's observations are done (same test in every wavefront)
            conv_a(tilesB + ((n + 1) & 1) * FB_TILE_B, obs_of(img + 2 * stride));
            __syncthreads();
            if (img + 2 * stride < p.B) stage_commit();
            __syncthreads();
        }
    } else {
        const int h = wave & 1, p0 = (wave >> 1) ? FB_NPIX2 - 48 : 0;
        v4i wB[16][2];
#pragma unroll
        for (int st = 0; st < 16; ++st)
#pragma unroll
            for (int t = 0; t < 2; ++t) wB[st][t] = p.wB[(st * 4 + 2 * h + t) * 64 + lane];
        const v4f bi0 = *(const v4f*)(p.biasB + 16 * g + 8 * h), bi1 = *(const v4f*)(p.biasB + 16 * g + 8 * h + 4);
        // window of the lane's pixel of each tile; K step st = kernel row st / 4, column st % 4, the lane's chunk its channels
        int rb[3];
#pragma unroll
        for (int u = 0; u < 3; ++u) {
            const int px = p0 + 16 * u + j;
            const int oy = (px * 7282) >> 16, ox = px - oy * 9;       // px / 9 for px < 81
            rb[u] = g * FB_CH_B + oy * (2 * FB_ROW_B) + ox * 16;
        }
        const int oofs = (p0 + j) * FB_PIX2_BYTES + 32 * g + 16 * h;
        auto frag_b = [&](const char* src, int q) {
            const int u = q >> 4, st = q & 15;
            return *(const v4i*)(src + rb[u] + (st >> 2) * FB_ROW_B + (st & 1) * FB_PAR_B + ((st >> 1) & 1) * 16);
        };
        __syncthreads();
        __syncthreads();
        __syncthreads();
        for (int n = 0;; ++n, img += stride) {
            const char* src = tilesB + (n & 1) * FB_TILE_B;
            char* out = p.out + img * (int64_t)(FB_NPIX2 * FB_PIX2_BYTES);
            const bool last = !(img + stride < p.B);
            v4i gq[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) gq[q] = frag_b(src, q);
            v4f o0 = bi0, o1 = bi1;
#pragma unroll
            for (int u = 0; u < 3; ++u) {
                v4f n0 = bi0, n1 = bi1;
#pragma unroll
                for (int st = 0; st < 16; ++st) {
                    const int q = u * 16 + st;
                    n0 = fb_mfma(wB[st][0], gq[q & 7], n0);
                    n1 = fb_mfma(wB[st][1], gq[q & 7], n1);
                    if (q + 8 < 48) gq[q & 7] = frag_b(src, q + 8);
                }
                if (u > 0) *(v4i*)(out + oofs + (u - 1) * (16 * FB_PIX2_BYTES)) = fb_relu_pack(o0, o1);
                o0 = n0; o1 = n1;
                if (u == 0 && !last) __syncthreads();    // the other wavefronts may replace the observation copy
            }
            *(v4i*)(out + oofs + 2 * (16 * FB_PIX2_BYTES)) = fb_relu_pack(o0, o1);
            if (last) break;
            __syncthreads();
        }
    }
}

}  // namespace

// Exactly the first two layers of the paper's original network as the planner describes them for bf16.
bool conv_front_bf16_supported(const ConvParams& a, int NTA, const ConvParams& b) {
    if (!a.src_u8 || a.mode != CM_U8T || a.Cin_real != 4 || a.Cs_in != 4 || a.H != 84 || a.W != 84) return false;
    if (a.k != 8 || a.s != 4 || a.sx != 4 || a.pad != 0 || a.Ho != 20 || a.Wo != 20 || a.Cs_out != 32) return false;
    if (NTA != 2 || a.k_steps != 8 || a.cpr != 4 || !a.relu || a.pool || a.res) return false;
    if (b.H != 20 || b.W != 20 || b.Cs_in != 32 || b.k != 4 || b.s != 2 || b.sx != 2 || b.pad != 0) return false;
    return b.Ho == 9 && b.Wo == 9 && b.Cs_out == 64 && b.k_steps == 16 && b.cpr == 16 && b.relu && !b.relu_in && !b.pool && !b.res;
}

hipError_t launch_conv_front_bf16(const ConvParams& a, const ConvParams& b, hipStream_t s) {
    if (a.B <= 0) return hipSuccess;
    static bool set = false;
    if (!set) {
        hipError_t e = hipFuncSetAttribute((const void*)conv_front_bf16_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, FB_LDS);
        if (e != hipSuccess) return e;
        set = true;
    }
    FrontBParams p;
    p.obs = (const uint8_t*)a.in; p.out = (char*)b.out;
    p.wA = (const v4i*)a.wfrag; p.biasA = (const float*)a.bias;
    p.wB = (const v4i*)b.wfrag; p.biasB = (const float*)b.bias;
    p.B = a.B;
    // one resident workgroup per compute unit, in even rounds
    const int64_t cap = conv_num_cus(), rounds = (p.B + cap - 1) / cap;
    conv_front_bf16_kernel<<<dim3((unsigned)((p.B + rounds - 1) / rounds)), dim3(FB_THREADS), FB_LDS, s>>>(p);
    return hipGetLastError();
}

}  // namespace accerl
