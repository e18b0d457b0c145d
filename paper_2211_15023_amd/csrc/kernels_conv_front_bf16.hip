// The first two convolutions of the paper's original network (32 filters of 8x8 stride 4, 64 of 4x4 stride 2, no padding,
// on a 4x84x84 uint8 observation) for the bf16 teacher, as one pipelined kernel with every size known at compile time.
//
// A workgroup of eight wavefronts (one per compute unit, two per SIMD) walks over observations.  In one tick wavefronts
// 4..7 compute the first convolution of observation n+1 from its bf16 copy in LDS and write the 20x20x32 image to LDS,
// wavefronts 0..3 compute the second convolution of observation n from the image written in the tick before, and the bytes
// of observation n+2 are in flight; then all eight convert those bytes to bf16 (v / 255) into LDS.  The first layer's output
// never leaves the chip.
//
//  * Weights stay in registers: 8 K steps x 2 channel tiles for the first layer (64), 16 x 2 for one half of the second
//    layer's filters (128).
//  * Observation copy.  A unit is 4 horizontally adjacent pixels of all four planes; its 16 values are two chunks of two
//    pixels, and the first and the second chunks of all units lie in planes of their own.  A K step of the first layer is one
//    kernel row: lane group g reads chunk kind g & 1 of unit ox + g / 2, so 16 pixels of an output row are 256 consecutive
//    bytes.
//  * The first 16 output columns are tiled by output rows, five in a row per wavefront: rows 4..7 of a window are rows 0..3
//    of the window below, so a tile fetches four of its eight fragments; the other 4 columns are five 4 x 4 tiles.
//  * First-layer image: [8 channels][row parity][row / 2][column parity][column / 2][16 B], rows of 25 chunks (ten columns of
//    either parity and a gap): the stride-2 second layer's output pixels 9 oy + ox read chunks 25 oy + ox, which are the same
//    modulo the 16 chunks of a bank round, so any 16 consecutive pixels are free of conflicts.  All planes are multiples of
//    256 bytes apart, since a pass of a 16-byte read mixes lanes of neighbouring groups.
//  * K steps, weight fragments and bias are the planner's, in its order: results are bit-identical to conv_kernel.h.
//  * The second layer's 81 pixels are the tiles 0..47 and 33..80; the overlap is stored twice with the same bytes.
//
// What bounds it (clocks per observation inside the kernel): the two layers 3 900, 3 330 of them at the matrix cores' rate; the
// conversion 1 400 to 1 600, at the vector ALUs' rate, with the matrix cores idle.  4096 states: 59 us (the generic kernels
// 79 + 97 us; medians of kernel traces).  Without effect on the time: bank conflicts of the fragment reads (six million clocks of 15 removed), the
// order of the loads, two accumulator chains or four in the first layer.
#include <type_traits>

#include "conv_kernel.h"

namespace accerl {

namespace {

constexpr int FB_THREADS = 512;
constexpr int FB_PLANE_IN = 84 * 84;                     // bytes of a channel plane of the observation
constexpr int FB_UNITS = FB_PLANE_IN / 4;                // 1764
constexpr int FB_RAW = (4 * FB_PLANE_IN + 4095) / 4096 * 4096;   // the observation's bytes as they are, whole KiB per wavefront
constexpr int FB_ROW_A = 21 * 16, FB_KIND_A = (FB_UNITS * 16 + 255) / 256 * 256, FB_TILE_A = 2 * FB_KIND_A;
constexpr int FB_ROW_B = 25 * 16, FB_XPAR_B = 10 * 16, FB_YPAR_B = 10 * FB_ROW_B, FB_CH_B = 8192, FB_TILE_B = 4 * FB_CH_B;
static_assert(2 * FB_YPAR_B <= FB_CH_B, "two row parities of ten rows");
constexpr int FB_LDS = FB_TILE_A + 2 * FB_TILE_B;      // besides FB_RAW
constexpr int FB_NPIX2 = 81, FB_PIX2_BYTES = 128;

struct FrontBParams {
    const uint8_t* obs;      // [B, 4, 84, 84]
    const int32_t* rows;     // observation i is row rows[i] of obs (NULL = row i)
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
// ReLU of eight accumulators (consecutive channels) as bf16: a negative bf16 is a negative 16-bit integer, and so is the only NaN
// that the matrix cores produce (0xffc0), which becomes 0 as in fmaxf
__device__ __forceinline__ v4i fb_relu_pack(v4f a, v4f b) {
    typedef short v8s __attribute__((ext_vector_type(8)));
    const v8s z = {0, 0, 0, 0, 0, 0, 0, 0};
    const v4i v = {fb_pack2(a[0], a[1]), fb_pack2(a[2], a[3]), fb_pack2(b[0], b[1]), fb_pack2(b[2], b[3])};
    return __builtin_bit_cast(v4i, __builtin_elementwise_max(__builtin_bit_cast(v8s, v), z));
}
// two pixels of four channels, bf16(v / 255): bytes LO and LO + 1 of the four planes' dwords
template <int LO>
__device__ __forceinline__ v4i fb_obs(const uint32_t (&d)[4]) {
    constexpr float k = 1.0f / 255.0f;
    auto v = [&](int c, int px) { return (float)((d[c] >> (8 * (LO + px))) & 0xffu) * k; };
    return (v4i){fb_pack2(v(0, 0), v(1, 0)), fb_pack2(v(2, 0), v(3, 0)), fb_pack2(v(0, 1), v(1, 1)), fb_pack2(v(2, 1), v(3, 1))};
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

    // Staging.  The second-layer wavefronts, which have time to spare, send the bytes of an observation straight from memory
    // to `raw` (the memory queue of a compute unit fills up and holds the wavefront that issues into it); from there all eight
    // wavefronts convert their share.
    __shared__ __attribute__((aligned(16))) uint8_t raw[FB_RAW];
    auto fetch = [&](int64_t im) {
        const uint8_t* src = p.obs + (p.rows ? (int64_t)p.rows[im] : im) * (int64_t)(4 * FB_PLANE_IN);
#pragma unroll
        for (int k = 0; k < FB_RAW / 4096; ++k) {
            const uint32_t at = (wave + 4 * k) * 1024;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(src + min(at + lane * 16, (uint32_t)(4 * FB_PLANE_IN - 16))),
                                             (__attribute__((address_space(3))) void*)(raw + at), 16, 0, 0);
        }
    };
    auto fetched = [&]() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };   // by the wavefronts that fetch, before the barrier
    auto convert = [&]() {
#pragma unroll
        for (int k = 0; k < (FB_UNITS + FB_THREADS - 1) / FB_THREADS; ++k) {
            const int u = tid + k * FB_THREADS;
            if (u < FB_UNITS) {
                uint32_t d[4];
#pragma unroll
                for (int c = 0; c < 4; ++c) d[c] = *(const uint32_t*)(raw + c * FB_PLANE_IN + 4 * u);
                *(v4i*)(tileA + 16 * u) = fb_obs<0>(d);
                *(v4i*)(tileA + FB_KIND_A + 16 * u) = fb_obs<2>(d);
            }
        }
    };

    if (wave >= 4) {
        const int aw = wave - 4;
        v4i wA[8][2];
#pragma unroll
        for (int st = 0; st < 8; ++st)
#pragma unroll
            for (int t = 0; t < 2; ++t) wA[st][t] = p.wA[(st * 2 + t) * 64 + lane];
        const v4f bi0 = *(const v4f*)(p.biasA + 8 * g), bi1 = *(const v4f*)(p.biasA + 8 * g + 4);

        // chain tiles: output row 5 aw + r, column j; then the 4 x 4 tiles aw and (first wavefront only) 4
        const int lane_in = (g >> 1) * 16 + (g & 1) * FB_KIND_A;
        const int rb_chain = (5 * aw) * (4 * FB_ROW_A) + j * 16 + lane_in;
        auto at_b = [&](int oy, int ox) { return g * FB_CH_B + (oy & 1) * FB_YPAR_B + (oy >> 1) * FB_ROW_B + (ox & 1) * FB_XPAR_B + (ox >> 1) * 16; };
        int wb_chain[5], rb_blk[2], wb_blk[2];
#pragma unroll
        for (int r = 0; r < 5; ++r) wb_chain[r] = at_b(5 * aw + r, j);
#pragma unroll
        for (int k = 0; k < 2; ++k) {
            const int b = k == 0 ? aw : 4, oy = 4 * b + (j >> 2), ox = 16 + (j & 3);
            rb_blk[k] = oy * (4 * FB_ROW_A) + ox * 16 + lane_in;
            wb_blk[k] = at_b(oy, ox);
        }
        // window row i below the lane's first chain pixel (tile r: rows 4r .. 4r + 7), window row i of 4 x 4 tile k
        auto chain = [&](int i) { return *(const v4i*)(tileA + rb_chain + i * FB_ROW_A); };
        auto blk = [&](int k, int i) { return *(const v4i*)(tileA + rb_blk[k] + i * FB_ROW_A); };
        auto store_a = [&](char* dst, v4f a, v4f b) { *(v4i*)dst = fb_relu_pack(a, b); };
        // Two tiles at a time: four accumulator chains (with two, the matrix core waits for the result of the MFMA before last:
        // 25 clocks each instead of 16).  Chain tiles (0, 1), (2, 3), then chain tile 4 with the 4 x 4 tile, in the first
        // wavefront with the fifth 4 x 4 tile too.  Meanwhile the fragments of the next two tiles are requested and the two
        // tiles before are packed and stored.
        auto conv_a = [&](char* dstB) {
            v4i f[12], b[8];
#pragma unroll
            for (int i = 0; i < 12; ++i) f[i] = chain(i);
            __builtin_amdgcn_sched_barrier(0);
            v4f o[4];
#pragma unroll
            for (int pr = 0; pr < 2; ++pr) {
                v4f n[4] = {bi0, bi1, bi0, bi1};
                v4i fn[12];
#pragma unroll
                for (int st = 0; st < 8; ++st) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) n[t] = fb_mfma(wA[st][t & 1], f[st + 4 * (t >> 1)], n[t]);
                    if (st < 4) fn[st] = f[st + 8];
                    if (pr == 0 || st < 4) fn[st + 4] = chain(8 * pr + 12 + st);
                    if (pr == 1) b[st] = blk(0, st);
                }
                if (pr > 0) {
                    store_a(dstB + wb_chain[0], o[0], o[1]);
                    store_a(dstB + wb_chain[1], o[2], o[3]);
                }
#pragma unroll
                for (int t = 0; t < 4; ++t) o[t] = n[t];
#pragma unroll
                for (int i = 0; i < (pr == 0 ? 12 : 8); ++i) f[i] = fn[i];
                // the instruction stream in this order (the scheduler alone moves the reads next to their use)
#pragma unroll
                for (int st = 0; st < 8; ++st) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 4, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    if (pr == 1 && st < 4) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    if (pr > 0) __builtin_amdgcn_sched_group_barrier(0x002, 2, 0);
                }
                if (pr > 0) __builtin_amdgcn_sched_group_barrier(0x200, 2, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            auto last = [&](auto THIRD) {
                constexpr bool third = decltype(THIRD)::value;
                v4f n[6] = {bi0, bi1, bi0, bi1, bi0, bi1};
                v4i c[8];
                if constexpr (third) {
#pragma unroll
                    for (int st = 0; st < 8; ++st) c[st] = blk(1, st);
                }
#pragma unroll
                for (int st = 0; st < (third ? 12 : 8); ++st) {
                    if (st < 8) {
#pragma unroll
                        for (int t = 0; t < 4; ++t) n[t] = fb_mfma(wA[st][t & 1], t < 2 ? f[st] : b[st], n[t]);
                    }
                    if (third && st >= 4) {
#pragma unroll
                        for (int t = 0; t < 2; ++t) n[4 + t] = fb_mfma(wA[st - 4][t], c[st - 4], n[4 + t]);
                    }
                }
                store_a(dstB + wb_chain[2], o[0], o[1]);
                store_a(dstB + wb_chain[3], o[2], o[3]);
                store_a(dstB + wb_chain[4], n[0], n[1]);
                store_a(dstB + wb_blk[0], n[2], n[3]);
                if constexpr (third) store_a(dstB + wb_blk[1], n[4], n[5]);
            };
            if (aw == 0) last(std::true_type());
            else last(std::false_type());
        };

        __syncthreads();                                 // the first observation's bytes are there
        convert();
        __syncthreads();                                 // observation copy complete
        conv_a(tilesB);
        __syncthreads();                                 // first image complete, observation copy free, next bytes there
        if (img + stride < p.B) convert();
        __syncthreads();
        for (int n = 0;; ++n, img += stride) {
            if (!(img + stride < p.B)) break;            // the workgroup's observations are done (same test in every wavefront)
            conv_a(tilesB + ((n + 1) & 1) * FB_TILE_B);
            __syncthreads();
            if (img + 2 * stride < p.B) convert();
            __syncthreads();
        }
    } else {
        fetch(img);
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
            rb[u] = g * FB_CH_B + oy * FB_ROW_B + ox * 16;
        }
        const int oofs = (p0 + j) * FB_PIX2_BYTES + 32 * g + 16 * h;
        auto frag_b = [&](const char* src, int q) {
            const int u = q >> 4, st = q & 15;
            return *(const v4i*)(src + rb[u] + ((st >> 2) & 1) * FB_YPAR_B + (st >> 3) * FB_ROW_B + (st & 1) * FB_XPAR_B + ((st >> 1) & 1) * 16);
        };
        fetched();
        __syncthreads();
        convert();
        __syncthreads();
        if (img + stride < p.B) fetch(img + stride);
        fetched();
        __syncthreads();
        if (img + stride < p.B) convert();
        __syncthreads();
        for (int n = 0;; ++n, img += stride) {
            if (img + 2 * stride < p.B) fetch(img + 2 * stride);
            const char* src = tilesB + (n & 1) * FB_TILE_B;
            char* out = p.out + img * (int64_t)(FB_NPIX2 * FB_PIX2_BYTES);
            v4i gq[8];
#pragma unroll
            for (int q = 0; q < 8; ++q) gq[q] = frag_b(src, q);
            __builtin_amdgcn_sched_barrier(0);
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
                // the instruction stream in this order: two MFMAs, the fragment eight steps ahead (the scheduler alone moves the
                // reads next to their use, and every MFMA pair waits for LDS)
#pragma unroll
                for (int st = 0; st < 16; ++st) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                    if (u * 16 + st + 8 < 48) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    if (u > 0 && st < 8) __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);
                }
                if (u > 0) __builtin_amdgcn_sched_group_barrier(0x040, 1, 0);
                __builtin_amdgcn_sched_barrier(0);
            }
            *(v4i*)(out + oofs + 2 * (16 * FB_PIX2_BYTES)) = fb_relu_pack(o0, o1);
            if (!(img + stride < p.B)) break;
            fetched();
            __syncthreads();
            if (img + 2 * stride < p.B) convert();
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
    p.obs = (const uint8_t*)a.in; p.rows = a.rows; p.out = (char*)b.out;
    p.wA = (const v4i*)a.wfrag; p.biasA = (const float*)a.bias;
    p.wB = (const v4i*)b.wfrag; p.biasB = (const float*)b.bias;
    p.B = a.B;
    // one resident workgroup per compute unit, in even rounds
    const int64_t cap = conv_num_cus(), rounds = (p.B + cap - 1) / cap;
    conv_front_bf16_kernel<<<dim3((unsigned)((p.B + rounds - 1) / rounds)), dim3(FB_THREADS), FB_LDS, s>>>(p);
    return hipGetLastError();
}

}  // namespace accerl
