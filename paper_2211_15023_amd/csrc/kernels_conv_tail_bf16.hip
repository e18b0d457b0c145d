// The third convolution of the paper's original network (64 filters of 3x3, stride 1, no padding, on a 9x9x64 image) for the
// bf16 teacher: the int8 kernel's scheme (kernels_conv_tail_i8.hip) with twice the K steps.
//
// Four wavefronts work on two images at a time: wavefronts 2s and 2s + 1 own image slot s, one half of the filters each, in
// registers for the whole kernel (18 K steps -- a filter tap and half of the channels each -- x 2 channel tiles = 144
// registers).  An image is four tiles (three of two output rows, one of the last row; the spare lanes repeat a pixel).  LDS
// holds two copies of every slot's image as eight planes of 8 channels, [channel block][pixel][16 B]: the 14 pixels of a
// two-row tile fall into 14 different 16-byte bank groups.  While image n is multiplied, image n + 1 goes to the idle copy and
// image n + 2 is requested: one barrier per image.
//
// What bounds it: each LDS fragment feeds two MFMAs (144 KB and 288 MFMAs per image: 1 152 clocks of either).  4096 states:
// 23 us (the generic kernel 46 us).
#include "conv_kernel.h"

namespace accerl {

namespace {
constexpr int TB_SLOTS = 2, TB_THREADS = 128 * TB_SLOTS;
constexpr int TB_IMG = 81 * 128;                 // bytes per input image
constexpr int TB_UNITS = TB_IMG / 16;            // 648 staging chunks
constexpr int TB_PLANE = 1536;                   // 81 pixels of 16 bytes, padded to a multiple of 256
constexpr int TB_COPY = 8 * TB_PLANE;
constexpr int TB_PF = (TB_UNITS + 127) / 128;    // staging chunks per lane of a slot's two wavefronts (6)
constexpr int TB_LDS = TB_SLOTS * 2 * TB_COPY;
constexpr int TB_NPIX = 49, TB_PIX_BYTES = 128;

struct TailBParams {
    const char* in;          // bf16 [B, 9, 9, 64]
    char* out;               // bf16 [B, 7, 7, 64] or fragment order
    const v4i* w; const float* bias;
    int64_t B;
    int out_frag, frag_ks;
};

__device__ __forceinline__ v4f tb_mfma(v4i a, v4i b, v4f c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(v8bf, a), __builtin_bit_cast(v8bf, b), c, 0, 0, 0);
}

__global__ __launch_bounds__(TB_THREADS, 2) void conv_tail_bf16_kernel(const TailBParams p) {
    extern __shared__ __attribute__((aligned(16))) char smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    const int slot = wave >> 1, h = wave & 1;
    char* tiles = smem + slot * (2 * TB_COPY);

    const int64_t stride = TB_SLOTS * (int64_t)gridDim.x;
    int64_t img = TB_SLOTS * (int64_t)blockIdx.x + slot;
    const int64_t img_first = TB_SLOTS * (int64_t)blockIdx.x;     // the workgroup's first image (the same in every wavefront)
    if (img_first >= p.B) return;

    // staging: chunk u = (pixel u / 8, channel block u % 8) goes to plane u % 8
    const int stid = tid & 127;
    v4i pre[TB_PF];
    auto stage_load = [&](int64_t im) {
        const char* src = p.in + im * (int64_t)TB_IMG;
#pragma unroll
        for (int k = 0; k < TB_PF; ++k) pre[k] = *(const v4i*)(src + 16 * min(stid + 128 * k, TB_UNITS - 1));
    };
    auto stage_commit = [&](char* dst) {
#pragma unroll
        for (int k = 0; k < TB_PF; ++k) {
            const int u = stid + 128 * k;
            if (u < TB_UNITS) *(v4i*)(dst + (u & 7) * TB_PLANE + (u >> 3) * 16) = pre[k];
        }
    };

    if (img < p.B) stage_load(img);
    v4i w[18][2];
#pragma unroll
    for (int st = 0; st < 18; ++st)
#pragma unroll
        for (int t = 0; t < 2; ++t) w[st][t] = p.w[(st * 4 + 2 * h + t) * 64 + lane];
    const v4f bi0 = *(const v4f*)(p.bias + 16 * g + 8 * h), bi1 = *(const v4f*)(p.bias + 16 * g + 8 * h + 4);

    // the lane's pixel in each of the four tiles: tile u = output rows 2u and 2u+1 (tile 3: row 6 and, again, row 5);
    // lanes 14 and 15 repeat lane 13's pixel
    int rb[4], oofs[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int jj = min(j, 13), r = jj >= 7 ? 1 : 0, ox = jj - 7 * r;
        const int oy = (u < 3 ? 2 * u : 5) + r;
        rb[u] = g * TB_PLANE + (oy * 9 + ox) * 16;
        const int px = oy * 7 + ox, ci = 2 * g + h;      // the lane's 8 output channels are chunk ci of the pixel
        oofs[u] = p.out_frag ? (2 * px + (ci >> 2)) * 1024 + (ci & 3) * 256 : px * TB_PIX_BYTES + 16 * ci;
    }
    // step q = 18 * tile + 2 * tap + channel half; fragments rotate through eight slots
    auto frag = [&](const char* src, int q) {
        const int u = q / 18, st = q - 18 * u, tap = st >> 1;
        return *(const v4i*)(src + rb[u] + (st & 1) * (4 * TB_PLANE) + ((tap / 3) * 9 + (tap % 3)) * 16);
    };
    auto store = [&](char* outp, int u, v4f a, v4f b) {   // ReLU on the rounded values: see fb_relu_pack
        typedef float v2f __attribute__((ext_vector_type(2)));
        typedef __bf16 v2bf __attribute__((ext_vector_type(2)));
        typedef short v8s __attribute__((ext_vector_type(8)));
        auto pk = [](float x, float y) { return __builtin_bit_cast(int, __builtin_convertvector((v2f){x, y}, v2bf)); };
        const v8s z = {0, 0, 0, 0, 0, 0, 0, 0};
        const v4i v = {pk(a[0], a[1]), pk(a[2], a[3]), pk(b[0], b[1]), pk(b[2], b[3])};
        *(v4i*)(outp + oofs[u]) = __builtin_bit_cast(v4i, __builtin_elementwise_max(__builtin_bit_cast(v8s, v), z));
    };
    auto compute = [&](const char* src, char* outp) {
        v4i gq[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) gq[q] = frag(src, q);
        __builtin_amdgcn_sched_barrier(0);
        v4f o0 = bi0, o1 = bi1;
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            v4f n0 = bi0, n1 = bi1;
#pragma unroll
            for (int st = 0; st < 18; ++st) {
                const int q = u * 18 + st;
                n0 = tb_mfma(w[st][0], gq[q & 7], n0);
                n1 = tb_mfma(w[st][1], gq[q & 7], n1);
                if (q + 8 < 72) gq[q & 7] = frag(src, q + 8);
            }
            if (u > 0) store(outp, u - 1, o0, o1);
            o0 = n0; o1 = n1;
            // two MFMAs, then the fragment eight steps ahead (left alone, the scheduler moves the reads next to their use)
#pragma unroll
            for (int st = 0; st < 18; ++st) {
                __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
                if (u * 18 + st + 8 < 72) __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                if (u > 0 && st < 8) __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);
            }
            if (u > 0) __builtin_amdgcn_sched_group_barrier(0x040, 1, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        store(outp, 3, o0, o1);
    };
    auto out_of = [&](int64_t im) -> char* {
        return p.out_frag ? p.out + (im >> 4) * ((int64_t)p.frag_ks << 10) + (((int)im & 15) << 4)
                          : p.out + im * (int64_t)(TB_NPIX * TB_PIX_BYTES);
    };

    if (img < p.B) stage_commit(tiles);
    if (img + stride < p.B) stage_load(img + stride);
    __syncthreads();
    for (int n = 0;; ++n, img += stride) {
        if (img + stride < p.B) stage_commit(tiles + ((n + 1) & 1) * TB_COPY);
        if (img + 2 * stride < p.B) stage_load(img + 2 * stride);
        if (img < p.B) compute(tiles + (n & 1) * TB_COPY, out_of(img));
        if (!(img_first + (n + 1) * stride < p.B)) break;
        __syncthreads();
    }
}
}  // namespace

// Exactly the third layer of the paper's original network as the planner describes it for bf16.
bool conv_tail_bf16_supported(const ConvParams& p, int NT) {
    if (p.src_u8 || p.mode != CM_FLAT || p.H != 9 || p.W != 9 || p.Cs_in != 64 || p.Cin_real != 64) return false;
    if (p.k != 3 || p.s != 1 || p.sx != 1 || p.pad != 0 || p.Ho != 7 || p.Wo != 7 || p.Cs_out != 64 || NT != 4) return false;
    if (p.k_steps != 18 || p.cpr != 24 || !p.relu || p.relu_in || p.pool || p.res || p.tap_acc) return false;
    return !p.out_frag || p.frag_ks == 98;
}

hipError_t launch_conv_tail_bf16(const ConvParams& c, hipStream_t s) {
    if (c.B <= 0) return hipSuccess;
    static int occ = 0;
    if (!occ) {
        hipError_t e = hipFuncSetAttribute((const void*)conv_tail_bf16_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, TB_LDS);
        if (e != hipSuccess) return e;
        int o = 0;
        e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&o, (const void*)conv_tail_bf16_kernel, TB_THREADS, TB_LDS);
        if (e != hipSuccess) return e;
        occ = o < 1 ? 1 : o;
    }
    TailBParams p;
    p.in = (const char*)c.in; p.out = (char*)c.out;
    p.w = (const v4i*)c.wfrag; p.bias = (const float*)c.bias;
    p.B = c.B; p.out_frag = c.out_frag; p.frag_ks = c.frag_ks;
    // resident workgroups striding over groups of TB_SLOTS images, in even rounds
    const int64_t groups = (p.B + TB_SLOTS - 1) / TB_SLOTS;
    const int64_t cap = (int64_t)occ * conv_num_cus();
    const int64_t rounds = (groups + cap - 1) / cap;
    conv_tail_bf16_kernel<<<dim3((unsigned)((groups + rounds - 1) / rounds)), dim3(TB_THREADS), TB_LDS, s>>>(p);
    return hipGetLastError();
}

}  // namespace accerl
