// Large-batch int8 dense layer with requantizing epilogue, out[b, n] = requant(bias[n] + sum_k W[n, k] x[b, k]),
// as a streaming pipeline.  The tiling is gemm_kernel's (a workgroup owns 64 features and 16 states per wavefront;
// weight fragments are shared through LDS, a wavefront's state fragments come straight from memory), but
// measured per stage of four MFMA steps the generic kernel spends about as long
// issuing its burst of eight loads into a full memory pipeline and then waiting for them as it spends on
// the MFMAs.  Here
//   * every load is requested two stages before its use: the state fragments of stage s+2 go into the registers
//     that step st of stage s has just consumed, the weight fragments of stage s+3 into the registers whose
//     contents went to LDS at the top of stage s;
//   * the loads are spread between the MFMAs of the stage, two after every four MFMAs, instead of one burst;
//   * LDS holds two stages of weight fragments, so one barrier per stage suffices.
// Rows are whole MFMA steps here (Kp_bytes == 64 * k_steps, no ReLU on the input), which leaves no fix-ups in
// the loop, or at large batches whole 16-byte chunks; other shapes stay with gemm_kernel.  Integer accumulation: results are bit-identical.
#include <type_traits>

#include "gemm_epilogue.h"

namespace accerl {

int conv_num_cus();   // compute units of the current device

namespace {
constexpr int SG_KS = 4;                           // MFMA steps per stage
constexpr int SG_NT = 4;                           // feature tiles per workgroup (one per wavefront to fetch)
constexpr int SG_BUF = SG_NT * SG_KS * 1024;       // one stage of weight fragments: [tile][step][64 lanes][16 B]
constexpr int SG_LDS = 2 * SG_BUF;

// WAVES wavefronts of 16 states each: eight when that still gives every compute unit a workgroup (the weight
// fragments are then fetched and written to LDS once per 128 states), else four
// RELU: of the input.  TAIL: rows of whole 16-byte chunks that end inside a step: the chunks behind the row re-read its last one
// (their weights are zero).
template <int WAVES, bool RELU, bool TAIL>
__global__ __launch_bounds__(64 * WAVES, 2) void gemm_stream_i8_kernel(const GemmParams p) {
    constexpr int SG_ROWS = 16 * WAVES;
    constexpr int SG_WF = SG_NT * SG_KS / WAVES;    // weight fragments a wavefront fetches per stage
    extern __shared__ __attribute__((aligned(16))) char sg_smem[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int j = lane & 15, g = lane >> 4;
    const GemmTile tile = gemm_tile<true>((RELU || TAIL) && p.by_xcd);
    const int64_t b0 = (int64_t)tile.x * SG_ROWS;
    const int nt0 = tile.y * SG_NT;
    const int ks = p.k_steps;

    // a state past the batch re-reads the last one; its results are not stored
    int64_t xrow = b0 + wave * 16 + j;
    if (xrow >= p.B) xrow = p.B - 1;
    const char* xb;
    int xstep;
    if (p.x_frag) { xb = (const char*)p.x + (xrow >> 4) * ((int64_t)ks << 10) + lane * 16; xstep = 1024; }
    else { xb = (const char*)p.x + xrow * p.Kp_bytes + g * 16; xstep = 64; }
    // this wavefront fetches fragments wave * SG_WF ... of the stage's [tile][step] grid for all wavefronts
    const int wstep0 = (wave * SG_WF) % SG_KS;
    const char* wb = (const char*)p.wfrag + (int64_t)(nt0 + (wave * SG_WF) / SG_KS) * ks * 1024 + lane * 16;
    char* wdst = sg_smem + wave * SG_WF * 1024 + lane * 16;
    const char* wsrc = sg_smem + lane * 16;

    v4i acc[SG_NT];
#pragma unroll
    for (int t = 0; t < SG_NT; ++t) acc[t] = *(const v4i*)((const int*)p.bias + (nt0 + t) * 16 + 4 * g);

    // steps past the end of K load the last step again (never multiplied)
    const int xlast = p.Kp_bytes - 16 - g * 16;
    auto load_x = [&](v4i& d, int step) {
        if constexpr (TAIL) d = *(const v4i*)(xb + min(step * 64, xlast));
        else d = *(const v4i*)(xb + (int64_t)min(step, ks - 1) * xstep);
    };
    auto load_w = [&](v4i& d, int step) { d = *(const v4i*)(wb + (int64_t)min(step + wstep0, ks - 1) * 1024); };
    auto commit = [&](const v4i (&w)[SG_WF], int buf) {
#pragma unroll
        for (int r = 0; r < SG_WF; ++r) *(v4i*)(wdst + buf * SG_BUF + r * 1024) = w[r];
    };

    v4i xs[2][SG_KS], ws[2][SG_WF];
#pragma unroll
    for (int r = 0; r < SG_WF; ++r) load_w(ws[0][r], r);
#pragma unroll
    for (int r = 0; r < SG_KS; ++r) load_x(xs[0][r], r);
#pragma unroll
    for (int r = 0; r < SG_WF; ++r) load_w(ws[1][r], SG_KS + r);
#pragma unroll
    for (int r = 0; r < SG_KS; ++r) load_x(xs[1][r], SG_KS + r);
    commit(ws[0], 0);
#pragma unroll
    for (int r = 0; r < SG_WF; ++r) load_w(ws[0][r], 2 * SG_KS + r);
    __syncthreads();

    // stage s multiplies from LDS buffer s & 1 and the state registers xs[s & 1]; the weights of stage s+1 go
    // from ws[(s+1) & 1] to the other buffer first.  A full stage has no conditions at all (loads past the end
    // of K are clamped, the fragments they bring are never multiplied); the last, partial stage only multiplies.
    auto stage = [&](int s, auto CUR, auto FULL) {
        constexpr int cur = decltype(CUR)::value, nxt = cur ^ 1;
        constexpr bool full = decltype(FULL)::value;
        if (full) commit(ws[nxt], nxt);
        const char* src = wsrc + cur * SG_BUF;
        v4i fa[2][SG_NT];
#pragma unroll
        for (int t = 0; t < SG_NT; ++t) fa[0][t] = *(const v4i*)(src + (t * SG_KS) * 1024);
        if (full) {
            __builtin_amdgcn_sched_group_barrier(0x200, SG_WF, 0);
            __builtin_amdgcn_sched_group_barrier(0x100, SG_NT, 0);
        }
#pragma unroll
        for (int st = 0; st < SG_KS; ++st) {
            if (st + 1 < SG_KS) {
#pragma unroll
                for (int t = 0; t < SG_NT; ++t) fa[(st + 1) & 1][t] = *(const v4i*)(src + (t * SG_KS + st + 1) * 1024);
            }
            v4i x = xs[cur][st];
            if constexpr (RELU) {
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = (int)g_relu_i8x4((uint32_t)x[e]);
            }
            if (full || s * SG_KS + st < ks) {
#pragma unroll
                for (int t = 0; t < SG_NT; ++t)
                    acc[t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(fa[st & 1][t], x, acc[t], 0, 0, 0);
            }
            if (full) {
                load_x(xs[cur][st], (s + 2) * SG_KS + st);
                if (st < SG_WF) load_w(ws[nxt][st], (s + 3) * SG_KS + st);
                // keep this order in the instruction stream: the LDS reads of the next step, this step's MFMAs, two loads
                if (st + 1 < SG_KS) __builtin_amdgcn_sched_group_barrier(0x100, SG_NT, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, SG_NT, 0);
                if (st < SG_WF) __builtin_amdgcn_sched_group_barrier(0x020, 2, 0);
                else __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);
            }
        }
        if (full) __syncthreads();
    };
    using std::true_type; using std::false_type;
    typedef std::integral_constant<int, 0> even; typedef std::integral_constant<int, 1> odd;
    const int n_full = ks / SG_KS;
    int s = 0;
    for (; s + 2 <= n_full; s += 2) {
        stage(s, even(), true_type());
        stage(s + 1, odd(), true_type());
    }
    if (s < n_full) {
        stage(s, even(), true_type());
        if (ks % SG_KS) stage(s + 1, odd(), false_type());
    } else if (ks % SG_KS) {
        stage(s, even(), false_type());
    }

    // ---- epilogue: lane holds features n0 .. n0+3 of state b; int8 rows are whole tiles of features (Np == 16 * n_tiles; padding features
    //      have zero weights and bias and are stored as zeros)
    const int64_t b = b0 + wave * 16 + j;
    if (b >= p.B) return;
#pragma unroll
    for (int t = 0; t < SG_NT; ++t) {
        const int n0 = (nt0 + t) * 16 + 4 * g;
        const v4f ml = *(const v4f*)(p.mult + n0);
        uint32_t pk = 0;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int v = acc[t][r];
            if (p.tap_acc && n0 + r < p.N) p.tap_acc[b * p.N + n0 + r] = v;
            if (p.relu) {   // clamp(rint(y), 0, 127): the pack instruction rounds to nearest even, saturates at 0
                pk = __builtin_amdgcn_cvt_pk_u8_f32(__builtin_amdgcn_fmed3f((float)v * ml[r], 0.0f, 127.0f), r, pk);
            } else {
                const float y = __builtin_amdgcn_fmed3f(rintf((float)v * ml[r]), -127.0f, 127.0f);
                pk |= ((uint32_t)(int)y & 0xffu) << (8 * r);
            }
        }
        *(uint32_t*)((int8_t*)p.out + b * p.Np + n0) = pk;
    }
}
}  // namespace

bool gemm_stream_supported(const GemmParams& p) {
    return p.B > 0 && p.Np == 16 * p.n_tiles && !p.relu_in && p.k_steps >= 2 * SG_KS && p.Kp_bytes == 64 * p.k_steps && p.n_tiles % SG_NT == 0;
}

template <int WAVES>
static int64_t stream_groups(const GemmParams& p) { return (p.B + 16 * WAVES - 1) / (16 * WAVES) * (p.n_tiles / SG_NT); }

// Rows with a ReLU or an end inside a step take this kernel where eight wavefronts are used: 1936 -> 256 behind the int8
// stacks, 16384 states, 26.3 -> 22.0 us (kernel traces); whole forwards through a small convolution: 1936 -> 256 at 8192 states
// 36.1 -> 32.2 us, 3600 -> 500 at 4096 39.7 -> 36.6, 784 -> 512 at 16384 45.6 -> 41.5.  With four it is not always the faster one
// (3600 -> 500 at 2100 states 35.9 -> 38.4, 1936 -> 256 at 4200 34.8 -> 32.5), nor with up to one and a half workgroups per compute
// unit, or little more than two, if gemm_kernel's groups of 64 states are a multiple of eight (see below) or its workgroups, half the
// size, need no round more (gemm_kernel / this: 3600 -> 768 at 4096 46.7 / 48.6, -> 1024 at 2500 43.5 / 44.9, -> 1536 at 1300 42.3 / 50.4,
// 2048 50.8 / 52.5, -> 3000 at 1300 65.7 / 70.0; else 3600 -> 512 at 5000 55.5 / 49.8, -> 1024 at 3000 50.3 / 46.5, -> 1536 at 1700
// 54.5 / 51.9, 3000 79.5 / 68.4, 1936 -> 512 at 6000 38.6 / 38.4).
bool gemm_stream_rows_supported(const GemmParams& p) {
    if (p.B <= 0 || p.Np != 16 * p.n_tiles || p.x_frag || p.k_steps < 2 * SG_KS || p.Kp_bytes % 16 != 0 || p.n_tiles % SG_NT != 0) return false;
    const int64_t cus = conv_num_cus(), g = stream_groups<8>(p), x4 = (p.B + 63) / 64;
    if (g <= cus) return g == cus;
    const bool thin_round = 2 * g <= 3 * cus || (g > 2 * cus && 4 * g <= 9 * cus);
    return !thin_round || (x4 % 8 != 0 && stream_groups<4>(p) > 2 * cus * (g / cus));
}

template <int WAVES, bool RELU, bool TAIL>
static hipError_t stream_go(const GemmParams& p, hipStream_t s) {
    static bool set = false;
    if (!set) {
        hipError_t e = hipFuncSetAttribute((const void*)gemm_stream_i8_kernel<WAVES, RELU, TAIL>, hipFuncAttributeMaxDynamicSharedMemorySize, SG_LDS);
        if (e != hipSuccess) return e;
        set = true;
    }
    const dim3 grid((unsigned)((p.B + 16 * WAVES - 1) / (16 * WAVES)), (unsigned)(p.n_tiles / SG_NT));
    // Rows: the workgroups of a group of states that do not meet on an XCD by themselves are brought together; fetched by up to eight
    // of them, rows made this kernel slower than gemm_kernel (whole forwards, us, gemm_kernel / not / brought together: 3600 -> 512 at 6000
    // states 53.2 / 60.0 / 50.0, 3600 -> 1024 at 4200 70.8 / 78.5 / 62.7, 3600 -> 2048 at 4200 117 / 128 / 101, 1936 -> 256 at 10000
    // 42.3 / 44.9 / 42.0).  Groups that are a multiple of eight do meet: in the grid's order / by XCD 3600 -> 512 at
    // 4096 36.0 / 37.5, 16384 95.8 / 92.4, 3600 -> 2048 at 4096 84.5 / 86.3.
    GemmParams q = p;
    q.by_xcd = (RELU || TAIL) && grid.y > 1 && (grid.x & 7) != 0;
    gemm_stream_i8_kernel<WAVES, RELU, TAIL><<<grid, dim3(64 * WAVES), SG_LDS, s>>>(q);
    return hipGetLastError();
}

hipError_t launch_gemm_stream(const GemmParams& p, hipStream_t s) {
    if (gemm_stream_supported(p))
        return stream_groups<8>(p) >= conv_num_cus() ? stream_go<8, false, false>(p, s) : stream_go<4, false, false>(p, s);
    if (p.Kp_bytes == 64 * p.k_steps) return stream_go<8, true, false>(p, s);
    return p.relu_in ? stream_go<8, true, true>(p, s) : stream_go<8, false, true>(p, s);
}

}  // namespace accerl
