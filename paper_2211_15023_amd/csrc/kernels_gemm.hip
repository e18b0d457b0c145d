// Dense layers on the matrix cores: out[b, n] = sum_k W[n, k] x[b, k], int8 (int32 accumulate) or
// bf16 (fp32 accumulate).  Output features are the MFMA rows and states the columns, so one lane ends
// up with 4 consecutive features of one state.  A workgroup owns 64 features x 64 states and walks K
// in stages of 256 bytes per row: weights through LDS, every wavefront's 16 states straight from memory
// into its B fragments; the epilogue is chosen at compile time:
// requantize to int8, bias+ReLU to bf16, policy heads (logits / value in fp32), or the LSTM cell
// (weight rows are interleaved on the host so that the 4 accumulators of a lane are the i,f,g,o
// pre-activations of one hidden unit).
#include <stdlib.h>

#include "gemm_epilogue.h"

namespace accerl {

constexpr int GM_THREADS = 256;
constexpr int GM_NT = 4;          // feature tiles (of 16) per workgroup
constexpr int GM_RT = 1;          // row tiles (of 16 states) per wave
constexpr int GM_WAVES = GM_THREADS / 64;
constexpr int GM_ROWS = 16 * GM_WAVES * GM_RT;   // states per workgroup
constexpr int GM_KS = 4;          // MFMA steps per LDS stage (64 bytes of K each); a multiple of 4

// PARTS > 1: K is summed in that many parts, which are then added to the bias in order -- the sums of the kernel whose
// wavefronts split K (kernels_gemm_ksplit.hip), bit for bit, so that a bf16 state's result does not depend on its batch.
template <int EL, int EPI, int PARTS>
__global__ __launch_bounds__(GM_THREADS, PARTS > 1 ? 4 : 2) void gemm_kernel(const GemmParams p) {
    extern __shared__ __attribute__((aligned(16))) char gm_smem[];
    char* s_w = gm_smem;                              // [GM_NT][GM_KS][64 lanes][16 B]
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // wave-uniform: what depends on it stays scalar
    const int j = lane & 15, g = lane >> 4;
    const int64_t b0 = (int64_t)blockIdx.x * GM_ROWS;
    const int nt0 = blockIdx.y * GM_NT;
    const int nts = (p.n_tiles - nt0 < GM_NT) ? (p.n_tiles - nt0) : GM_NT;

    // accumulators start from the bias (features n = 16*(nt0+t) + 4g + r)
    v4i acc_i[GM_RT][GM_NT];
    v4f acc_f[GM_RT][GM_NT];
#pragma unroll
    for (int t = 0; t < GM_NT; ++t) {
        const int n0 = (nt0 + (t < nts ? t : 0)) * 16 + 4 * g;
#pragma unroll
        for (int u = 0; u < GM_RT; ++u) {
            if constexpr (EL == EL_I8) acc_i[u][t] = *(const v4i*)((const int*)p.bias + n0);
            else acc_f[u][t] = *(const v4f*)((const float*)p.bias + n0);
        }
    }
    // PARTS > 1: the bias and the parts so far
    static_assert(PARTS == 1 || EL == EL_BF16, "integer sums do not depend on the order");
    v4f sum[GM_RT][GM_NT];
    int part = 0, part_end = p.k_steps / PARTS;
    if constexpr (PARTS > 1) {
#pragma unroll
        for (int u = 0; u < GM_RT; ++u)
#pragma unroll
            for (int t = 0; t < GM_NT; ++t) { sum[u][t] = acc_f[u][t]; acc_f[u][t] = (v4f){0.0f, 0.0f, 0.0f, 0.0f}; }
    }

    // Stage s0 of K: the weight fragments [GM_NT tiles][GM_KS steps] go through LDS (all four wavefronts
    // read them); a wavefront's own 16 states need no sharing: lane (j, g) loads state j's 16 bytes of K
    // block g straight from memory, which is exactly its MFMA B fragment.  The loads of the next stage are
    // issued into registers before the MFMA work of the current one.  They are unconditional (clamped
    // addresses, fixed up afterwards) so that nothing serialises them.
    constexpr int WPRE = GM_NT * GM_KS * 64 / GM_THREADS;       // weight units per lane
    v4i wpre[WPRE], xpre[GM_RT][GM_KS], xcur[GM_RT][GM_KS];
    const char* xptr[GM_RT];
#pragma unroll
    for (int u = 0; u < GM_RT; ++u) {
        int64_t xrow = b0 + (wave * GM_RT + u) * 16 + j;
        if (xrow >= p.B) xrow = p.B - 1;        // a state past the batch re-reads the last one; its results are not stored
        xptr[u] = (const char*)p.x + xrow * p.Kp_bytes;
        if (p.x_frag)                           // fragment order: the tile of 16 states of this wavefront, one KiB per step
            xptr[u] = (const char*)p.x + (xrow >> 4) * ((int64_t)p.k_steps << 10) + lane * 16;
    }
    auto prefetch = [&](int s0) {
        const int ns = (p.k_steps - s0 < GM_KS) ? (p.k_steps - s0) : GM_KS;
#pragma unroll
        for (int r = 0; r < WPRE; ++r) {                         // unit r of a lane: (tile, step) pair number wave + GM_WAVES * r
            const int tr = (wave + GM_WAVES * r) % GM_NT, sr = (wave + GM_WAVES * r) / GM_NT;
            const int t = (tr < nts) ? tr : 0, st = (sr < ns) ? sr : 0;
            wpre[r] = ((const v4i*)p.wfrag)[((int64_t)(nt0 + t) * p.k_steps + s0 + st) * 64 + lane];
        }
#pragma unroll
        for (int st = 0; st < GM_KS; ++st) {
            int kb = (s0 + st) * 64 + g * 16;
            if (kb > p.Kp_bytes - 16) kb = (p.Kp_bytes - 16) & ~3;
            if (p.x_frag) kb = min(s0 + st, p.k_steps - 1) << 10;
#pragma unroll
            for (int u = 0; u < GM_RT; ++u) xpre[u][st] = *(const v4i*)(xptr[u] + kb);
        }
    };
    auto commit = [&](int s0) {
        const int ns = (p.k_steps - s0 < GM_KS) ? (p.k_steps - s0) : GM_KS;
#pragma unroll
        for (int r = 0; r < WPRE; ++r) {
            const int tr = (wave + GM_WAVES * r) % GM_NT, sr = (wave + GM_WAVES * r) / GM_NT;
            v4i v = wpre[r];
            if (!(tr < nts && sr < ns)) v = (v4i){0, 0, 0, 0};
            ((v4i*)s_w)[(tr * GM_KS + sr) * 64 + lane] = v;
        }
        // only the stage that reaches the end of the rows needs the chunk fix-ups (states past the batch
        // need none: their results are never stored)
        if ((s0 + GM_KS) * 64 <= p.Kp_bytes && !p.relu_in) {
#pragma unroll
            for (int st = 0; st < GM_KS; ++st)
#pragma unroll
                for (int u = 0; u < GM_RT; ++u) xcur[u][st] = xpre[u][st];
            return;
        }
#pragma unroll
        for (int st = 0; st < GM_KS; ++st)
#pragma unroll
        for (int u = 0; u < GM_RT; ++u) {
            const int kb = (s0 + st) * 64 + g * 16;
            v4i v = xpre[u][st];
            // a chunk that starts inside the row but runs past it re-read the row's last 16 bytes: rebuild
            // it from the bytes that belong to it (rows are padded with zero weights, not zero data)
            if (kb >= p.Kp_bytes) {
                v = (v4i){0, 0, 0, 0};
            } else if (kb > p.Kp_bytes - 16) {
                const int have = p.Kp_bytes - kb;              // 4, 8 or 12 valid bytes, at the end of v
                const int sh = (16 - have) >> 2;
                v4i w = {0, 0, 0, 0};
#pragma unroll
                for (int e = 0; e < 4; ++e) if (e + sh < 4) w[e] = v[(e + sh) & 3];
                v = w;
            }
            if (p.relu_in) {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    v[e] = (int)((EL == EL_I8) ? g_relu_i8x4((uint32_t)v[e]) : g_relu_bf16x2((uint32_t)v[e]));
            }
            xcur[u][st] = v;
        }
    };

    prefetch(0);
    for (int s0 = 0; s0 < p.k_steps; s0 += GM_KS) {
        const int ns = (p.k_steps - s0 < GM_KS) ? (p.k_steps - s0) : GM_KS;
        commit(s0);
        __syncthreads();
        if (s0 + GM_KS < p.k_steps) prefetch(s0 + GM_KS);
        // the weight fragments of step st+1 are requested from LDS before the MFMAs of step st are issued
        auto load_a = [&](v4i (&a)[GM_NT], int st) {
#pragma unroll
            for (int t = 0; t < GM_NT; ++t) a[t] = *(const v4i*)(s_w + ((t * GM_KS + st) * 64 + lane) * 16);
        };
        auto mfma = [&](const v4i (&a)[GM_NT], int st) {
#pragma unroll
            for (int t = 0; t < GM_NT; ++t)
#pragma unroll
                for (int u = 0; u < GM_RT; ++u) {
                    if constexpr (EL == EL_I8) {
                        acc_i[u][t] = __builtin_amdgcn_mfma_i32_16x16x64_i8(a[t], xcur[u][st], acc_i[u][t], 0, 0, 0);
                    } else {
                        acc_f[u][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(v8bf, a[t]), __builtin_bit_cast(v8bf, xcur[u][st]), acc_f[u][t], 0, 0, 0);
                    }
                }
        };
        {
            v4i fa[2][GM_NT];
            load_a(fa[0], 0);
#pragma unroll
            for (int st = 0; st < GM_KS; ++st) {
                if (st < ns) {
                    if (st + 1 < ns) load_a(fa[(st + 1) & 1], st + 1);
                    mfma(fa[st & 1], st);
                    if constexpr (PARTS > 1) {
                        if (s0 + st + 1 == part_end) {
                            ++part;
                            part_end = (part + 1) * p.k_steps / PARTS;
#pragma unroll
                            for (int u = 0; u < GM_RT; ++u)
#pragma unroll
                                for (int t = 0; t < GM_NT; ++t) { sum[u][t] += acc_f[u][t]; acc_f[u][t] = (v4f){0.0f, 0.0f, 0.0f, 0.0f}; }
                        }
                    }
                }
            }
        }
        __syncthreads();
    }

    // ---- epilogue: lane holds features n0 .. n0+3 of state b
    int ln = lane;
    if constexpr (PARTS > 1) {                               // counted anew: a register kept for it through the loop is one too many
        uint32_t zero = 0;
        asm volatile("" : "+v"(zero));
        ln = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, zero));
    }
#pragma unroll
    for (int u = 0; u < GM_RT; ++u) {
        const int64_t b = b0 + (wave * GM_RT + u) * 16 + (ln & 15);
        if (b >= p.B) continue;
#pragma unroll
        for (int t = 0; t < GM_NT; ++t) {
            if (t >= nts) continue;
            const int n0 = (nt0 + t) * 16 + 4 * (ln >> 4);
            // stored activations: rows past N up to the row pitch are written too (zero weights and bias give zeros)
            if (n0 >= ((EPI == EPI_REQUANT || EPI == EPI_BF16) ? p.Np : p.N)) continue;
            if constexpr (EL == EL_I8) gemm_finish<EPI>(p, acc_i[u][t], b, n0);
            else gemm_finish<EPI>(p, PARTS > 1 ? sum[u][t] : acc_f[u][t], b, n0);
        }
    }
}

template <int EL, int EPI, int PARTS = 1>
static hipError_t gemm_go(const GemmParams& p, dim3 grid, hipStream_t s) {
    constexpr size_t lds = GM_NT * GM_KS * 1024;
    auto kfn = gemm_kernel<EL, EPI, PARTS>;
    static bool set = false;   // per instantiation: the stage buffers exceed the default dynamic LDS limit
    if (!set) {
        hipError_t e = hipFuncSetAttribute((const void*)kfn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        set = true;
    }
    kfn<<<grid, dim3(GM_THREADS), lds, s>>>(p);
    return hipGetLastError();
}

hipError_t launch_gemm(const GemmParams& p, Elem el, GemmEpi epi, hipStream_t s) {
    if (p.B <= 0) return hipSuccess;
    dim3 grid((unsigned)((p.B + GM_ROWS - 1) / GM_ROWS), (unsigned)((p.n_tiles + GM_NT - 1) / GM_NT));
    if (gemm_ksplit_supported(p, el, epi)) return launch_gemm_ksplit(p, el, s);
    if (el == EL_I8 && epi == EPI_REQUANT) {
        static const bool no_stream = getenv("ACCERL_NO_GEMM_STREAM") != nullptr;
        if (!no_stream && (gemm_stream_supported(p) || gemm_stream_rows_supported(p))) return launch_gemm_stream(p, s);
        return gemm_go<EL_I8, EPI_REQUANT>(p, grid, s);
    }
    if (el == EL_I8 && epi == EPI_HEADS_I8) return gemm_go<EL_I8, EPI_HEADS_I8>(p, grid, s);
    if (el == EL_BF16 && epi == EPI_BF16)
        return p.k_steps >= KSPLIT_PARTS ? gemm_go<EL_BF16, EPI_BF16, KSPLIT_PARTS>(p, grid, s) : gemm_go<EL_BF16, EPI_BF16>(p, grid, s);
    if (el == EL_BF16 && epi == EPI_HEADS_F32ACC) return gemm_go<EL_BF16, EPI_HEADS_F32ACC>(p, grid, s);
    if (el == EL_BF16 && epi == EPI_LSTM) return gemm_go<EL_BF16, EPI_LSTM>(p, grid, s);
    return hipErrorInvalidValue;
}

}  // namespace accerl
