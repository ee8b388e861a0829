// Gate-weighted unpermute / combine (paper Sec. 2: y = sum_i G(x)_i * E_i(x)), the shared-expert term, and the
// sigmoid gate in front of a gated shared expert (evaluated inside the combine).  fp32, fixed slot order, no atomics: same bits on every run.
#include "kernels.hpp"

namespace lexi {

template <int N> struct Count { static constexpr int value = N; };

// u = h * inv rounded to the layer dtype, four consecutive elements (the chained stack's normalised MoE input).
template <bool U_BF16>
__device__ __forceinline__ void store_normalised(void* u, size_t idx, const f32x4_t& v, float inv) {
    if (U_BF16) {
        u32x2_t pk;
        pk[0] = pack_bf16x2(v[0] * inv, v[1] * inv);
        pk[1] = pack_bf16x2(v[2] * inv, v[3] * inv);
        *(u32x2_t*)((bf16_t*)u + idx) = pk;
    } else {
        f32x4_t o;
#pragma unroll
        for (int i = 0; i < 4; ++i) o[i] = v[i] * inv;
        *(f32x4_t*)((float*)u + idx) = o;
    }
}

// One workgroup per token; each thread owns 4 consecutive output features in each of NP pieces of 1024.  For a sigmoid-gated
// shared expert the workgroup first evaluates its token's gate coefficient 1 / (1 + exp(-(x[t] . w_sg))) itself (wave sums
// by DPP, the four wave results added in wave order), which saves a launch.  It stands in front of the slot rows: a thread
// adds up elements j, j + 256, ..., chains of d / 256 however narrow the row is, and requests eight of x and of w_sg together (one of each
// at a time: 64 tokens 7.7 us instead of 6.0, 8192 tokens, two slots 52 instead of 42).  16 bytes a thread as eight neighbouring
// elements are no faster (+-1 % of the call) and round differently; through LDS to the same sums they cost 0.4 us.
// Bound by reading the k slot rows (HBM) for many tokens, by latency for few: the rows of GS slots in NP pieces are
// requested together, and the shared expert's row and the hidden state before them (16 tokens, chained: 6.8 -> 4.0 us; 256
// tokens: 6.5 -> 5.0 us).
// Chained stack: `residual` (the hidden state) is added to the block's output, and with `u_next` the same workgroup
// also writes the NEXT block's normalised input from the row it has just produced -- the sum of squares in exactly
// the order start_chain_kernel uses, so either route gives the same bits.  (x and u_next may be the same buffer: a
// workgroup reads its row of x before it writes its row of u_next.)
template <bool Y_BF16, bool X_BF16, int NP, int GS>
__global__ void __launch_bounds__(256)
combine_kernel(const float* __restrict__ y_slot, const int32_t* __restrict__ inv_perm, const float* __restrict__ gates,
               const float* __restrict__ y_shared, const void* x, const void* __restrict__ w_shared_gate,
               const float* residual, int d, int k, void* y, void* u_next, float eps, int slot_planes,
               size_t slot_plane_stride, int shared_planes, size_t shared_plane_stride) {
    __shared__ float wave_part[4];
    const int t = blockIdx.x;
    const int32_t* ip = inv_perm + (size_t)t * k;
    const float* gt = gates + (size_t)t * k;
    float coef = (y_shared != nullptr) ? 1.0f : 0.0f;
    if (y_shared != nullptr && w_shared_gate != nullptr) {
        float acc = 0.0f;
        for (int j = threadIdx.x; j < d; j += 2048) {
            float a[8], b[8];
#pragma unroll
            for (int m = 0; m < 8; ++m) {               // (past the row: element j again, unused)
                const int e = j + 256 * m < d ? j + 256 * m : j;
                a[m] = load_as_f32<X_BF16>(x, (size_t)t * d + e);
                b[m] = load_as_f32<X_BF16>(w_shared_gate, (size_t)e);
            }
#pragma unroll
            for (int m = 0; m < 8; ++m)
                if (j + 256 * m < d) acc = __builtin_fmaf(a[m], b[m], acc);
        }
        const float ws = wave_sum(acc);
        if ((threadIdx.x & 63) == 0) wave_part[threadIdx.x >> 6] = ws;
        __syncthreads();
        const float z = ((wave_part[0] + wave_part[1]) + wave_part[2]) + wave_part[3];
        coef = 1.0f / (1.0f + __expf(-z));
    }
    const bool one_round = d <= 1024 * NP;              // the row fits the registers
    float ss = 0.0f;
    f32x4_t acc[NP];
    for (int c0 = 0; c0 < d; c0 += 1024 * NP) {
        int j[NP];                                      // (pieces past the row all read its first 16 bytes; never stored)
        bool on[NP];
        f32x4_t sh[NP], hid[NP];
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            j[p] = c0 + 1024 * p + threadIdx.x * 4;
            on[p] = j[p] < d;
            if (!on[p]) j[p] = 0;
            acc[p] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
            if (y_shared != nullptr) sh[p] = *(const f32x4_t*)(y_shared + (size_t)t * d + j[p]);
            if (residual != nullptr) hid[p] = *(const f32x4_t*)(residual + (size_t)t * d + j[p]);
        }
        auto slots = [&](int s0, auto n_tag) {          // slots s0 .. s0 + N - 1, in slot order = rank order
            constexpr int N = decltype(n_tag)::value;
            f32x4_t v[N][NP];
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const float* row = y_slot + (size_t)ip[s0 + u] * d;
#pragma unroll
                for (int p = 0; p < NP; ++p) v[u][p] = *(const f32x4_t*)(row + j[p]);
            }
            for (int q = 1; q < slot_planes; ++q) {     // the down GEMM's reduction was cut: the parts are added first
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    const float* row = y_slot + q * slot_plane_stride + (size_t)ip[s0 + u] * d;
#pragma unroll
                    for (int p = 0; p < NP; ++p) {
                        const f32x4_t v1 = *(const f32x4_t*)(row + j[p]);
#pragma unroll
                        for (int i = 0; i < 4; ++i) v[u][p][i] = v[u][p][i] + v1[i];
                    }
                }
            }
#pragma unroll
            for (int u = 0; u < N; ++u) {
                const float g = gt[s0 + u];
#pragma unroll
                for (int p = 0; p < NP; ++p)
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[p][i] = __builtin_fmaf(g, v[u][p][i], acc[p][i]);
            }
        };
        int s = 0;
        for (; s + GS <= k; s += GS) slots(s, Count<GS>{});
        if (GS > 4 && s + 4 <= k) { slots(s, Count<4>{}); s += 4; }
        if (s + 2 <= k) { slots(s, Count<2>{}); s += 2; }
        if (s < k) slots(s, Count<1>{});
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            if (y_shared != nullptr) {
                for (int q = 1; q < shared_planes; ++q) {
                    const f32x4_t v1 = *(const f32x4_t*)(y_shared + q * shared_plane_stride + (size_t)t * d + j[p]);
#pragma unroll
                    for (int i = 0; i < 4; ++i) sh[p][i] = sh[p][i] + v1[i];
                }
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[p][i] = __builtin_fmaf(coef, sh[p][i], acc[p][i]);
            }
            if (residual != nullptr) {   // chained stack: the hidden state plus this block's output (may alias y: same element)
#pragma unroll
                for (int i = 0; i < 4; ++i) acc[p][i] = hid[p][i] + acc[p][i];
            }
            if (!on[p]) continue;
#pragma unroll
            for (int i = 0; i < 4; ++i) ss = __builtin_fmaf(acc[p][i], acc[p][i], ss);
            if (Y_BF16) {
                u32x2_t pk;
                pk[0] = pack_bf16x2(acc[p][0], acc[p][1]);
                pk[1] = pack_bf16x2(acc[p][2], acc[p][3]);
                *(u32x2_t*)((bf16_t*)y + (size_t)t * d + j[p]) = pk;
            } else {
                *(f32x4_t*)((float*)y + (size_t)t * d + j[p]) = acc[p];
            }
        }
    }
    if (Y_BF16 || u_next == nullptr) return;   // (the chained stack keeps its hidden state in fp32)
    __syncthreads();                            // wave_part may still be read for the gate coefficient
    const float ws = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) wave_part[threadIdx.x >> 6] = ws;
    __syncthreads();
    const float total = ((wave_part[0] + wave_part[1]) + wave_part[2]) + wave_part[3];
    const float inv = 1.0f / sqrtf(total / (float)d + eps);
    if (one_round) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int j = 1024 * p + threadIdx.x * 4;
            if (j < d) store_normalised<X_BF16>(u_next, (size_t)t * d + j, acc[p], inv);
        }
        return;
    }
    for (int j = threadIdx.x * 4; j < d; j += 256 * 4) {
        const f32x4_t v = *(const f32x4_t*)((const float*)y + (size_t)t * d + j);   // this thread's own stores
        store_normalised<X_BF16>(u_next, (size_t)t * d + j, v, inv);
    }
}

template <bool Y_BF16, bool X_BF16>
static void launch_combine_t(const CombineArgs& a, hipStream_t s) {
    auto launch = [&](auto np, auto gs) {
        hipLaunchKernelGGL((combine_kernel<Y_BF16, X_BF16, decltype(np)::value, decltype(gs)::value>), dim3(a.T), dim3(256), 0, s,
                           a.y_slot, a.inv_perm, a.gates, a.y_shared, a.x, a.w_shared_gate, a.residual, a.d, a.k, a.y, a.u_next,
                           kRmsEps, a.slot_planes, a.slot_plane_stride, a.shared_planes, a.shared_plane_stride);
    };
    // Many tokens: few loads per thread in few registers, the other workgroups of the CU cover the latency.  (8192 tokens, two
    // or four slots, gated shared expert: 83 us, against 92 with eight slots and 104 with two pieces of them.)
    if (a.T > 1024) launch(Count<1>{}, Count<4>{});
    else if (a.d <= 1024) launch(Count<1>{}, Count<8>{});
    else if (a.d <= 2048) launch(Count<2>{}, Count<8>{});
    else launch(Count<4>{}, Count<4>{});
}

// The start of a chained stack: h = x widened exactly to fp32 (the hidden state starts as the input), and u[t] = h[t] / sqrt(mean_j h[t][j]^2
// + eps) rounded to the layer dtype.  One workgroup per token; the sum of squares in combine_kernel's order (per-thread strided fused
// multiply-adds, DPP tree, the four waves in order).  A thread reads its four pieces of x together and keeps them (a wider row is read again
// from h, the thread's own stores).  A thread reads and writes only its own pieces of a row: u may be x, and so may h where x is fp32.
// Widening in a launch of its own cost a launch for few tokens and a pass over h for many: 1 token of d 2048 4.3 -> 2.0 us, 777 of d 1280
// 7.5 -> 4.3, 4096 of d 4096 48.4 -> 20.4 (134 MB at 6.6 TB/s), of d 8192 119 -> 66.
template <bool X_BF16>
__global__ void __launch_bounds__(256)
start_chain_kernel(const void* x, int d, float eps, float* h, void* u) {
    constexpr int NP = 4;
    __shared__ float wave_part[4];
    constexpr int ES = X_BF16 ? 2 : 4;
    const size_t row = (size_t)blockIdx.x * d;
    // (a buffer of this row alone: lanes past its end read nothing)
    const auto x_row = __builtin_amdgcn_make_buffer_rsrc((void*)((const char*)x + row * ES), 0, (unsigned)d * ES, 0x00020000);
    f32x4_t v[NP];
    float ss = 0.0f;
    for (int c0 = 0; c0 < d; c0 += 1024 * NP) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int j = c0 + 1024 * p + threadIdx.x * 4;
            if constexpr (X_BF16) {
                const u32x2_t pk = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(x_row, (unsigned)j * ES, 0, 0));
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    v[p][2 * i] = __uint_as_float(pk[i] << 16);
                    v[p][2 * i + 1] = __uint_as_float(pk[i] & 0xFFFF0000u);
                }
            } else {
                v[p] = __builtin_bit_cast(f32x4_t, __builtin_amdgcn_raw_buffer_load_b128(x_row, (unsigned)j * ES, 0, 0));
            }
        }
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int j = c0 + 1024 * p + threadIdx.x * 4;
            if (j >= d) continue;
            *(f32x4_t*)(h + row + j) = v[p];
#pragma unroll
            for (int i = 0; i < 4; ++i) ss = __builtin_fmaf(v[p][i], v[p][i], ss);
        }
    }
    const float ws = wave_sum(ss);
    if ((threadIdx.x & 63) == 0) wave_part[threadIdx.x >> 6] = ws;
    __syncthreads();
    const float total = ((wave_part[0] + wave_part[1]) + wave_part[2]) + wave_part[3];
    const float inv = 1.0f / sqrtf(total / (float)d + eps);
    if (d <= 1024 * NP) {
#pragma unroll
        for (int p = 0; p < NP; ++p) {
            const int j = 1024 * p + threadIdx.x * 4;
            if (j < d) store_normalised<X_BF16>(u, row + j, v[p], inv);
        }
        return;
    }
    for (int j = threadIdx.x * 4; j < d; j += 1024) store_normalised<X_BF16>(u, row + j, *(const f32x4_t*)(h + row + j), inv);
}

hipError_t launch_start_chain(const void* x, bool is_bf16, int T, int d, float eps, float* h, void* u, hipStream_t s) {
    if (is_bf16) hipLaunchKernelGGL(start_chain_kernel<true>, dim3(T), dim3(256), 0, s, x, d, eps, h, u);
    else hipLaunchKernelGGL(start_chain_kernel<false>, dim3(T), dim3(256), 0, s, x, d, eps, h, u);
    return hipGetLastError();
}

hipError_t launch_combine(const CombineArgs& a, hipStream_t s) {
    if (a.y_bf16) { if (a.x_bf16) launch_combine_t<true, true>(a, s); else launch_combine_t<true, false>(a, s); }
    else          { if (a.x_bf16) launch_combine_t<false, true>(a, s); else launch_combine_t<false, false>(a, s); }
    return hipGetLastError();
}

}  // namespace lexi
