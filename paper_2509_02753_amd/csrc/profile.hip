// Stage-1 top-k perturbation profiling (paper Algorithm 1), one iteration on one input X:
//     Delta_k = || f_moe(X; k) - f_moe(X; k_base) ||_F          for every k of a list, k <= k_base.
// The selection is a total order, so TopK_k is the first k slots of TopK_{k_base}; the gates of k are the baseline
// gates of those slots renormalised over them.  One routing pass and one pass of the expert GEMMs at k_base therefore
// serve every k:
//     Y_k[t] - Y_base[t] = sum_{s < k_base} ( [s < k] * g[t][s] / P_k[t] - g[t][s] ) * y_slot[t][s],
//     P_k[t] = g[t][0] + ... + g[t][k-1]   (ascending),
// and a shared expert, which adds the same vector to both outputs, drops out.  fp32 throughout, fixed summation
// orders (same bits on every run); the final sum over tokens and the square root are taken in fp64.
#include "kernels.hpp"

namespace lexi {

// One workgroup per token: squared norm of the difference vector for every listed k -> part[i][t].
// Bound by reading the token's k_base slot rows (4 * d * k_base bytes per token), so a row element is loaded once per
// kProfileGroup listed k, whose accumulators stay in registers, and not once per k: OLMoE-shaped layer, T = 2048,
// k = 1..8, 134 MB of rows: 130 us -> 28 us (4.8 TB/s).  Eight is where one 16-byte LDS read feeds four k and the
// accumulators (32 registers) still leave eight workgroups per CU.  The coefficients [s < k] * g_s / P_k - g_s of all
// (k, slot) pairs are formed once per token in LDS; groups are padded with zero columns.
constexpr int kProfileGroup = 8;

__global__ void __launch_bounds__(256)
profile_diff_kernel(const float* __restrict__ y_slot, const int32_t* __restrict__ inv_perm, const float* __restrict__ gates,
                    int T, int d, int k_base, ProfileKList kl, float* __restrict__ part) {
    __shared__ __attribute__((aligned(16))) float coef[64][kProfileGroup];   // this group's coefficients, by slot
    __shared__ float wave_part[4][kProfileGroup];
    const int t = blockIdx.x;
    const int32_t* ip = inv_perm + (size_t)t * k_base;
    const float* gt = gates + (size_t)t * k_base;
    for (int i0 = 0; i0 < kl.n; i0 += kProfileGroup) {
        const int n = min(kProfileGroup, kl.n - i0);
        for (int c = threadIdx.x; c < k_base * kProfileGroup; c += 256) {
            const int s = c / kProfileGroup, i = c % kProfileGroup;
            float v = 0.0f;
            if (i < n) {
                const int k = kl.k[i0 + i];
                float pk = 0.0f;
                for (int q = 0; q < k; ++q) pk += gt[q];
                v = (s < k ? gt[s] * (1.0f / pk) : 0.0f) - gt[s];
            }
            coef[s][i] = v;
        }
        __syncthreads();
        float sq[kProfileGroup];
#pragma unroll
        for (int i = 0; i < kProfileGroup; ++i) sq[i] = 0.0f;
        for (int j = threadIdx.x * 4; j < d; j += 256 * 4) {
            f32x4_t acc[kProfileGroup];
#pragma unroll
            for (int i = 0; i < kProfileGroup; ++i) acc[i] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
            auto slot = [&](int s, const f32x4_t& v) {
                const f32x4_t c0 = *(const f32x4_t*)&coef[s][0], c1 = *(const f32x4_t*)&coef[s][4];
#pragma unroll
                for (int i = 0; i < kProfileGroup; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q) acc[i][q] = __builtin_fmaf(i < 4 ? c0[i & 3] : c1[i & 3], v[q], acc[i][q]);
            };
            int s = 0;
            for (; s + 4 <= k_base; s += 4) {   // slot order, the loads of four slots in flight
                f32x4_t v[4];
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = *(const f32x4_t*)(y_slot + (size_t)ip[s + u] * d + j);
#pragma unroll
                for (int u = 0; u < 4; ++u) slot(s + u, v[u]);
            }
            for (; s < k_base; ++s) slot(s, *(const f32x4_t*)(y_slot + (size_t)ip[s] * d + j));
#pragma unroll
            for (int i = 0; i < kProfileGroup; ++i)
#pragma unroll
                for (int q = 0; q < 4; ++q) sq[i] = __builtin_fmaf(acc[i][q], acc[i][q], sq[i]);
        }
#pragma unroll
        for (int i = 0; i < kProfileGroup; ++i) {
            const float ws = wave_sum(sq[i]);
            if ((threadIdx.x & 63) == 0) wave_part[threadIdx.x >> 6][i] = ws;
        }
        __syncthreads();                        // (also: the coefficients may be overwritten from here)
        if ((int)threadIdx.x < n) {
            const int i = threadIdx.x;
            const float v = ((wave_part[0][i] + wave_part[1][i]) + wave_part[2][i]) + wave_part[3][i];
            // k == k_base: Delta is exactly 0, whatever the rows hold
            part[(size_t)(i0 + i) * T + t] = kl.k[i0 + i] == k_base ? 0.0f : v;
        }
        __syncthreads();                        // wave_part has been read
    }
}

// One workgroup per listed k: sum of the T per-token squared norms in a fixed order (strided partial sums per thread,
// then the DPP tree and the four wave results in wave order), in fp64; delta = sqrt(sum).
__global__ void __launch_bounds__(256)
profile_reduce_kernel(const float* __restrict__ part, int T, float* __restrict__ delta) {
    __shared__ double wave_part[4];
    const float* p = part + (size_t)blockIdx.x * T;
    double s = 0.0;
    for (int t = threadIdx.x; t < T; t += 256) s += (double)p[t];
    // fixed-order tree over the 64 lanes (xor butterfly: every lane ends with the same sum)
    for (int off = 32; off >= 1; off >>= 1) {
        const int lo = __shfl_xor((int)(__double_as_longlong(s) & 0xFFFFFFFFll), off);
        const int hi = __shfl_xor((int)(__double_as_longlong(s) >> 32), off);
        s += __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
    }
    if ((threadIdx.x & 63) == 0) wave_part[threadIdx.x >> 6] = s;
    __syncthreads();
    if (threadIdx.x == 0) delta[blockIdx.x] = (float)sqrt(((wave_part[0] + wave_part[1]) + wave_part[2]) + wave_part[3]);
}

hipError_t launch_profile(const ProfileArgs& a, hipStream_t s) {
    hipLaunchKernelGGL(profile_diff_kernel, dim3(a.T), dim3(256), 0, s, a.y_slot, a.inv_perm, a.gates, a.T, a.d,
                       a.k_base, a.klist, a.part);
    hipError_t err = hipGetLastError();
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(profile_reduce_kernel, dim3(a.klist.n), dim3(256), 0, s, a.part, a.T, a.delta);
    return hipGetLastError();
}

}  // namespace lexi
