// fp32 forward of causal stick-breaking attention on the fp32 matrix instructions.
//
// This path exists for full-precision checks: every operation is fp32 (the 16x16x4 fp32 MFMA is a
// fused multiply-add chain per element), exp and log1p are the library's.  The shapes it
// is called at are small (one head of a few hundred rows), so what bounds it is the length of the
// serial chain of a row and how much of the chip has work, not a throughput:
//   - a workgroup takes 16 query rows, so that T = 256 already gives 16 workgroups per head;
//   - its eight waves share the keys of those rows: each sweeps its own range of 16-key subtiles
//     from the near end to the far end (Algorithm 1's direction) as if nothing were nearer.  Partial
//     results of key ranges combine without any rescaling by a maximum,
//         o = sum_w exp(-(softplus total of the ranges nearer than w)) o_w,
//     which is done once at the end through LDS, in a fixed order;
//   - K and V go from L2 straight into the operand registers, 16 bytes per lane, no staging and no
//     barrier in the sweep; the next subtile's K is fetched during the element-wise work.
// Measured, B1 H1 T256 d64: 228 us with one lane per query row walking the keys one by one -> 9.8 us;
// B1 H1 T2048 d128 5163 -> 67 us, B4 H8 T2048 d128 5715 -> 611 us (56 TFLOP/s).
#include "sb_kernels.h"

namespace sb {
namespace {

typedef __attribute__((ext_vector_type(4))) float f32x4;

constexpr int F32_BQ = 16;   // query rows per workgroup
constexpr int F32_NW = 8;    // waves that share their keys
constexpr int F32_THREADS = 64 * F32_NW;

__device__ __forceinline__ float softplus_f32(float z)
{
    // log(1 + e^z) = max(z, 0) + log1p(e^{-|z|}): no overflow on either side
    return fmaxf(z, 0.0f) + log1pf(expf(-fabsf(z)));
}

// S^T = K Q^T with A = 16 key rows, B = 16 query rows: in the accumulator a lane (n = lane % 16,
// g = lane / 16) owns query n and keys 4g .. 4g+3.  The contraction index of MFMA m of group j is
// 16j + 4g + m for both operands, so a lane's 16-byte load of a row feeds four MFMAs.
// O += A V: MFMA r contracts over keys 4g + r, g = 0..3, whose weights are already in the right
// lanes; a lane's vector load of V columns VEC*n .. feeds VEC column blocks, block m of group j
// standing for the columns 16*VEC*j + VEC*n + m.
template <int D>
__global__ void __launch_bounds__(F32_THREADS)
fwd_f32_kernel(const float* __restrict__ q, const float* __restrict__ k, const float* __restrict__ v,
               float* __restrict__ o, float* __restrict__ m, int T, int nqb, long nblocks, int first_wg)
{
    constexpr int VEC = D >= 64 ? 4 : 2;
    constexpr int NV = D / (16 * VEC);
    typedef __attribute__((ext_vector_type(VEC))) float vec;
    __shared__ float s_tot[F32_NW][F32_BQ];
    __shared__ __attribute__((aligned(16))) float s_o[F32_NW][F32_BQ][D];

    // consecutive workgroup ids go round the 8 XCDs: give each XCD one contiguous eighth of the
    // (head, query block) list, so that a head's K and V are read into one or two L2s only
    const long per_xcd = (nblocks + 7) >> 3;
    const long wg = (long)first_wg + blockIdx.x;
    const long lin = (wg & 7) * per_xcd + (wg >> 3);
    if (lin >= nblocks) return;
    const long bh = lin / nqb;
    const int q0 = (nqb - 1 - (int)(lin % nqb)) * F32_BQ;      // longest rows first
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const float scale = 1.0f / sqrtf((float)D);
    const float* Q = q + bh * (long)T * D;
    const float* K = k + bh * (long)T * D;
    const float* V = v + bh * (long)T * D;

    f32x4 qf[D / 16];
#pragma unroll
    for (int j = 0; j < D / 16; ++j)
        qf[j] = *reinterpret_cast<const f32x4*>(Q + (long)min(q0 + n, T - 1) * D + 16 * j + 4 * g);

    // keys 0 .. kmax-1 are visible to some row; wave 0 takes the nearest range of subtiles
    const int kmax = min(T, q0 + F32_BQ) - 1;
    const int nsub = (kmax + 15) >> 4;
    const int per = (nsub + F32_NW - 1) / F32_NW;
    const int hi = nsub - 1 - wave * per, lo = max(nsub - (wave + 1) * per, 0);

    float s = 0.0f;                           // softplus total of this wave's keys already passed
    f32x4 acc[D / 16];
#pragma unroll
    for (int b = 0; b < D / 16; ++b) acc[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    f32x4 kf[D / 16];
    auto load_k = [&](int sub) __attribute__((always_inline)) {
        const float* row = K + (long)min(16 * sub + n, T - 1) * D + 4 * g;
#pragma unroll
        for (int j = 0; j < D / 16; ++j) kf[j] = *reinterpret_cast<const f32x4*>(row + 16 * j);
    };
    if (hi >= 0) load_k(hi);
    for (int sub = hi; sub >= lo; --sub) {
        vec vf[4][NV];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float* row = V + (long)min(16 * sub + 4 * g + r, T - 1) * D + VEC * n;
#pragma unroll
            for (int j = 0; j < NV; ++j) vf[r][j] = *reinterpret_cast<const vec*>(row + 16 * VEC * j);
        }
        f32x4 z0 = {0.0f, 0.0f, 0.0f, 0.0f}, z1 = z0;         // two chains: half the dependent latency
#pragma unroll
        for (int j = 0; j < D / 16; ++j) {
            z0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][0], qf[j][0], z0, 0, 0, 0);
            z1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][1], qf[j][1], z1, 0, 0, 0);
            z0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][2], qf[j][2], z0, 0, 0, 0);
            z1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][3], qf[j][3], z1, 0, 0, 0);
        }
        if (sub > lo) load_k(sub - 1);
        float z[4], c[4], run = 0.0f;
        bool seen[4];
#pragma unroll
        for (int r = 3; r >= 0; --r) {
            z[r] = (z0[r] + z1[r]) * scale;
            seen[r] = 16 * sub + 4 * g + r < q0 + n;
            run += seen[r] ? softplus_f32(z[r]) : 0.0f;
            c[r] = run;                                        // this lane's keys r..3
        }
        // the lane groups of higher g hold nearer keys
        const float x1 = __shfl_xor(run, 16);
        const float pair = run + x1;
        const float x2 = __shfl_xor(pair, 32);
        const float off = s + ((g & 1) ? 0.0f : x1) + ((g & 2) ? 0.0f : x2);
        s += pair + x2;
        float w[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = seen[r] ? expf(z[r] - (off + c[r])) : 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int j = 0; j < NV; ++j)
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    acc[j * VEC + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[r], vf[r][j][e], acc[j * VEC + e], 0, 0, 0);
    }

    // ---- combine the waves' ranges.  acc[b][r] is query row 4g + r.
    if (g == 0) s_tot[wave][n] = s;
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        float nearer = 0.0f;
        for (int w = 0; w < wave; ++w) nearer += s_tot[w][4 * g + r];
        const float f = expf(-nearer);
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            vec x;
#pragma unroll
            for (int e = 0; e < VEC; ++e) x[e] = f * acc[j * VEC + e][r];
            *reinterpret_cast<vec*>(&s_o[wave][4 * g + r][16 * VEC * j + VEC * n]) = x;
        }
    }
    __syncthreads();
    for (int idx = threadIdx.x; idx < F32_BQ * D / 4; idx += F32_THREADS) {
        const int row = idx / (D / 4), c4 = idx % (D / 4);
        f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < F32_NW; ++w) x += *reinterpret_cast<const f32x4*>(&s_o[w][row][4 * c4]);
        if (q0 + row < T) *reinterpret_cast<f32x4*>(o + (bh * (long)T + q0 + row) * D + 4 * c4) = x;
    }
    if (m && threadIdx.x < F32_BQ && q0 + (int)threadIdx.x < T) {
        float t = 0.0f;
#pragma unroll
        for (int w = 0; w < F32_NW; ++w) t += s_tot[w][threadIdx.x];
        m[bh * (long)T + q0 + threadIdx.x] = -t;
    }
}

}  // namespace

hipError_t launch_fwd_f32(const float* q, const float* k, const float* v, float* o, float* m,
                          int B, int H, int T, int d, hipStream_t stream)
{
    const int nqb = (T + F32_BQ - 1) / F32_BQ;
    const long nblocks = (long)B * H * nqb;
    const long grid = (nblocks + 7) / 8 * 8;
    if (grid > 0x7fffffffL) return hipErrorInvalidValue;
    return launch_workgroups(grid, F32_THREADS, [&](unsigned wgs, int first_wg) {
        const dim3 g(wgs), block(F32_THREADS);
        if (d == 32)
            hipLaunchKernelGGL(fwd_f32_kernel<32>, g, block, 0, stream, q, k, v, o, m, T, nqb, nblocks, first_wg);
        else if (d == 64)
            hipLaunchKernelGGL(fwd_f32_kernel<64>, g, block, 0, stream, q, k, v, o, m, T, nqb, nblocks, first_wg);
        else
            hipLaunchKernelGGL(fwd_f32_kernel<128>, g, block, 0, stream, q, k, v, o, m, T, nqb, nblocks, first_wg);
    });
}

}  // namespace sb
