// fp32 forward of causal stick-breaking attention on the fp32 matrix instructions.
//
// This path exists for full-precision checks: every operation is fp32 (the 16x16x4 fp32 MFMA is a
// fused multiply-add chain per element), exponential and logarithm are good to an ulp.  The shapes it
// is called at are small (one head of a few hundred rows), so what bounds it is the length of the
// serial chain of a row and how much of the chip has work, not a throughput:
//   - a workgroup takes 16 query rows, so that T = 256 already gives 16 workgroups per head;
//   - its eight waves share the keys of those rows: each sweeps its own range of 16-key subtiles
//     from the near end to the far end (Algorithm 1's direction) as if nothing were nearer.  Partial
//     results of key ranges combine without any rescaling by a maximum,
//         o = sum_w exp(-(softplus total of the ranges nearer than w)) o_w,
//     which is done once at the end through LDS, in a fixed order;
//   - V goes from L2 straight into the operand registers, whole rows a load, K through LDS, every wave its own subtile,
//     asked for again as soon as it is in registers; no barrier in the sweep.  (A load whose lanes are the rows of
//     the operand brings a CU 15 bytes a clock, one whose lanes lie side by side 55.)
// Measured, B1 H1 T256 d64: 228 us with one lane per query row walking the keys one by one -> 9.8 us;
// B1 H1 T2048 d128 5163 -> 66 us, B4 H8 T2048 d128 5715 -> 603 us.  With K and Q by whole rows and exponential and logarithm
// of its own: 9.8 -> 6.5, 66 -> 50, 605 -> 443 us (78 TFLOP/s); B4 H8 T2048 d32 279 -> 166 us.  Against fp64 the error of o
// is at most what it was with the library's functions, a third less where logits are of the order of 1.  With the logarithm as a polynomial, the longest rows of all
// heads first and masks on the diagonal alone (d <= 64): 6.5 -> 6.1, 49.7 -> 48.3, 442 -> 440, 166 -> 131 us; B1 H3 T1984 d32 37 -> 24.
#include <type_traits>

#include "sb_kernels.h"
#include "sb_mma.h"
#include "sb_share.h"

namespace sb {
namespace {

constexpr int F32_BQ = 16;   // query rows per workgroup
constexpr int F32_NW = 8;    // waves that share their keys
constexpr int F32_THREADS = 64 * F32_NW;

// e^x for the x <= 0 that occur here, to about an ulp: what the rounding of x log2(e) and of log2(e) itself leaves
// over is put back to first order.  (The library's expf and log1pf, 30 and 100 instructions with branches, took half the
// time of a subtile.)  v_exp_f32 gives no subnormals: with LOW, where the result may be one, it is taken 2^64 times as large.
template <bool LOW> __device__ __forceinline__ float exp_f32(float x)
{
    constexpr float L = 1.44269504088896340736f, LO = (float)(1.44269504088896340736 - (double)L);
    const float p = x * L;
    const float rest = __builtin_fmaf(x, LO, __builtin_fmaf(x, L, -p));
    const bool low = LOW && p < -126.0f;
    const float r = fast_exp2(low ? p + 64.0f : p);
    const float e = __builtin_fmaf(r * rest, SB_LN2, r);
    if constexpr (!LOW) return e;
    return r == 0.0f ? 0.0f : __builtin_amdgcn_ldexpf(e, low ? -64 : 0);      // (x = -inf: rest is not a number)
}
// of four: with LOW where one of a wave's is below log(2^-126) (in every case, us: B1 H1 T256 d64 6.9 in place of 6.5)
__device__ __forceinline__ void exp_of_four(float (&x)[4])
{
    const bool low = fminf(fminf(x[0], x[1]), fminf(x[2], x[3])) < -87.3f;
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(low) != 0, 0)) {
#pragma unroll
        for (int r = 0; r < 4; ++r) x[r] = exp_f32<true>(x[r]);
        return;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = exp_f32<false>(x[r]);
}
// log(1 + e), 0 <= e <= 1, as e - e^2 P(e): P of degree 9 by a least maximum of the error relative to the sum, its coefficients rounded one after the other (9e-10 of
// the sum with those below).  2 atanh(e / (2 + e)) by its series takes a reciprocal and nine instructions more, a fifth of what a logit costs on the vector ALU: B4 H8 T2048 d32
// 149 -> 131 us, B1 H1 T256 d64 6.3 -> 6.1.  Against 64 bits, series / polynomial: given e, with an exact reciprocal, 2.6e-8 / 2.8e-8 in the mean square, 6.8e-8 / 9.7e-8 at most; on the card, of e^z
// for 65536 z each, -z below 1e-3 3.5e-8 / 3.3e-8, 1.07e-7 / 1.15e-7, below 1 4.2e-8 / 3.6e-8, 1.6e-7 / 1.2e-7, below 4 4.8e-8 / 4.1e-8, 2.0e-7 / 1.6e-7, 4 to 12 5.1e-8 / 4.4e-8, 2.3e-7 / 1.8e-7;  of o and m
// (d 32 to 128, T 40 to 1500, logits near 0, of order 1, times three and ten, far) 0.99 to 1.001 and 0.97 to 1.004 of what they were in the mean of each kind.
__device__ __forceinline__ float log1p_f32(float e)
{
    float p = -0.00208444008604f;
    p = __builtin_fmaf(p, e, 0.01369118690491f);
    p = __builtin_fmaf(p, e, -0.04211390763521f);
    p = __builtin_fmaf(p, e, 0.08323805034161f);
    p = __builtin_fmaf(p, e, -0.12479481101036f);
    p = __builtin_fmaf(p, e, 0.16135157644749f);
    p = __builtin_fmaf(p, e, -0.19899621605873f);
    p = __builtin_fmaf(p, e, 0.24988864362240f);
    p = __builtin_fmaf(p, e, -0.33332714438438f);
    p = __builtin_fmaf(p, e, 0.49999988079071f);
    return __builtin_fmaf(-(e * e), p, e);
}
// Rows of fp32 in LDS: byte offset of 16-byte chunk c of row `row`, the chunk xor-ed so that 16 lanes that read the same chunk of
// 16 rows meet different banks.
template <int D> __device__ __forceinline__ int f32_off(int row, int c)
{
    return row * (4 * D) + ((c ^ (D >= 64 ? row & 15 : (row >> 1) & 7)) << 4);
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
               float* __restrict__ o, float* __restrict__ m, int T, int nqb, int heads, int run, int first_wg)
{
    constexpr int VEC = D >= 64 ? 4 : 2;
    constexpr int NV = D / (16 * VEC);
    typedef __attribute__((ext_vector_type(VEC))) float vec;
    constexpr int RB = 4 * D, CPR = RB / 16;              // bytes and 16-byte chunks of a row
    constexpr int SUB = 16 * RB, LOADS = SUB / 1024;      // of a subtile of 16 rows; its loads by a wave
    __shared__ __attribute__((aligned(16))) float s_tot[F32_NW][F32_BQ];
    __shared__ __attribute__((aligned(1024))) char s_q[SUB];
    __shared__ __attribute__((aligned(1024))) char s_k[F32_NW * SUB];       // the waves' subtiles, later their partial results
    float (*const s_o)[F32_BQ][D] = reinterpret_cast<float (*)[F32_BQ][D]>(s_k);
    static_assert(SUB == F32_BQ * D * 4, "a wave's partial result takes the place of its subtile");

    const unsigned wg = (unsigned)first_wg + blockIdx.x;
    const Share sh = in_scalars(run == EIGHTHS ? share_in_eighths(wg, heads, nqb) : share_of(wg, heads, run));
    if (sh.bh >= heads) return;
    const long bh = sh.bh;
    const int q0 = (nqb - 1 - sh.i) * F32_BQ;                  // longest rows first
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, g = lane >> 4;
    const float scale = 1.0f / sqrtf((float)D);
    const float* Q = q + bh * (long)T * D;
    const float* K = k + bh * (long)T * D;
    const float* V = v + bh * (long)T * D;

    // keys 0 .. kmax-1 are visible to some row; wave 0 takes the nearest range of subtiles
    const int kmax = min(T, q0 + F32_BQ) - 1;
    const int nsub = (kmax + 15) >> 4;
    const int per = (nsub + F32_NW - 1) / F32_NW;
    const int hi = nsub - 1 - wave * per, lo = max(nsub - (wave + 1) * per, 0);

    float s = 0.0f;                           // softplus total of this wave's keys already passed
    f32x4 acc[D / 16];
#pragma unroll
    for (int b = 0; b < D / 16; ++b) acc[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    // load i of the 16 rows from `row0` of X on (those past T clamped)
    auto stage = [&](const float* X, int row0, int i, uint32_t at) __attribute__((always_inline)) {
        const int row = i * (1024 / RB) + lane / CPR;
        const int off = min(row, T - 1 - row0) * RB + (((lane % CPR) ^ (D >= 64 ? row & 15 : (row >> 1) & 7)) << 4);
        dma16_to_lds_at(scalar_base(X + (long)row0 * D), off, at + i * 1024);
    };
    const uint32_t q_at = lds_offset(s_q), k_at = lds_offset(s_k) + wave * SUB;
    auto load_k = [&](int sub) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < LOADS; ++i) stage(K, 16 * sub, i, k_at);
    };
    for (int i = wave; i < LOADS; i += F32_NW) stage(Q, q0, i, q_at);
    if (hi >= lo) load_k(hi);
    dma_wait<0>();
    barrier_nofence();
    f32x4 qf[D / 16], kf[D / 16];
    const uint32_t row_at = f32_off<D>(n, g);                 // chunk 4j + g: ^ (j << 6)
#pragma unroll
    for (int j = 0; j < D / 16; ++j) qf[j] = __builtin_bit_cast(f32x4, lds_load16((q_at + row_at) ^ (j << 6)));
    auto step = [&](auto masked, int sub) __attribute__((always_inline)) {
        dma_wait<0>();                                        // K has landed
        vec vf[4][NV];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const float* row = V + (long)min(16 * sub + 4 * g + r, T - 1) * D + VEC * n;
#pragma unroll
            for (int j = 0; j < NV; ++j) vf[r][j] = *reinterpret_cast<const vec*>(row + 16 * VEC * j);
        }
#pragma unroll
        for (int j = 0; j < D / 16; ++j) kf[j] = __builtin_bit_cast(f32x4, lds_load16((k_at + row_at) ^ (j << 6)));
        if (sub > lo) {
            asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");       // ... and is in registers
            load_k(sub - 1);
        }
        f32x4 z0 = {0.0f, 0.0f, 0.0f, 0.0f}, z1 = z0;         // two chains: half the dependent latency
#pragma unroll
        for (int j = 0; j < D / 16; ++j) {
            z0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][0], qf[j][0], z0, 0, 0, 0);
            z1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][1], qf[j][1], z1, 0, 0, 0);
            z0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][2], qf[j][2], z0, 0, 0, 0);
            z1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[j][3], qf[j][3], z1, 0, 0, 0);
        }
        float z[4], e[4], x[4], c[4], run = 0.0f;              // x: log sigmoid(z); c: this lane's keys r+1..3
        bool seen[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            z[r] = (z0[r] + z1[r]) * scale;
            asm("" : "+v"(z[r]));                              // rounded, the same in every use
            e[r] = -fabsf(z[r]);
        }
        exp_of_four(e);
#pragma unroll
        for (int r = 3; r >= 0; --r) {
            seen[r] = !decltype(masked)::value || 16 * sub + 4 * g + r < q0 + n;
            // softplus(z) = max(z, 0) + log(1 + e^{-|z|}); z less that, each part by itself, loses nothing where z is large
            const float over = fmaxf(z[r], 0.0f), l = log1p_f32(e[r]);
            x[r] = (z[r] - over) - l;
            c[r] = run;
            run += seen[r] ? over + l : 0.0f;
        }
        // the lane groups of higher g hold nearer keys
        const float x1 = __shfl_xor(run, 16);
        const float pair = run + x1;
        const float x2 = __shfl_xor(pair, 32);
        const float off = s + ((g & 1) ? 0.0f : x1) + ((g & 2) ? 0.0f : x2);
        s += pair + x2;
        float w[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = x[r] - (off + c[r]);
        exp_of_four(w);
#pragma unroll
        for (int r = 0; r < 4; ++r) w[r] = seen[r] ? w[r] : 0.0f;
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int j = 0; j < NV; ++j)
#pragma unroll
                for (int e = 0; e < VEC; ++e)
                    acc[j * VEC + e] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[r], vf[r][j][e], acc[j * VEC + e], 0, 0, 0);
    };
    int sub = hi;
    if constexpr (D < 128)                                     // (the matrix pipe bounds d = 128: twice the code cost 3 % of a short call there)
        if (sub >= lo && 16 * sub == q0) step(std::true_type(), sub--);       // the one subtile that not every row sees all of
    for (; sub >= lo; --sub) step(std::bool_constant<D == 128>(), sub);

    // ---- combine the waves' ranges.  acc[b][r] is query row 4g + r.
    if (g == 0) s_tot[wave][n] = s;
    __syncthreads();
    f32x4 tot[F32_NW], nearer = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int w = 0; w < F32_NW; ++w) tot[w] = *reinterpret_cast<const f32x4*>(&s_tot[w][4 * g]);
#pragma unroll
    for (int w = 0; w < F32_NW; ++w)
        if (w < wave) nearer += tot[w];
    float f[4] = {-nearer[0], -nearer[1], -nearer[2], -nearer[3]};
    exp_of_four(f);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            vec x;
#pragma unroll
            for (int e = 0; e < VEC; ++e) x[e] = f[r] * acc[j * VEC + e][r];
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
    const int heads = B * H, nqb = (T + F32_BQ - 1) / F32_BQ;
    const int run = f32_run(heads, nqb, T, d);
    const long grid = run == EIGHTHS ? ((long)heads * nqb + 7) / 8 * 8 : (long)heads * nqb;
    if (grid > 0x7fffffffL) return hipErrorInvalidValue;
    return launch_workgroups(grid, F32_THREADS, [&](unsigned wgs, int first_wg) {
        const dim3 g(wgs), block(F32_THREADS);
        if (d == 32)
            hipLaunchKernelGGL(fwd_f32_kernel<32>, g, block, 0, stream, q, k, v, o, m, T, nqb, heads, run, first_wg);
        else if (d == 64)
            hipLaunchKernelGGL(fwd_f32_kernel<64>, g, block, 0, stream, q, k, v, o, m, T, nqb, heads, run, first_wg);
        else
            hipLaunchKernelGGL(fwd_f32_kernel<128>, g, block, 0, stream, q, k, v, o, m, T, nqb, heads, run, first_wg);
    });
}

}  // namespace sb
