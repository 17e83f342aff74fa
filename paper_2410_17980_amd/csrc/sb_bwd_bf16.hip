// bf16 backward of causal stick-breaking attention on the gfx950 matrix cores
// (Eq. 4 evaluated tile by tile; the per-tile steps are those of Algorithm 2).
//
// Two kernels instead of Algorithm 2's single query-stationary kernel with
// atomic adds into dK and dV.  The dependency that forces the paper's atomics is
// the cumulative sum over keys inside each query row; it is cut by saving, per
// query row and per 32-key subtile, the two carried scalars
//     ca = sum of sp2 over the keys to the right of the subtile (up to the query),
//     cb = sum of G = A*(dO.v) over the keys to the left of the subtile,
// (2 floats per 32x1 strip of the attention matrix; sp2 = base-2 softplus).  With
// them any subtile can be recomputed on its own, so dK and dV are accumulated by a
// key-stationary kernel in registers and written once, with no atomics and no
// zero fill, and the result is bit-reproducible.
//
//   bwd_dq_kernel  (query-stationary, 128 query rows per block, sweep from key 0
//                   to the diagonal as Algorithm 2): recomputes A from m, forms G
//                   and dZ, accumulates dQ += dZ K, stores ca, cb.
//   bwd_dkv_kernel (key-stationary, 128 key rows per block = 32 per wave, K and V
//                   rows held in registers, sweep over query tiles from the
//                   diagonal to the end): recomputes A, G, dZ from ca, cb and
//                   accumulates dV += A^T dO, dK += dZ^T Q.
// The element-wise arithmetic runs in the linear domain inside a lane (one exponential
// and one reciprocal per element, see subtile_stage1/2); where its running product
// leaves the fp32 range (sharp logits) the wave takes the logits of that subtile once
// more from LDS and redoes its first stage in the log domain (subtile_stage1_log).
// Recomputing them there, instead of keeping the accumulator for the case, is what keeps
// the kernels within their register budget; a second launch of a log-domain variant for
// flagged blocks, which this replaces, cost 7 us a pass with nothing flagged.
// Far keys: once every row of a 32-row strip of queries has less than 2^-160 of its stick
// left, all weights and logit gradients beyond are zero (CARRY_EXHAUSTED).  The
// query-stationary pass first looks for that point from the diagonal, with the logits alone
// (find_start()), starts each wave's sweep there and leaves the 32-key strip in `first`, one
// 16-bit number per strip of queries; the key-stationary pass visits only the query tiles that
// reach its keys, and in those only the pairs of strips that reach each other.
// Which blocks a workgroup takes: share_of().  Streamed tiles are staged with direct
// global->LDS loads, double buffered, one barrier per 64-row tile.  The 1/sqrt(d)
// of dQ and dK is applied once, to the accumulators, on store.
//
// Register layout is the forward's: S^T = K Q^T and P^T = V dO^T with the
// 32x32x16 bf16 MFMA, a lane owns one query column and 16 consecutive keys, so
// both cumulative quantities are serial inside the lane plus one exchange between
// the half-waves.  dZ feeds the "query-major" product (dQ) straight from
// registers; for the "key-major" products (dK, dV) A and dZ are written to a small
// per-wave LDS scratch row-wise and read back with the transposing load.
#include <algorithm>
#include <type_traits>

#include "sb_kernels.h"
#include "sb_mma.h"
#include "sb_share.h"

namespace sb {
namespace {

constexpr int NTHREADS = 256;
constexpr int NW = 4;        // wavefronts per workgroup
constexpr int BQ = 128;      // dq kernel: query rows per block
constexpr int BKW = 128;     // dkv kernel: key rows per block (32 per wave)
constexpr int TK = 64;       // rows per staged tile (keys in the dq kernel, queries in the dkv kernel)
constexpr int SCR_MAT = 32 * 64;   // one 32x32 bf16 matrix of the A / dZ transposition scratch

// Byte offset of 16-byte chunk c (0..3) of row `row` of a scratch matrix.  16-byte LDS writes
// are taken eight lanes at a time (measured: 8 cycles per conflict-free ds_write_b128), so the
// eight rows 8i .. 8i+7 that write the same chunk together must land in eight different 16-byte
// slots of a 128-byte window: the chunk index is xor-ed with bits 1-2 of the row (rows 2j and
// 2j+1 already differ by 64 bytes).  The transposing reads take four whole rows at a time and
// do not care how a row's chunks are permuted.  Counters: no bank conflicts either way (the
// same layout with bits 2-3 of the row costs 8 conflict cycles per write).
__device__ __forceinline__ int scr_off(int row, int c)
{
    return row * 64 + ((c ^ ((row >> 1) & 3)) << 4);
}

template <bool B> using bc = std::integral_constant<bool, B>;

// ------------------------------------------------------------------ element-wise core
// One 32x32 subtile in the lane layout (query n; keys 16hh + r).
struct SubtileOut {
    bf16x8 pa[2];    // A, as MFMA operand (K-dim element e of half s <-> key 16hh + 8s + e)
    bf16x8 pz[2];    // dZ (without the 1/sqrt(d)), same layout
    float ca_right;  // sum of sp2 over the keys right of the subtile
    float g_tot;     // sum of G over the subtile's 32 keys
    float g_lo;      // and over its first 16
};

// In the linear domain inside the lane, as in the forward: with e_r = 2^{x_r}
// the chain t_r = W_r e_r, W_{r+1} = W_r + t_r over ascending keys gives
// A[r] = t_r / W_16 * 2^-(sp2 total of all nearer keys), and sigma = e / (1 + e):
// one exponential and one reciprocal per element instead of three exponentials and
// a logarithm.  W_0 = 2^-60; a chain that gets beyond 2^80 (or overflows) makes the
// caller redo the stage with subtile_stage1_log.  Two stages, so that the dO.v
// accumulator need not be live during the first:
//   stage 1 (logits only): sigma, chain.  Returns false in a lane whose chain left its range.
//   stage 2 (needs dO.v): A, G, dZ.
// sacc: q.k accumulator, pacc: dO.v accumulator.  cb: sum of G over the keys left
// of the subtile.  ca: sum of sp2 over the keys right of the subtile, or, with
// CA_INCLUDES_SUBTILE, over the subtile's own keys as well (Algorithm 2 carries
// that and subtracts the subtile's total before use).  With MASK, key 16hh + r is
// visible to query n iff 16hh + r < n (the subtile on the diagonal).
struct Chain {
    float be[16];    // sigma(z)
    float t[16];     // chain terms: A = t * 2^-(norm + sp2 total of all nearer lanes' keys); later G
    float l;         // sp2 total of this lane's 16 keys
    float norm;      // log2 of what t is still to be divided by
};

// sigma = e / (1 + e) = t_r / W_{r+1}, with the 16 reciprocals from ONE reciprocal and a second chain run
// backwards, 1/W_r = 1/W_{r+1} * (1 + e_r): a fused multiply-add per element in place of a reciprocal
// (a transcendental, about twice the cost of a plain instruction here).
template <bool MASK>
__device__ __forceinline__ bool subtile_stage1(Chain& ch, const f32x16& sacc, float c2, int n, int hh)
{
    float W = 0x1p-60f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        float e = fast_exp2(sacc[r] * c2);
        if (MASK) e = (16 * hh + r < n) ? e : 0.0f;
        ch.t[r] = W * e;
        W += ch.t[r];
        ch.be[r] = e;                                      // kept for the backward chain below
    }
    ch.norm = fast_log2(W);                                // W_16 = 2^(l - 60)
    ch.l = ch.norm + 60.0f;
    float inv = __builtin_amdgcn_rcpf(W);                  // 1 / W_16; 0 where the chain overflowed
#pragma unroll
    for (int r = 15; r >= 0; --r) {
        const float e = ch.be[r];
        ch.be[r] = ch.t[r] * inv;                          // t_r / W_{r+1}
        inv = __builtin_fmaf(inv, e, inv);                 // 1 / W_r
    }
    return W < 0x1p80f;                                    // false: this lane's chain left its range
}

// Stage 1 in the log form of Eq. 2, overflow-proof: t = 2^(x - sum of sp2 over this lane's keys
// from its own on), sigma = 2^(x - sp2(x)).
template <bool MASK>
__device__ __forceinline__ void subtile_stage1_log(Chain& ch, const f32x16& sacc, float c2, int n, int hh)
{
    float run = 0.0f;
#pragma unroll
    for (int r = 15; r >= 0; --r) {
        float x = sacc[r] * c2;
        if (MASK) x = (16 * hh + r < n) ? x : -INFINITY;
        const float sp = sp2(x);
        run += sp;
        ch.be[r] = fast_exp2(x - sp);
        ch.t[r] = fast_exp2(x - run);
    }
    ch.l = run;
    ch.norm = 0.0f;
}

// subtile_g() up to the sums of G, subtile_dz() with cb in hand.
template <bool CA_INCLUDES_SUBTILE, bool NEED_A>
__device__ __forceinline__ void subtile_g(SubtileOut& out, Chain& ch, const f32x16& pacc, float ca, int hh)
{
    float l_lo, l_hi;
    both_halves(ch.l, l_lo, l_hi);
    const float car = CA_INCLUDES_SUBTILE ? ca - (l_lo + l_hi) : ca;
    out.ca_right = car;
    // keys 16..31 (hh = 1) are nearer to the query than keys 0..15
    const float kf = fast_exp2(-(car + (hh == 0 ? l_hi : 0.0f) + ch.norm));
    // dZ = G - sigma * (prefix of G + boff), boff = cb + the partner half's total for the
    // nearer half: the part that needs boff is added once boff is known
    float grun = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float w = ch.t[r] * kf;                      // A
        if (NEED_A) out.pa[r >> 3][r & 7] = (__bf16)w;
        const float g = w * pacc[r];                       // G = dL/dlogA = A * dL/dA
        grun += g;                                         // inclusive prefix inside the lane
        ch.t[r] = g - ch.be[r] * grun;
    }
    float g_hi;
    both_halves(grun, out.g_lo, g_hi);
    out.g_tot = out.g_lo + g_hi;
}
__device__ __forceinline__ void subtile_dz(SubtileOut& out, const Chain& ch, float cb, int hh)
{
    const float boff = cb + (hh == 1 ? out.g_lo : 0.0f);
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float dz = ch.t[r] - ch.be[r] * boff;        // Eq. 4
        out.pz[r >> 3][r & 7] = (__bf16)dz;
    }
}
template <bool CA_INCLUDES_SUBTILE, bool NEED_A>
__device__ __forceinline__ void subtile_stage2(SubtileOut& out, Chain& ch, const f32x16& pacc,
                                               float ca, float cb, int hh)
{
    subtile_g<CA_INCLUDES_SUBTILE, NEED_A>(out, ch, pacc, ca, hh);
    subtile_dz(out, ch, cb, hh);
}

// ------------------------------------------------------------------ staging
// Direct global -> LDS staging of 64-row tiles of two [T][D] matrices (X then Y in
// one stage).  One instruction moves 16 B per lane to 1 KB of consecutive LDS; the
// swizzle is applied on the global side.  PERM selects the swizzle (see sb_mma.h).
template <int D> struct StageCfg {
    static constexpr int ROW = D * 2;
    static constexpr int TILE = TK * ROW;               // one 64-row tile
    static constexpr int STAGE = 2 * TILE;
    static constexpr int CPR = ROW / 16;
    static constexpr int BLK_ROWS = 1024 / ROW;
    static constexpr int NPW = TILE / 1024 / NW;        // loads per wave per tile
};

// goff[i]: byte offset inside a tile of the 16 B this lane fetches with its i-th load
template <int D, bool PERM>
__device__ __forceinline__ void stage_offsets(int (&goff)[StageCfg<D>::NPW], int wave, int lane)
{
    using C = StageCfg<D>;
#pragma unroll
    for (int i = 0; i < C::NPW; ++i) {
        const int row = (wave * C::NPW + i) * C::BLK_ROWS + lane / C::CPR;
        const int swz = PERM ? swz_perm<D>(row) : swz_nat<D>(row);
        goff[i] = (row * D + (((lane % C::CPR) ^ swz) << 3)) * 2;
    }
}

// one 64-row tile of X alone
template <int D, bool PERM>
__device__ __forceinline__ void stage_one(const uint16_t* X, int jt, int T, char* sp,
                                          const int (&goff)[StageCfg<D>::NPW], int wave, int lane)
{
    using C = StageCfg<D>;
    const uint16_t* xb = X + (long)jt * TK * D;
    char* dst = sp + wave * C::NPW * 1024;
    if ((jt + 1) * TK <= T) dma16_to_lds_run(xb, goff, dst);
    else                                                // rows past T are clamped (their results are masked)
        dma16_to_lds_run_clamped<C::ROW, C::BLK_ROWS>(xb, goff, wave * C::NPW * C::BLK_ROWS + lane / C::CPR, T - 1 - jt * TK, dst);
}

// and of X, then Y
template <int D, bool PERM>
__device__ __forceinline__ void stage_tile(const uint16_t* X, const uint16_t* Y, int jt, int T, char* sp,
                                           const int (&goff)[StageCfg<D>::NPW], int wave, int lane)
{
    using C = StageCfg<D>;
    stage_one<D, PERM>(X, jt, T, sp, goff, wave, lane);
    stage_one<D, PERM>(Y, jt, T, sp + C::TILE, goff, wave, lane);
}

// A strip's accumulators, times f, to its 32 rows from `out` on (wave-uniform), of which `rows` exist: acc[b][r] is
// row 8*(r/4) + 4*hh + r%4, column 32b + n.  Whole strips without a test per element: 64 tests with their
// addresses, reloaded from scratch each, took as long as the stores (bwd_dkv_pair_kernel, see there).
// With SHARED for other workgroups of the launch, on any XCD, to read.
template <bool SHARED> __device__ __forceinline__ void store_float(float* p, float x)
{
    if constexpr (SHARED) __hip_atomic_store(p, x, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    else *p = x;
}
template <int D, bool SHARED = false>
__device__ __forceinline__ void store_strip(float* out, int rows, const f32x16 (&acc)[D / 32], float f, int n, int hh)
{
    float* const o = reinterpret_cast<float*>(scalar_base(out));
    const int at = 4 * hh * D + n;
    if (rows >= 32) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
#pragma unroll
            for (int b = 0; b < D / 32; ++b) store_float<SHARED>(&o[(8 * (r >> 2) + (r & 3)) * D + 32 * b + at], acc[b][r] * f);
        return;
    }
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        if (8 * (r >> 2) + 4 * hh + (r & 3) < rows)
#pragma unroll
            for (int b = 0; b < D / 32; ++b) store_float<SHARED>(&o[(8 * (r >> 2) + (r & 3)) * D + 32 * b + at], acc[b][r] * f);
    }
}

// ------------------------------------------------------------------ gradient of the remainder bias
// dr[h][c] = sum over the batch and the rows j of exp(m_j) dO[j][c] (Appendix C: the
// output holds (stick left of row j) * r_h).  Two deterministic steps: per (batch entry,
// head, 128-row chunk) partial sums, then, per head, their sum in a fixed order.  They are the last workgroups of the launches of
// the two passes, the first step's behind the query-stationary blocks, the second's behind the key-stationary ones, and fill CUs
// that have no block left: as launches of their own they took 5 us of 25 (B2 H4 T124 d64), 10 us of 220 (B4 H12 T2048 d128).
// Rows that used up their stick (exp(m) = 0 in fp32) are not read (nor is a NaN in them).  Both steps are a few memory
// latencies long, all loads of a thread in flight at once.  A packed batch is one batch entry whose chunks are those of its sequences, one
// sequence after the other, found as its strips are (place_of()): as many as pieces() counts, not as max_T leaves room for in every sequence (64 of 32
// rows, H4 d64, max_T 2048, whole backward 47.7 -> 18.8 us; H24 d64, 19 up to 4096, 385 -> 359).
struct BiasGrad {
    float* part;              // [B * H][nchunk][D]
    float* dr;                // [H][D]
    int work;                 // workgroups of the pass; those from here on are the bias's
    int B, H, nchunk;         // packed batch: B = 1
};

// part of head bh's rows from m, dout on, of which `rows` (at most DR_ROWS) exist; red: (NTHR * 8 / D) * (D + 4) floats of LDS
template <int D, int NTHR>
__device__ __forceinline__ void bias_partial(float* red, const float* __restrict__ m, const uint16_t* __restrict__ dout, float* __restrict__ out,
                                             int rows, int tid)
{
    constexpr int CG = D / 8;                 // lanes per row, eight columns each
    constexpr int RG = NTHR / CG;             // rows per pass
    constexpr int NP = DR_ROWS / RG;
    static_assert(NP * RG == DR_ROWS && D <= NTHR, "whole passes");
    const int cg = tid % CG, rg = tid / CG;
    float w[NP];
    u32x4 g[NP];
#pragma unroll
    for (int i = 0; i < NP; ++i) w[i] = i * RG + rg < rows ? __expf(m[i * RG + rg]) : 0.0f;
#pragma unroll
    for (int i = 0; i < NP; ++i) {
        g[i] = u32x4{0u, 0u, 0u, 0u};
        if (w[i] != 0.0f) g[i] = *reinterpret_cast<const u32x4*>(dout + (i * RG + rg) * D + 8 * cg);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float a0 = 0.0f, a1 = 0.0f;
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            a0 += w[i] * __builtin_bit_cast(float, g[i][e] << 16);
            a1 += w[i] * __builtin_bit_cast(float, g[i][e] & 0xffff0000u);
        }
        red[rg * (D + 4) + 8 * cg + 2 * e] = a0;
        red[rg * (D + 4) + 8 * cg + 2 * e + 1] = a1;
    }
    __syncthreads();
    if (tid < D) {
        float s = 0.0f;
#pragma unroll 16
        for (int i = 0; i < RG; ++i) s += red[i * (D + 4) + tid];
        out[tid] = s;
    }
}
// chunk `at` of the launch, of all heads and batch entries (packed batch: cu, of nseq sequences)
template <int D, int NTHR>
__device__ __forceinline__ void bias_partial_at(float* red, int at, const BiasGrad& bias, const float* __restrict__ m, const uint16_t* __restrict__ dout,
                                                int T, const int* __restrict__ cu, int nseq, int Ttot, int tid)
{
    const int bh = at / bias.nchunk;
    int chunk = at - bh * bias.nchunk;
    long row0 = (long)bh * T;
    if (cu) {
        const Place p = place_of<DR_ROWS>(chunk, cu, nseq, Ttot, T, tid & 63);     // (none: T = 0, a sum of no rows)
        chunk = p.i;
        T = p.T;
        row0 = (long)bh * Ttot + p.c0;
    }
    row0 += chunk * DR_ROWS;
    bias_partial<D, NTHR>(red, m + row0, dout + row0 * D, bias.part + (long)at * D, min(T - chunk * DR_ROWS, DR_ROWS), tid);
}

// head h's partial sums; red: NTHR floats of LDS
template <int D, int NTHR>
__device__ __forceinline__ void bias_sum(float* red, const BiasGrad& bias, int h, int tid)
{
    constexpr int NG = NTHR / D;              // groups of threads share the (batch entry, chunk) pairs
    const int c = tid % D, n = bias.B * bias.nchunk;
    float s = 0.0f;
#pragma unroll 16
    for (int i = tid / D; i < n; i += NG)
        s += bias.part[((long)(i / bias.nchunk * bias.H + h) * bias.nchunk + i % bias.nchunk) * D + c];
    red[tid] = s;
    __syncthreads();
    if (tid < D) {
        float t = 0.0f;
#pragma unroll
        for (int i = 0; i < NG; ++i) t += red[i * D + tid];
        bias.dr[h * D + tid] = t;
    }
}

// ------------------------------------------------------------------ dQ kernel
// VL (both kernels): packed variable-length batch, tensors [H][Ttot][D] ([H/G][Ttot][D] for
// k, v, dk, dv) with sequence s at rows cu[s] .. cu[s+1]-1.  BH counts sequences; T_arg
// and the block counts describe the longest one (they size the array `first` and the
// carries, which are then laid out [head][strip][Ttot]).
template <int D, bool RB, Packed VL>
__global__ void __launch_bounds__(NTHREADS, 2)
bwd_dq_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
              const uint16_t* __restrict__ v, const uint16_t* __restrict__ rb,
              const float* __restrict__ m,
              const uint16_t* __restrict__ dout, float* __restrict__ dq,
              float* __restrict__ ca, float* __restrict__ cb, uint16_t* __restrict__ first,
              int T_arg, int BH, int H, int G, int nqb_arg, int nt32, const int* __restrict__ cu, int Ttot,
              int run, BiasGrad bias, int* __restrict__ arrived, int first_wg)      // arrived: of the key-stationary pass's parts, or null
{
    using C = StageCfg<D>;
    __shared__ __attribute__((aligned(1024))) char smem[2 * C::STAGE];
    __shared__ __attribute__((aligned(16))) int s_done[2][NW];   // find_start(): per parity and wave

    // what the first loads need is fetched together with the share, not behind the branches of share_of()
    asm volatile("" :: "s"(q), "s"(k), "s"(v), "s"(m), "s"(dout), "s"(T_arg), "s"(G));
    const int wg = first_wg + blockIdx.x;
    if constexpr (RB) {
        static_assert(NTHREADS * 8 / D * (D + 4) * 4 <= 2 * C::STAGE, "the partial sums fit");
        if (wg >= bias.work) {
            bias_partial_at<D, NTHREADS>(reinterpret_cast<float*>(smem), wg - bias.work, bias, m, dout, T_arg, VL != Packed::NO ? cu : nullptr, BH, Ttot, threadIdx.x);
            return;
        }
    }
    Share sh;
    int bh, T = T_arg, nqb = nqb_arg;
    long row0, kvrow0, cbase, cstride;      // first q / k row of this head; carries: base and strip stride
    int head;
    if constexpr (VL != Packed::NO) {
        const Place at = block_of<BQ, VL == Packed::BY_LENGTH>(head, wg, H, G, cu, BH, Ttot, T_arg, threadIdx.x & 63);
        if (at.T == 0) return;
        bh = at.seq * H + head;
        sh.i = at.i;
        T = at.T;
        nqb = (T + BQ - 1) / BQ;
        row0 = (long)head * Ttot + at.c0;
        kvrow0 = (long)(head / G) * Ttot + at.c0;
        cbase = (long)head * nt32 * Ttot + at.c0;
        cstride = Ttot;
    } else {
        // grouped kv heads: G consecutive query heads read the same K and V
        sh = in_scalars(share_of(wg, BH, run));
        bh = sh.bh;
        head = bh % H;
        row0 = bh * (long)T;
        kvrow0 = (long)(G == 1 ? bh : (int)((unsigned)bh / (unsigned)G)) * T;
        cbase = (long)bh * nt32 * T;
        cstride = T;
    }

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, hh = lane >> 5;
    const int gg = lane >> 4, li = lane & 15;

    const long base = row0 * D;
    const long kvbase = kvrow0 * D;
    const uint16_t* Kg = k + kvbase;
    const uint16_t* Vg = v + kvbase;

    // Per-lane LDS offsets inside a 32-row subtile.  The swizzle xors the chunk index, and the
    // chunk indices a lane reads differ in bits the swizzle leaves alone, so one offset per
    // access pattern is kept and the others follow by xor with a constant:
    //   A-operand read of chunk pair s (K rows for S^T, V rows for P^T):  aoff0 ^ (s << 5)
    //   transposing read of K, column block b, row group t (dQ = dZ K):    ktr0[t] ^ (b << 6)
    const uint32_t aoff0 = tile_off_perm<D>(perm_row(n), hh);
    uint32_t ktr0[2];
    {
        const int row_l = 16 * (gg >> 1) + (li >> 2);
        const int cl = 2 * (gg & 1) + ((li & 3) >> 1);
#pragma unroll
        for (int t = 0; t < 2; ++t) ktr0[t] = tile_off_perm<D>(row_l + 4 * t, cl) + 8 * (li & 1);
    }
    const uint32_t smem0 = lds_offset(smem);
    int goff[C::NPW];
    stage_offsets<D, true>(goff, wave, lane);

    const float scale = 1.0f / sqrtf((float)D);
    const float c2 = SB_LOG2E * scale;
    float* const cag = ca + cbase;
    float* const cbg = cb + cbase;

    bf16x8 qf[D / 16], gf[D / 16];          // B operands: this lane's query row of Q and dO
    f32x16 dqacc[D / 32];
    float a2 = 0.0f;                        // sum of sp2 from the sweep position up to the query
    float bsum = 0.0f;                      // sum of G over the keys already passed
    int q0 = 0;

    // one 32-key subtile at keys key0 .. key0+31
    // ktile: LDS address of the subtile's K rows (its V rows lie C::TILE further)
    auto subtile = [&](auto mask_c, uint32_t ktile, int key0) __attribute__((always_inline)) {
        constexpr bool MASK = decltype(mask_c)::value;
        const uint32_t ka = ktile + aoff0;
        // the operand reads of a product are issued before its first MFMA: the LDS latency
        // is then paid once per product, not once per MFMA
        auto s_mfma = [&]() __attribute__((always_inline)) {
            u32x4 kw[D / 16];
#pragma unroll
            for (int s = 0; s < D / 16; ++s) kw[s] = lds_load16(ka ^ (s << 5));
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
            for (int s = 0; s < D / 16; ++s)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kw[s]), qf[s], acc, 0, 0, 0);
            return acc;
        };
        auto p_mfma = [&]() __attribute__((always_inline)) {
            u32x4 vw[D / 16];
#pragma unroll
            for (int s = 0; s < D / 16; ++s) vw[s] = lds_load16((ka ^ (s << 5)) + C::TILE);
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
            for (int s = 0; s < D / 16; ++s)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, vw[s]), gf[s], acc, 0, 0, 0);
            return acc;
        };
        SubtileOut so;
        Chain ch;
        const bool fits = subtile_stage1<MASK>(ch, s_mfma(), c2, n, hh);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!fits) != 0, 0)) subtile_stage1_log<MASK>(ch, s_mfma(), c2, n, hh);
        const f32x16 pacc = p_mfma();
        subtile_stage2<true, false>(so, ch, pacc, a2, bsum, hh);
        // carries of this (subtile, query) for the key-stationary kernel
        if (hh == 0 && q0 + n < T) {
            const long ci = (long)(key0 >> 5) * cstride + q0 + n;
            cag[ci] = so.ca_right;
            cbg[ci] = bsum;
        }
        a2 = so.ca_right;
        bsum += so.g_tot;
        // dQ += dZ K: dZ from registers, K (rows = keys) through the transposing load
        bf16x8 kt[D / 16];
        const uint32_t k0a = ktile + ktr0[0], k1a = ktile + ktr0[1];
#pragma unroll
        for (int b = 0; b < D / 32; ++b)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const int ro = (8 * s) * C::ROW;
                kt[2 * b + s] = tr_pair_at((k0a ^ (b << 6)) + ro, (k1a ^ (b << 6)) + ro);
            }
#pragma unroll
        for (int b = 0; b < D / 32; ++b)
#pragma unroll
            for (int s = 0; s < 2; ++s)
                dqacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(so.pz[s], kt[2 * b + s], dqacc[b], 0, 0, 0);
    };

    // Where the sweep of the block at Q0 has to start.  Every wave looks for the 32-key strip beyond which
    // its own rows are exhausted, from its diagonal towards key 0, logits and softplus totals only (a third of
    // the sweep's matrix work, a quarter of its vector work), and sets `start` to it and a2 to the carry at its
    // left edge, which also spares the sweep a sum over all keys that is then subtracted again; 0 and a2 as it
    // is if there is none.  Returns the tile at which the first of the waves has to start.
    // Bound by its steps' latencies: 9 of the 29 us of a short-reaching block at d = 128.  Two strips a wave and
    // barrier, out of a ring of eight in the staging buffers, each wave its own distance from its diagonal, not
    // all of them the same tile pairs (of which the first wave sees only the masked subtile of the first); and
    // whether to look at all is known from m before the first tiles are asked for.  All heads near, us:
    // B8 H16 T4096 d128 242 -> 230, B4 H12 T2048 d128 60 -> 47, B8 H16 T2048 d64 68 -> 61, T1024 36 -> 32.6;
    // a third far 493 -> 481, 84 -> 83, 95.5 -> 93, 40 -> 37; all far within 1 %.
    // Tried only where m says that the rows have at least twice what exhausts them, so that the
    // point is expected in the nearer half, and given up after that half: at worst a sixth more.
    auto ring = [&](int s) __attribute__((always_inline)) { return ((s + 1) & 7) * 32 * C::ROW; };
    auto stage_strips = [&](const uint16_t* Kg, int T, int s) __attribute__((always_inline)) {    // s and s + 1; s is odd
        stage_one<D, true>(Kg + (long)s * 32 * D, 0, T - s * 32, smem + ring(s), goff, wave, lane);
    };
    // what the first step takes: the block's strips sb .. sb + 3 and the one in front
    auto stage_first = [&](const uint16_t* Kg, int T, int sb) __attribute__((always_inline)) {
        stage_strips(Kg, T, sb - 1);
        if ((sb + 1) * 32 < T) stage_strips(Kg, T, sb + 1);
        if ((sb + 3) * 32 < T && wave < NW / 2) stage_strips(Kg, T, sb + 3);
    };
    auto find_start = [&](const uint16_t* Kg, int T, int ntile, int sb, bool wave_live, int& start) __attribute__((always_inline)) {
        const int limit = ntile >> 1;                        // steps
        float l = 0.0f;                                      // this lane's keys only
        int found = wave_live ? 0 : 0x7fffffff;              // the strip, plus one
        auto logits = [&](int s) __attribute__((always_inline)) {
            const uint32_t ka = smem0 + ring(s) + aoff0;
            u32x4 kw[D / 16];
#pragma unroll
            for (int x = 0; x < D / 16; ++x) kw[x] = lds_load16(ka ^ (x << 5));
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
            for (int x = 0; x < D / 16; ++x)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kw[x]), qf[x], acc, 0, 0, 0);
            return acc;
        };
        auto look = [&](int s) __attribute__((always_inline)) {
            float l_lo, l_hi;
            both_halves(l, l_lo, l_hi);
            if (__builtin_amdgcn_ballot_w64(!(l_lo + l_hi >= CARRY_EXHAUSTED)) == 0) {
                a2 = l_lo + l_hi;
                start = s;
                found = s + 1;
            }
        };
        for (int i = 0;; ++i) {
            dma_wait<0>();
            barrier_lds();
            if (i > 0) {
                // what the waves found up to step i - 1; all read the same words and leave together
                const u32x4 f = lds_load16(lds_offset(reinterpret_cast<const char*>(s_done[(i + 1) & 1])));
                const int least = __builtin_amdgcn_readfirstlane((int)min(min(f[0], f[1]), min(f[2], f[3])));
                if (least > 0) return (least - 1) >> 1;
                if (i == limit) return 0;
            }
            if (i + 1 < limit) stage_strips(Kg, T, sb - 2 * i - 3);
            if (!found) {
                const int s = sb + wave - 2 * i;
                const f32x16 s0 = logits(s), s1 = logits(s - 1);
                if (i == 0) l += sp2_total<true>(s0, c2, n, hh);             // the strip's first row sees none of these
                else {
                    l += sp2_total<false>(s0, c2, n, hh);
                    look(s);
                }
                if (!found) {
                    l += sp2_total<false>(s1, c2, n, hh);
                    look(s - 1);
                }
            }
            if (lane == 0) s_done[i & 1][wave] = found;
        }
    };

    const int qb = nqb - 1 - sh.i;
    const int Q0 = qb * BQ;
    if (arrived && head % G == 0 && tid < 4 && 4 * qb + tid < nt32) arrived[(long)(bh / G) * nt32 + 4 * qb + tid] = 0;
    q0 = Q0 + wave * 32;
    const bool wave_live = q0 < T;
    const int jq = min(q0 + n, T - 1);
    const int kmax = min(T, Q0 + BQ) - 1;            // keys 0 .. kmax-1 are visible to some row
    const int ntile = (kmax + TK - 1) / TK;
    const int nclean = min(ntile, Q0 / TK);          // tiles entirely left of the block's rows
    const bool far = nclean >= 6 && ntile <= 32768;  // long enough to look for a start, and `first` can hold it
    // what the block needs first, tiles and rows alike, is fetched together: one memory latency.  (m ahead of the
    // rows, so that which tiles it is to be is known by then.)
    bool seek = false;                               // look for a start
    {
        const float mj = m[row0 + jq];
        const u32x4* qs = reinterpret_cast<const u32x4*>(q + base + (long)jq * D + 8 * hh);
        const u32x4* gs = reinterpret_cast<const u32x4*>(dout + base + (long)jq * D + 8 * hh);
        u32x4 a[D / 16], g[D / 16];
        asm volatile("" ::: "memory");
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            a[s] = qs[2 * s];
            g[s] = gs[2 * s];
        }
        asm volatile("" ::: "memory");
        a2 = -mj * SB_LOG2E;
        if (far) {
            const int likely = !wave_live || __builtin_amdgcn_ballot_w64(!(a2 >= 2.0f * CARRY_EXHAUSTED)) == 0;
            if (lane == 0) s_done[1][wave] = likely;
            barrier_lds();
            seek = waves_done(s_done[1]);
        }
        if (seek) stage_first(Kg, T, Q0 / 32);
        else if (ntile > 0) stage_tile<D, true>(Kg, Vg, 0, T, smem, goff, wave, lane);
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            if (q0 + n >= T) g[s] = u32x4{0u, 0u, 0u, 0u};   // rows past T contribute nothing
            qf[s] = __builtin_bit_cast(bf16x8, a[s]);
            gf[s] = __builtin_bit_cast(bf16x8, g[s]);
        }
    }
    bsum = 0.0f;
    if constexpr (RB) {
        // remainder bias (Appendix C): the unused stick exp(m) acts like one more weight
        // in front of key 0, with "value" r_head: the cumulative sum of G starts at
        // exp(m_j) (dO_j . r_head)
        const u32x4* rs = reinterpret_cast<const u32x4*>(rb + head * D + 8 * hh);
        float dot = 0.0f;
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            const bf16x8 rr = __builtin_bit_cast(bf16x8, rs[2 * s]);
#pragma unroll
            for (int e = 0; e < 8; ++e) dot += (float)gf[s][e] * (float)rr[e];
        }
        float d_lo, d_hi;
        both_halves(dot, d_lo, d_hi);
        bsum = fast_exp2(-a2) * (d_lo + d_hi);
    }
    // wait for these loads once: the staging loads of the sweep
    // are counted in the same counter behind the compiler's back
#pragma unroll
    for (int s = 0; s < D / 16; ++s) { asm volatile("" :: "v"(qf[s])); asm volatile("" :: "v"(gf[s])); }
    asm volatile("" :: "v"(a2));
    asm volatile("" :: "v"(bsum));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int b = 0; b < D / 32; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) dqacc[b][r] = 0.0f;

    // ---- sweep over 64-key tiles, left to right; iteration it handles tile it in buffer it & 1
    int t0 = 0, start = 0;
    if (seek) {
        t0 = find_start(Kg, T, ntile, Q0 / 32, wave_live, start);
        stage_tile<D, true>(Kg, Vg, t0, T, smem + (t0 & 1) * C::STAGE, goff, wave, lane);
    }
    if (lane == 0) first[((long)bh * nqb_arg + qb) * 4 + wave] = (uint16_t)(wave_live ? start : 2 * t0);
    auto begin_iter = [&](int it) __attribute__((always_inline)) {
        dma_wait<0>();                               // this wave's share of tile `it` has landed
        barrier_nofence();                           // ... everyone's has, and tile it-1 is no longer read
        if (it + 1 < ntile)
            stage_tile<D, true>(Kg, Vg, it + 1, T, smem + ((it + 1) & 1) * C::STAGE, goff, wave, lane);
        return smem0 + (it & 1) * C::STAGE;
    };
    int it = t0;
    for (; it < nclean && 2 * it < start; ++it) {    // tiles in front of this wave's start
        const uint32_t sp = begin_iter(it);
        if (2 * it + 1 >= start) subtile(bc<false>{}, sp + 32 * C::ROW, it * TK + 32);
    }
    for (; it < nclean; ++it) {                      // fully visible tiles
        const uint32_t sp = begin_iter(it);
        subtile(bc<false>{}, sp, it * TK);
        subtile(bc<false>{}, sp + 32 * C::ROW, it * TK + 32);
    }
    for (; it < ntile; ++it) {                       // tiles that touch the diagonal band
        const uint32_t sp = begin_iter(it);
        if (wave_live) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int key0 = it * TK + 32 * u;
                if (key0 == q0) subtile(bc<true>{}, sp + u * 32 * C::ROW, key0);
                else if (key0 < q0 && 2 * it + u >= start) subtile(bc<false>{}, sp + u * 32 * C::ROW, key0);
            }
        }
    }

    if (wave_live) store_strip<D>(dq + base + (long)q0 * D, T - q0, dqacc, scale, n, hh);
}

// Where a kv head's rows and its query heads' rows and carries live (key-stationary kernels).
// A share's heads are kv heads (B * H / G of them); the G query heads of one are qh0 .. qh0+G-1.
struct KvHead {
    int T, nkb;                             // rows and key blocks (of `keys` keys) of this head's sequence
    long base;                              // first element of the kv head's K / V / dK / dV rows
    long qrow0, qrow_step;                  // first Q / dO row of query head qh0, step to the next head
    long cbase, cbase_step, cstride;        // carries: start for head qh0, step per head, strip stride
    long qhead0;                            // index of head qh0 in `first`
};

// the sequence found at a place of a packed batch
template <int D>
__device__ __forceinline__ void packed_kv_head(KvHead& kh, const Place& at, int hkv, int keys, int H, int G, int nt32, int Ttot)
{
    kh.T = at.T;
    kh.nkb = (kh.T + keys - 1) / keys;
    kh.base = ((long)hkv * Ttot + at.c0) * D;
    kh.qrow0 = (long)hkv * G * Ttot + at.c0;
    kh.qrow_step = Ttot;
    kh.qhead0 = (long)at.seq * H + hkv * G;
    kh.cbase = (long)hkv * G * nt32 * Ttot + at.c0;
    kh.cbase_step = (long)nt32 * Ttot;
    kh.cstride = Ttot;
}

// Head `bh` of a batch
__device__ __forceinline__ void kv_head(KvHead& kh, int bh, int D, int T, int nkb, int G, int nt32)
{
    const long qh0 = (long)bh * G;
    kh.T = T;
    kh.nkb = nkb;
    kh.base = (long)bh * T * D;
    kh.qrow0 = qh0 * (long)T;
    kh.qhead0 = qh0;
    kh.qrow_step = T;
    kh.cbase = qh0 * (long)nt32 * T;
    kh.cbase_step = (long)nt32 * T;
    kh.cstride = T;
}

// Workgroup wg's kv head and block of KEYS keys (.i < 0: none is left for it), and of a packed batch the sequence.  What follows
// from them, kv_head_of(), comes after the lane's own numbers: all at once, the paired kernel spills four times as much.
template <Packed VL, bool PAIRS, int KEYS>
__device__ __forceinline__ Share kv_block(Place& at, unsigned wg, int BH, int run, int T_arg, int nkb_arg, int Hkv, const int* __restrict__ cu, int Ttot)
{
    if constexpr (VL != Packed::NO) {
        int hkv;
        at = block_of<KEYS, VL == Packed::BY_LENGTH>(hkv, wg, Hkv, 1, cu, BH, Ttot, T_arg, threadIdx.x & 63);
        return {hkv, at.T == 0 ? -1 : at.i};
    } else {
        const Share sh = in_scalars(PAIRS ? share_in_pairs(wg, nkb_arg) : share_of(wg, BH, run));
        return {sh.bh, PAIRS && sh.bh >= BH ? -1 : sh.i};
    }
}
template <int D, Packed VL, int KEYS>
__device__ __forceinline__ void kv_head_of(KvHead& kh, const Share& sh, const Place& at, int T_arg, int nkb_arg, int H, int G, int nt32, int Ttot)
{
    if constexpr (VL != Packed::NO) packed_kv_head<D>(kh, at, sh.bh, KEYS, H, G, nt32, Ttot);
    else kv_head(kh, sh.bh, D, T_arg, nkb_arg, G, nt32);
}

// Key-stationary pass of grouped heads in parts: a block of keys is n workgroups', each with G / n of the group's query heads, if the
// block's weights reach far; else the first one takes all of them and the others have nothing to do.  Every part leaves its sums in `sums`: dV's
// of all heads, then dK's, laid out as dv and dk are with n kv heads in place of one; behind them a count for every kv head and strip of 32 keys of the
// parts that have come, cleared by the query-stationary pass.  The last of a block's adds them up, in their order whichever it is.
// Without parts a far group's heads are one chain, and what the launch waits for: figures beside key_plan().
// The sums pass from XCD to XCD: stored past the caches, a wait for them, one count a workgroup, loaded past the caches.  (With fences in their place, which
// write a whole L2 back for every workgroup, B4 H12 Hkv4 T2048 d128, a third of the heads far, 215 -> 304 us instead of 188.)
struct Parts {
    float* sums;
    int n, beyond, blocks, heads;           // parts, see in_parts(), workgroups and query heads of a part
};
// The sums of kv head `kv` in part 0: where element x of dk and dv is, and the counts.  rows: of a kv head (of a packed batch all)
template <int D> struct PartSums {
    float *dv, *dk;
    int* arrived;
    long step;                              // from part to part
    __device__ __forceinline__ PartSums(const Parts& parts, int kv, int heads, long rows)
    {
        const long all = heads * rows * D * parts.n;
        step = rows * D;
        dv = parts.sums + kv * (parts.n - 1) * step;
        dk = dv + all;
        arrived = reinterpret_cast<int*>(parts.sums + 2 * all);
    }
};
// The part that workgroup `wg` takes of the block of the workgroup of that number in one part.  The first part's come last, behind those that
// have nothing to do: far blocks' parts start at once, and near blocks fill up what they leave.
__device__ __forceinline__ int take_part(int& wg, const Parts& parts)
{
    int at = 0;
    for (; at < parts.n - 1 && wg >= parts.blocks; ++at) wg -= parts.blocks;
    return parts.n - 1 - at;
}
// Of a block whose first 32-key strip is `lo`: do the queries `beyond` strips further on still attend to it, in any head of the group?  In two steps: the
// first part asks together with what it needs first (and waits for it here where the group has more heads than the wave lanes).
__device__ __forceinline__ int start_beyond(const Parts& parts, const uint16_t* __restrict__ first, long qhead0, int G, int nqb, int lo, int T, int lane)
{
    const int at = lo + parts.beyond;
    if (32 * at >= T) return 0x7fffffff;
    int start = lane < G ? first[(qhead0 + lane) * nqb * 4 + at] : 0x7fffffff;
    if (__builtin_expect(G > 64, 0))
        for (int h = lane + 64; h < G; h += 64) start = min(start, (int)first[(qhead0 + h) * nqb * 4 + at]);
    return start;
}
// (What only parts do stands out of the way of the workgroups that have their block to themselves, the quotient G / n comes from the host: in line with the
// rest it cost those of strips 0.7 to 1.0 us, a launch of them 12.2 -> 12.9 us in B1 H4 Hkv2 T469 d128, 11.1 -> 12.1 in B1 H4 Hkv1 T1846 d64; now 12.5 and 11.9.)
__device__ __forceinline__ bool in_parts(int start, int lo) { return __builtin_amdgcn_ballot_w64(start <= lo) != 0; }
typedef __attribute__((ext_vector_type(2))) unsigned long long u64x2;
__device__ __forceinline__ f32x4 load_shared4(const float* p)
{
    const auto* q = reinterpret_cast<const unsigned long long*>(p);
    return __builtin_bit_cast(f32x4, u64x2{__hip_atomic_load(q, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT),
                                           __hip_atomic_load(q + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)});
}
__device__ __forceinline__ void store_shared4(float* p, f32x4 x)
{
    const u64x2 v = __builtin_bit_cast(u64x2, x);
    auto* q = reinterpret_cast<unsigned long long*>(p);
    __hip_atomic_store(q, v[0], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(q + 1, v[1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The workgroup's sums of `rows` rows from element `at` of dk and dv on have been stored; count: the block's in `arrived`
template <int D, int NTHR>
__device__ __forceinline__ void add_parts(const PartSums<D>& sums, int n, char* smem, long at, long count, int rows, float* __restrict__ dk,
                                          float* __restrict__ dv, float scale, int tid)
{
    int* const last = reinterpret_cast<int*>(smem);
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (tid == 0) *last = __hip_atomic_fetch_add(&sums.arrived[count], 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == n - 1;
    __syncthreads();
    if (!*last) return;
#pragma unroll 1
    for (int mat = 0; mat < 2; ++mat) {
        const float* const s = (mat == 0 ? sums.dv : sums.dk) + at;
        float* const out = (mat == 0 ? dv : dk) + at;
        const float f = mat == 0 ? 1.0f : scale;
        for (int i = tid; i < rows * (D / 4); i += NTHR) {
            f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll 4
            for (int p = 0; p < n; ++p) x += load_shared4(s + p * sums.step + 4 * i);
            *reinterpret_cast<f32x4*>(out + 4 * i) = x * f;
        }
    }
}

// Which query tiles reach the 32-key strips lo .. hi, a block's, from the start strips that the
// query-stationary pass left: f[jt] holds those of tile jt's two strips of queries.  None from tile `end` on;
// in all tiles before `sure` both strips reach every one of the keys.  In between strip u of a tile
// reaches key strip ks iff its start is not beyond it (reaching()).
struct Reach {
    int sure, end;
};
// The words of the first 64 blocks come from the caller (start_words()): bwd_dkv_kernel asks for them
// together with what else a block needs first, one memory latency less (1 to 3 % where heads are near); the
// paired kernel gains nothing that way.
struct StartWords {
    uint32_t f0, f1;
};
__device__ __forceinline__ StartWords start_words(const uint32_t* __restrict__ f, int b, int nqb, int lane)
{
    if (b + lane >= nqb) return {~0u, ~0u};
    return {f[2 * (b + lane)], f[2 * (b + lane) + 1]};
}
__device__ __forceinline__ Reach reach_of(const uint32_t* __restrict__ f, StartWords w, int lo, int hi, int nqb, int lane)
{
    static_assert(BQ == 2 * TK, "two tiles per query block");
    int last = lo >> 1, cut = nqb;
    for (int b = lo >> 2; b < nqb; b += 64) {
        const bool in = b + lane < nqb;
        if (b != lo >> 2) w = start_words(f, b, nqb, lane);
        const uint32_t f0 = w.f0, f1 = w.f1;
        const int lo0 = f0 & 0xffff, hi0 = f0 >> 16, lo1 = f1 & 0xffff, hi1 = f1 >> 16;
        const unsigned long long some0 = __builtin_amdgcn_ballot_w64(in && min(lo0, hi0) <= hi);
        const unsigned long long some1 = __builtin_amdgcn_ballot_w64(in && min(lo1, hi1) <= hi);
        const unsigned long long not_all = __builtin_amdgcn_ballot_w64(max(max(lo0, hi0), max(lo1, hi1)) > lo);
        if (some0) last = max(last, 2 * (b + 63 - __builtin_clzll(some0)));
        if (some1) last = max(last, 2 * (b + 63 - __builtin_clzll(some1)) + 1);
        if (not_all && cut == nqb) cut = min(nqb, b + __builtin_ctzll(not_all));
    }
    return {2 * cut, last + 1};
}
// The word of tile jt, asked for one tile ahead and looked at a tile later by reaching(), whose bit u says
// that strip u of the tile reaches key strip ks.
__device__ __forceinline__ uint32_t start_word(const uint32_t* __restrict__ f, int jt, int sure)
{
    return jt < sure ? 0u : f[jt];
}
__device__ __forceinline__ int reaching(uint32_t w, int ks)
{
    return ((int)(w & 0xffff) <= ks ? 1 : 0) | ((int)(w >> 16) <= ks ? 2 : 0);
}

// ------------------------------------------------------------------ dK / dV kernel
// SP groups of four waves take the block's query tiles in turn (tile t: group t % SP), each into
// accumulators of its own, added up at the end in LDS.  Which grids take two: take_in_turn().
template <int D, int SP> struct DkvCfg {
    static constexpr int T_OFF = SP * 2 * StageCfg<D>::STAGE;   // after the double buffers
    static constexpr int T_WAVE = 2 * SCR_MAT;             // A and dZ scratch of one wave
    static constexpr int LDS_BYTES = T_OFF + SP * NW * T_WAVE;
    static_assert(SP == 1 || NW * 2 * 32 * D * 4 <= LDS_BYTES, "the second group's accumulators fit");
};

template <int D, bool GQA, Packed VL, int SP, bool DR, bool PARTS>
__global__ void __launch_bounds__(SP * NTHREADS, D == 32 && SP == 1 ? 3 : 2)
bwd_dkv_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
               const uint16_t* __restrict__ v, const uint16_t* __restrict__ dout,
               const float* __restrict__ ca, const float* __restrict__ cb,
               float* __restrict__ dk, float* __restrict__ dv, const uint32_t* __restrict__ first,
               int T_arg, int BH, int H, int G_arg, int nkb_arg, int nt32, const int* __restrict__ cu, int Ttot,
               int run, BiasGrad bias, Parts parts, int first_wg)
{
    using C = StageCfg<D>;
    using CK = DkvCfg<D, SP>;
    const int G = GQA ? G_arg : 1;                      // query heads per kv head
    static_assert(GQA || !PARTS, "a part has some of a group's query heads");
    __shared__ __attribute__((aligned(1024))) char smem[CK::LDS_BYTES];

    asm volatile("" :: "s"(q), "s"(k), "s"(v), "s"(dout), "s"(ca), "s"(cb), "s"(first), "s"(T_arg));   // as in bwd_dq_kernel
    int wg = first_wg + blockIdx.x;
    if constexpr (DR) {
        if (wg >= bias.work) {
            bias_sum<D, SP * NTHREADS>(reinterpret_cast<float*>(smem), bias, wg - bias.work, threadIdx.x);
            return;
        }
    }
    Place at;
    int part = 0;
    if constexpr (PARTS) part = take_part(wg, parts);
    const Share sh = kv_block<VL, false, BKW>(at, wg, BH, run, T_arg, nkb_arg, H / G, cu, Ttot);
    if (sh.i < 0) return;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6) & (NW - 1);
    const int grp = SP == 1 ? 0 : __builtin_amdgcn_readfirstlane(tid / NTHREADS);
    char* const tiles = smem + grp * 2 * C::STAGE;      // the group's double buffer
    const int n = lane & 31, hh = lane >> 5;
    const int gg = lane >> 4, li = lane & 15;

    KvHead kh;
    kv_head_of<D, VL, BKW>(kh, sh, at, T_arg, nkb_arg, H, G, nt32, Ttot);
    const int T = kh.T, nkb = kh.nkb;
    int g0 = 0, g1 = G;                                 // the workgroup's query heads
    bool alone = true;
    int beyond = 0;
    if constexpr (PARTS) {
        beyond = start_beyond(parts, reinterpret_cast<const uint16_t*>(first), kh.qhead0, G, nkb_arg, sh.i * (BKW / 32), T, lane);
        if (__builtin_expect(part > 0, 0)) {
            if (!in_parts(beyond, sh.i * (BKW / 32))) return;
            alone = false;
            g0 = part * parts.heads;
            g1 = g0 + parts.heads;
        }
    }
    const long base = kh.base, qrow0 = kh.qrow0, qrow_step = kh.qrow_step;
    const long cbase = kh.cbase, cbase_step = kh.cbase_step, cstride = kh.cstride;
    const uint16_t* Qg = nullptr;
    const uint16_t* Gg = nullptr;

    // per-lane LDS offsets inside a 32-row Q / dO subtile (natural row order)
    int boff[D / 16];                       // B-operand reads: row = query n
#pragma unroll
    for (int s = 0; s < D / 16; ++s) boff[s] = tile_off_nat<D>(n, 2 * s + hh);
    int qtr[D / 32][2];                     // transposing reads (K-dim = queries)
    {
        const int row_l = 8 * (gg >> 1) + (li >> 2);
        const int cl = 2 * (gg & 1) + ((li & 3) >> 1);
#pragma unroll
        for (int b = 0; b < D / 32; ++b)
#pragma unroll
            for (int t = 0; t < 2; ++t)
                qtr[b][t] = tile_off_nat<D>(row_l + 4 * t, 4 * b + cl) + 8 * (li & 1);
    }
    int goff[C::NPW];
    stage_offsets<D, false>(goff, wave, lane);
    char* const scr = smem + CK::T_OFF + (grp * NW + wave) * CK::T_WAVE;               // [A, dZ][32 rows of 64 B]
    const int sw_off = scr_off(n, 2 * hh);                                // scratch write: row = query n; second chunk: ^ 16
    int st_off[2];                                                        // transposing reads, rows 8h + li/4 (+ 4t)
#pragma unroll
    for (int t = 0; t < 2; ++t)
        st_off[t] = scr_off(8 * (gg >> 1) + (li >> 2) + 4 * t, 2 * (gg & 1) + ((li & 3) >> 1)) + 8 * (li & 1);

    const float scale = 1.0f / sqrtf((float)D);
    const float c2 = SB_LOG2E * scale;

    bf16x8 kf[D / 16], vf[D / 16];          // A operands: this wave's K and V rows (MFMA row n <- key perm_row(n))
    f32x16 dkacc[D / 32], dvacc[D / 32];
    const float* cag = nullptr;
    const float* cbg = nullptr;
    // ca, cb of query tile jt for this wave's keys (of a strip that does not reach them: unwritten
    // memory, and not used).  Rows past T: an infinite carry gives A = 0 and G = 0, and with cb = 0 also
    // dZ = 0.  (A dead wave's rows lie outside the arrays.)
    auto load_carries = [&](float (&cn)[2][2], int jt, bool live) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int j = jt * TK + 32 * u + n;
            cn[u][0] = (j < T && live) ? cag[j] : INFINITY;
            cn[u][1] = (j < T && live) ? cbg[j] : 0.0f;
        }
    };

    // one 32-query subtile at query rows j0 .. j0+31
    // the steps of one 32-query subtile (Q rows at qtile, dO rows C::TILE further).  All
    // operand reads of a step are issued before its first MFMA, so that the LDS latency
    // is paid once per step and not once per MFMA.
    // S^T = K Q^T and P^T = V dO^T (two independent accumulation chains, interleaved)
    auto sp_mfma = [&](const char* qtile, f32x16& sacc, f32x16& pacc) __attribute__((always_inline)) {
        const char* gtile = qtile + C::TILE;
        u32x4 qw[D / 16], gw[D / 16];
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            qw[s] = *reinterpret_cast<const u32x4*>(qtile + boff[s]);
            gw[s] = *reinterpret_cast<const u32x4*>(gtile + boff[s]);
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) { sacc[r] = 0.0f; pacc[r] = 0.0f; }
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], __builtin_bit_cast(bf16x8, qw[s]), sacc, 0, 0, 0);
            pacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[s], __builtin_bit_cast(bf16x8, gw[s]), pacc, 0, 0, 0);
        }
    };
    // A and dZ into [key][query] operand layout through the wave's scratch
    auto transpose = [&](const SubtileOut& so, bf16x8 (&at)[2], bf16x8 (&zt)[2]) __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        *reinterpret_cast<bf16x8*>(scr + sw_off) = so.pa[0];
        *reinterpret_cast<bf16x8*>(scr + (sw_off ^ 16)) = so.pa[1];
        *reinterpret_cast<bf16x8*>(scr + SCR_MAT + sw_off) = so.pz[0];
        *reinterpret_cast<bf16x8*>(scr + SCR_MAT + (sw_off ^ 16)) = so.pz[1];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            const char* pa = scr + (16 * s2) * 64;         // rows 16 s2 + ..: same swizzle as rows 0..15
            const char* pz = pa + SCR_MAT;
            at[s2] = tr_pair(pa + st_off[0], pa + st_off[1]);
            zt[s2] = tr_pair(pz + st_off[0], pz + st_off[1]);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    };
    // dV += A^T dO, dK += dZ^T Q: K-dim = the 32 queries, B operands through the transposing load
    auto mm2_fetch = [&](const char* qtile, bf16x8 (&gop)[D / 16], bf16x8 (&qop)[D / 16]) __attribute__((always_inline)) {
        const char* gtile = qtile + C::TILE;
#pragma unroll
        for (int b = 0; b < D / 32; ++b)
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                const int ro = (16 * s2) * C::ROW;
                gop[2 * b + s2] = tr_pair(gtile + ro + qtr[b][0], gtile + ro + qtr[b][1]);
                qop[2 * b + s2] = tr_pair(qtile + ro + qtr[b][0], qtile + ro + qtr[b][1]);
            }
    };
    auto mm2 = [&](const bf16x8 (&gop)[D / 16], const bf16x8 (&qop)[D / 16], const bf16x8 (&at)[2], const bf16x8 (&zt)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < D / 32; ++b)
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                dvacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at[s2], gop[2 * b + s2], dvacc[b], 0, 0, 0);
                dkacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(zt[s2], qop[2 * b + s2], dkacc[b], 0, 0, 0);
            }
    };
    // one 32-query subtile, start to end
    auto subtile = [&](auto mask_c, const char* qtile, float car, float cbl) __attribute__((always_inline)) {
        constexpr bool MASK = decltype(mask_c)::value;
        if (MASK && n == 0) {
            // The first query of the diagonal subtile sees none of its keys, and where that
            // query is the last row of the sequence the query-stationary pass never visits
            // this subtile: its carries may be unwritten memory.  They multiply zeros, so
            // any finite value will do.
            car = 0.0f;
            cbl = 0.0f;
        }
        SubtileOut so;
        f32x16 sacc, pacc;
        sp_mfma(qtile, sacc, pacc);
        bf16x8 gop[D / 16], qop[D / 16];
        mm2_fetch(qtile, gop, qop);                          // lands during the element-wise work
        Chain ch;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!subtile_stage1<MASK>(ch, sacc, c2, n, hh)) != 0, 0)) {
            f32x16 again;
#pragma unroll
            for (int r = 0; r < 16; ++r) again[r] = 0.0f;
#pragma unroll
            for (int s = 0; s < D / 16; ++s)
                again = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], *reinterpret_cast<const bf16x8*>(qtile + boff[s]), again, 0, 0, 0);
            subtile_stage1_log<MASK>(ch, again, c2, n, hh);
        }
        subtile_stage2<false, true>(so, ch, pacc, car, cbl, hh);
        bf16x8 at[2], zt[2];
        transpose(so, at, zt);
        mm2(gop, qop, at, zt);
    };

    const int kb = sh.i;                                 // small kb = most later queries = first
    const int K0 = kb * BKW;
    const int k0 = K0 + wave * 32;                       // this wave's 32 keys
    const int kt32 = k0 >> 5;
    const bool wave_live = k0 < T;
    const int jt0 = K0 / TK;
    float cn[2][2];                                      // [subtile][ca, cb] of the next tile
    const uint32_t* fg = nullptr;
    StartWords sw;
    // the group's first tile of a head and its carries
    auto first_tile = [&](int g) __attribute__((always_inline)) {
        Qg = q + (qrow0 + g * qrow_step) * D;
        Gg = dout + (qrow0 + g * qrow_step) * D;
        cag = ca + cbase + g * cbase_step + kt32 * cstride;
        cbg = cb + cbase + g * cbase_step + kt32 * cstride;
        fg = first + (kh.qhead0 + g) * 2 * nkb_arg;
        sw = start_words(fg, kb, nkb, lane);
        load_carries(cn, jt0 + grp, wave_live);
        if (SP == 1 || (jt0 + grp) * TK < T) stage_tile<D, false>(Qg, Gg, jt0 + grp, T, tiles, goff, wave, lane);
    };
    first_tile(g0);                                      // fetched together with the stationary rows
    {
        const long kr = min(k0 + perm_row(n), T - 1);
        const u32x4* ks = reinterpret_cast<const u32x4*>(k + base + kr * D + 8 * hh);
        const u32x4* vs = reinterpret_cast<const u32x4*>(v + base + kr * D + 8 * hh);
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            kf[s] = __builtin_bit_cast(bf16x8, ks[2 * s]);
            vf[s] = __builtin_bit_cast(bf16x8, vs[2 * s]);
        }
    }
#pragma unroll
    for (int s = 0; s < D / 16; ++s) { asm volatile("" :: "v"(kf[s])); asm volatile("" :: "v"(vf[s])); }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    if (PARTS && part == 0 && __builtin_expect(in_parts(beyond, sh.i * (BKW / 32)), 0)) {
        alone = false;
        g1 = parts.heads;
    }
#pragma unroll
    for (int b = 0; b < D / 32; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) { dkacc[b][r] = 0.0f; dvacc[b][r] = 0.0f; }
    // the query heads of the group one after the other, into the same accumulators
    for (int g = g0; g < g1; ++g) {
    if (g > g0) {
        barrier_nofence();                               // everyone is done with the stages of the head before
        first_tile(g);
    }

    // ---- sweep over 64-row query tiles, from the block's diagonal to the end;
    // iteration it handles tile jt0 + it in buffer it & 1.  The carries of a tile are
    // fetched one iteration ahead, and BEFORE the staging loads of that iteration are
    // issued: vector memory operations complete in order, so a wait for a carry
    // issued after the staging loads would wait for those as well.
    const Reach reach = reach_of(fg, sw, 4 * kb, 4 * kb + 3, nkb, lane);
    const int ntile = min((T + TK - 1) / TK, reach.end) - jt0;
    const int niter = (ntile + SP - 1) / SP;
    const int ndiag = min(niter, BKW / TK / SP);         // iterations on tiles that touch the diagonal band
    const int nsure = min(niter, (reach.sure - jt0) / SP);
    float cc[2][2];
    int there = 0;
    uint32_t word_next = grp < ntile ? start_word(fg, jt0 + grp, reach.sure) : ~0u;
    auto begin_iter = [&](int it) __attribute__((always_inline)) {
        dma_wait<0>();
        barrier_nofence();
#pragma unroll
        for (int u = 0; u < 2; ++u) { cc[u][0] = cn[u][0]; cc[u][1] = cn[u][1]; }
        there = reaching(word_next, kt32);
        const int jt = jt0 + (it + 1) * SP + grp;
        if (jt < jt0 + ntile) {
            load_carries(cn, jt, wave_live);
            word_next = start_word(fg, jt, reach.sure);
            stage_tile<D, false>(Qg, Gg, jt, T, tiles + ((it + 1) & 1) * C::STAGE, goff, wave, lane);
        }
        return (const char*)(tiles + (it & 1) * C::STAGE);
    };
    int it = 0;
    for (; it < ndiag; ++it) {
        const char* sp = begin_iter(it);
        if (wave_live) {
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int j0 = (jt0 + it * SP + grp) * TK + 32 * u;
                if (j0 == k0) subtile(bc<true>{}, sp + u * 32 * C::ROW, cc[u][0], cc[u][1]);
                else if (j0 > k0 && j0 < T && (there >> u & 1)) subtile(bc<false>{}, sp + u * 32 * C::ROW, cc[u][0], cc[u][1]);
            }
        }
    }
    for (; it < nsure; ++it) {                           // tiles that reach all keys
        const char* sp = begin_iter(it);
        if (wave_live && (SP == 1 || it * SP + grp < ntile)) {
            const int j0 = (jt0 + it * SP + grp) * TK;
            subtile(bc<false>{}, sp, cc[0][0], cc[0][1]);
            if (j0 + 32 < T) subtile(bc<false>{}, sp + 32 * C::ROW, cc[1][0], cc[1][1]);
        }
    }
    for (; it < niter; ++it) {
        const char* sp = begin_iter(it);
#pragma unroll 1
        for (int u = 0; u < 2; ++u) {
            const int j0 = (jt0 + it * SP + grp) * TK + 32 * u;
            if (wave_live && (SP == 1 || it * SP + grp < ntile) && j0 < T && (there >> u & 1))
                subtile(bc<false>{}, sp + u * 32 * C::ROW, u ? cc[1][0] : cc[0][0], u ? cc[1][1] : cc[0][1]);
        }
    }
    }

    if constexpr (SP == 2) {
        barrier_lds();                                   // everyone is done with tiles and scratch
        f32x4* const red = reinterpret_cast<f32x4*>(smem) + wave * (D / 32 * 2 * 4) * 64 + lane;
#pragma unroll
        for (int i = 0; i < D / 32 * 2 * 4; ++i) {
            f32x16& acc = (i >> 2) & 1 ? dvacc[i >> 3] : dkacc[i >> 3];
            const int r = 4 * (i & 3);
            if (grp == 1) red[i * 64] = f32x4{acc[r], acc[r + 1], acc[r + 2], acc[r + 3]};
        }
        barrier_lds();
        if (grp == 1) return;
#pragma unroll
        for (int i = 0; i < D / 32 * 2 * 4; ++i) {
            f32x16& acc = (i >> 2) & 1 ? dvacc[i >> 3] : dkacc[i >> 3];
            const f32x4 o = red[i * 64];
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[4 * (i & 3) + e] += o[e];
        }
    }

    if (PARTS && !alone) {
        const PartSums<D> sums(parts, sh.bh, VL != Packed::NO ? H / G : BH, VL != Packed::NO ? Ttot : T_arg);
        if (wave_live) {
            store_strip<D, true>(sums.dk + part * sums.step + base + (long)k0 * D, T - k0, dkacc, 1.0f, n, hh);
            store_strip<D, true>(sums.dv + part * sums.step + base + (long)k0 * D, T - k0, dvacc, 1.0f, n, hh);
        }
        add_parts<D, NTHREADS>(sums, parts.n, smem, base + (long)K0 * D, kh.qhead0 / G * nt32 + (K0 >> 5), min(T - K0, BKW), dk, dv, scale, tid);
        return;
    }
    if (wave_live) {
        store_strip<D>(dk + base + (long)k0 * D, T - k0, dkacc, scale, n, hh);
        store_strip<D>(dv + base + (long)k0 * D, T - k0, dvacc, 1.0f, n, hh);
    }
}

// ------------------------------------------------------------------ dK / dV kernel, paired waves
// The same computation with eight waves per workgroup, two per 32-key strip, for d = 128.
// There one wave that holds both accumulators (128 registers) and both stationary operands
// (64) fills a SIMD's register file alone, and a lone wave cannot hide its own latencies.
// Here the two waves of a strip split the work so that each needs one accumulator only:
//   - "front": each takes one 32-query subtile of every 64-row tile through S^T, P^T and the
//     element-wise path and writes A and dZ (bf16) row-wise into the strip's LDS scratch;
//   - "back": role 0 accumulates dV += A^T dO and role 1 accumulates dK += dZ^T Q over both
//     subtiles, reading the transposed operands from the scratch.
// No arithmetic is duplicated.  The back of a tile is taken one barrier interval after its
// front, together with the front of the next tile: one workgroup barrier per tile, and in the
// steady state a wave's interval is one block of code in which the matrix instructions of the
// back are issued between the vector instructions of the front's element-wise path (step()).
// Price: the Q/dO tile of the interval before must stay in LDS (three tile buffers) and the
// A/dZ scratch is double buffered; with compact scratch rows (64 B, xor-swizzled) that is
// exactly the 160 KB of a CU at d = 128.  Two waves per SIMD.
// The steady-state intervals run in a loop of their own in which LDS addresses rotate through
// registers and global pointers advance by constants: with one barrier per interval all eight
// waves do their loop bookkeeping at the same time, and a hundred dependent scalar instructions
// there cost about 500 clocks per interval.
// Measured against the predecessor of this kernel (front and back as two phases with a
// barrier each, padded scratch rows): 1.35 -> 1.29 ms at B8 H16 T4096, 1.20 with the
// steady-state loop.  Also measured:
// the two roles taking front and back in opposite order within an interval (so that one
// wave of a SIMD is in its vector phase while the other is in its matrix phase) is slower,
// 1.47 ms: the compiler then copies the accumulator (64 registers) on every switch.
// KS: strips per block, 4 or, in small grids, 2 (small_kv_grid()).
template <int D, int KS> struct Dkv3Cfg {
    static constexpr int NW2 = 2 * KS;
    static constexpr int KEYS = 32 * KS;
    static constexpr int NBUF = 3;
    static constexpr int T_OFF = NBUF * StageCfg<D>::STAGE;  // after the tile buffers
    static constexpr int M_BYTES = 32 * 64;                  // one 32x32 bf16 matrix
    static constexpr int W_BYTES = 2 * M_BYTES;              // A and dZ of one wave's subtile
    static constexpr int SCR_BUF = NW2 * W_BYTES;            // the waves' subtiles of one tile
    static constexpr int LDS_BYTES = T_OFF + 2 * SCR_BUF;
    static constexpr int LOADS = StageCfg<D>::TILE / 1024;
    static constexpr int NPW = (LOADS + NW2 - 1) / NW2;
};

template <int D, int KS, bool GQA, Packed VL, bool PAIRS, bool DR, bool PARTS>
__global__ void __launch_bounds__(128 * KS, 1)
bwd_dkv_pair_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                    const uint16_t* __restrict__ v, const uint16_t* __restrict__ dout,
                    const float* __restrict__ ca, const float* __restrict__ cb,
                    float* __restrict__ dk, float* __restrict__ dv, const uint32_t* __restrict__ first,
                    int T_arg, int BH, int H, int G_arg, int nkb_arg, int nqb_arg, int nt32,
                    const int* __restrict__ cu, int Ttot, BiasGrad bias, Parts parts, int first_wg)
{
    using C = StageCfg<D>;
    using CK = Dkv3Cfg<D, KS>;
    constexpr int NW2 = CK::NW2;
    static_assert(CK::LDS_BYTES <= 160 * 1024, "LDS budget");
    const int G = GQA ? G_arg : 1;                      // query heads per kv head
    static_assert(GQA || !PARTS, "a part has some of a group's query heads");
    __shared__ __attribute__((aligned(1024))) char smem[CK::LDS_BYTES];

    int wg = first_wg + blockIdx.x;
    if constexpr (DR) {
        if (wg >= bias.work) {
            bias_sum<D, 64 * NW2>(reinterpret_cast<float*>(smem), bias, wg - bias.work, threadIdx.x);
            return;
        }
    }
    Place at;
    int part_of = 0;
    if constexpr (PARTS) part_of = take_part(wg, parts);
    const Share sh = kv_block<VL, PAIRS, CK::KEYS>(at, wg, BH, -1, T_arg, nkb_arg, H / G, cu, Ttot);
    if (sh.i < 0) return;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int strip = wave & (KS - 1);           // which 32 keys of the block
    const int role = wave / KS;             // the subtile of every tile this wave fronts; 0 accumulates dV, 1 dK
    const int n = lane & 31, hh = lane >> 5;
    const int gg = lane >> 4, li = lane & 15;

    KvHead kh;
    kv_head_of<D, VL, CK::KEYS>(kh, sh, at, T_arg, nkb_arg, H, G, nt32, Ttot);
    const int T = kh.T, nkb = kh.nkb;
    int g0 = 0, g1 = G;                                 // the workgroup's query heads
    bool alone = true;
    int beyond = 0;
    if constexpr (PARTS) {
        beyond = start_beyond(parts, reinterpret_cast<const uint16_t*>(first), kh.qhead0, G, nqb_arg, sh.i * KS, T, lane);
        if (__builtin_expect(part_of > 0, 0)) {
            if (!in_parts(beyond, sh.i * KS)) return;
            alone = false;
            g0 = part_of * parts.heads;
            g1 = g0 + parts.heads;
        }
    }
    const long base = kh.base, qrow0 = kh.qrow0, qrow_step = kh.qrow_step;
    const long cbase = kh.cbase, cbase_step = kh.cbase_step, cstride = kh.cstride;
    const uint16_t* Qg = nullptr;
    const uint16_t* Gg = nullptr;

    // Per-lane LDS offsets inside a 32-row Q / dO subtile.  The swizzle xors the chunk index,
    // and the chunk indices a lane reads differ in bits the swizzle leaves alone, so one
    // offset per access pattern is kept and the others follow by xor with a constant:
    //   B-operand read of chunk pair s (row = query n):        boff0 ^ (s << 5)
    //   transposing read of column block b, row group t:       qtr0[t] ^ (b << 6)
    const uint32_t boff0 = tile_off_nat<D>(n, hh);
    uint32_t qtr0[2];
    {
        const int row_l = 8 * (gg >> 1) + (li >> 2);
        const int cl = 2 * (gg & 1) + ((li & 3) >> 1);
#pragma unroll
        for (int t = 0; t < 2; ++t) qtr0[t] = tile_off_nat<D>(row_l + 4 * t, cl) + 8 * (li & 1);
    }
    int goff[CK::NPW];
#pragma unroll
    for (int i = 0; i < CK::NPW; ++i) {
        const int row = (wave + NW2 * i) * C::BLK_ROWS + lane / C::CPR;
        goff[i] = (row * D + (((lane % C::CPR) ^ swz_nat<D>(row)) << 3)) * 2;
    }
    const uint32_t smem0 = lds_offset(smem);
    auto stage = [&](int jt, char* sp) __attribute__((always_inline)) {
        const uint16_t* xb = Qg + (long)jt * TK * D;
        const uint16_t* yb = Gg + (long)jt * TK * D;
        if ((jt + 1) * TK <= T) {                           // all 64 rows exist
#pragma unroll
            for (int i = 0; i < CK::NPW; ++i)
                if (wave + NW2 * i < CK::LOADS) {
                    dma16_to_lds_saddr(xb, goff[i], sp + (wave + NW2 * i) * 1024);
                    dma16_to_lds_saddr(yb, goff[i], sp + C::TILE + (wave + NW2 * i) * 1024);
                }
        } else {                                            // rows past T are clamped (their results are masked)
            const int last = T - 1 - jt * TK;
#pragma unroll
            for (int i = 0; i < CK::NPW; ++i)
                if (wave + NW2 * i < CK::LOADS) {
                    const int o = goff[i] - max((wave + NW2 * i) * C::BLK_ROWS + lane / C::CPR - last, 0) * C::ROW;
                    dma16_to_lds_saddr(xb, o, sp + (wave + NW2 * i) * 1024);
                    dma16_to_lds_saddr(yb, o, sp + C::TILE + (wave + NW2 * i) * 1024);
                }
        }
    };
    // scratch: [tile parity][strip][subtile][A, dZ][32 rows of 64 B]
    const uint32_t scr = smem0 + CK::T_OFF + strip * 2 * CK::W_BYTES;
    const uint32_t sw_off = scr_off(n, 2 * hh);                                  // writes: row = query n; second chunk: ^ 16
    uint32_t st_off[2];                                                          // transposing reads
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int row = 8 * (gg >> 1) + (li >> 2) + 4 * t;
        st_off[t] = scr_off(row, 2 * (gg & 1) + ((li & 3) >> 1)) + 8 * (li & 1);
    }

    const float scale = 1.0f / sqrtf((float)D);
    const float c2 = SB_LOG2E * scale;

    bf16x8 kf[D / 16], vf[D / 16];          // A operands: the strip's K and V rows (MFMA row n <- key perm_row(n))
    f32x16 acc[D / 32];                     // dV (role 0) or dK (role 1) of the strip's 32 keys
    const float* cag = nullptr;
    const float* cbg = nullptr;

    // the logits once more, for the log form (see subtile_stage1_log)
    auto logits = [&](uint32_t qa) __attribute__((always_inline)) {
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
        for (int s = 0; s < D / 16; ++s)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], __builtin_bit_cast(bf16x8, lds_load16(qa ^ (s << 5))), acc, 0, 0, 0);
        return acc;
    };
    // this wave's subtile of a tile: logits, dO.v, element-wise path; A and dZ to the scratch
    // qtile: LDS address of the subtile's Q rows (its dO rows lie C::TILE further); sc: LDS
    // address of this strip's scratch for the tile
    auto front = [&](auto mask_c, uint32_t qtile, uint32_t sc, float car, float cbl) __attribute__((always_inline)) {
        constexpr bool MASK = decltype(mask_c)::value;
        if (MASK && n == 0) {               // sees none of the subtile's keys; its carries may be unwritten
            car = 0.0f;
            cbl = 0.0f;
        }
        const uint32_t qa = qtile + boff0;
        u32x4 qw[D / 16], gw[D / 16];
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            qw[s] = lds_load16(qa ^ (s << 5));
            gw[s] = lds_load16((qa ^ (s << 5)) + C::TILE);
        }
        f32x16 sacc, pacc;
#pragma unroll
        for (int r = 0; r < 16; ++r) { sacc[r] = 0.0f; pacc[r] = 0.0f; }
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], __builtin_bit_cast(bf16x8, qw[s]), sacc, 0, 0, 0);
            pacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[s], __builtin_bit_cast(bf16x8, gw[s]), pacc, 0, 0, 0);
        }
        SubtileOut so;
        Chain ch;
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!subtile_stage1<MASK>(ch, sacc, c2, n, hh)) != 0, 0))
            subtile_stage1_log<MASK>(ch, logits(qa), c2, n, hh);
        subtile_stage2<false, true>(so, ch, pacc, car, cbl, hh);
        const uint32_t w = sc + role * CK::W_BYTES + sw_off;
        lds_store16(w, so.pa[0]);
        lds_store16(w ^ 16, so.pa[1]);
        lds_store16(w + CK::M_BYTES, so.pz[0]);
        lds_store16((w ^ 16) + CK::M_BYTES, so.pz[1]);
    };
    // this wave's accumulator += (A or dZ of subtile u)^T (dO or Q rows of subtile u);
    // tile, sc: LDS addresses of the tile buffer and of this strip's scratch for the tile
    auto back = [&](uint32_t tile, uint32_t sc, int u) __attribute__((always_inline)) {
        const uint32_t m = sc + u * CK::W_BYTES + role * CK::M_BYTES;
        const uint32_t x = tile + (role == 0 ? C::TILE : 0) + u * 32 * C::ROW;
        const uint32_t x0 = x + qtr0[0], x1 = x + qtr0[1];
        bf16x8 mt[2], op[D / 16];
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) mt[s2] = tr_pair_at(m + st_off[0] + (16 * s2) * 64, m + st_off[1] + (16 * s2) * 64);
#pragma unroll
        for (int b = 0; b < D / 32; ++b)
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                const int ro = (16 * s2) * C::ROW;
                op[2 * b + s2] = tr_pair_at((x0 ^ (b << 6)) + ro, (x1 ^ (b << 6)) + ro);
            }
#pragma unroll
        for (int b = 0; b < D / 32; ++b)
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2)
                acc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(mt[s2], op[2 * b + s2], acc[b], 0, 0, 0);
    };

    // front of this wave's subtile (Q rows at qtile) and back of the tile before (buffer ptile,
    // scratch scp), unmasked and complete, written as one block so that the matrix
    // instructions of one part can be issued between the vector instructions of the other.
    // xn, yn: Q and dO rows of the tile to stage meanwhile, spn: its LDS buffer.
    // The wave's priority falls from part to part: of the two waves of a SIMD the one that is
    // behind wins the arbitration, so they reach the barrier closer together.
    auto step = [&](uint32_t qtile, uint32_t sc, uint32_t ptile, uint32_t scp, float car, float cbl,
                    const uint16_t* xn, const uint16_t* yn, const char* spn) __attribute__((always_inline)) {
        const uint32_t qa = qtile + boff0;
        // part A: logits
        __builtin_amdgcn_s_setprio(3);
        u32x4 qw[D / 16], gw[D / 16];
#pragma unroll
        for (int s = 0; s < D / 16; ++s) qw[s] = lds_load16(qa ^ (s << 5));
        f32x16 sacc, pacc;
#pragma unroll
        for (int r = 0; r < 16; ++r) { sacc[r] = 0.0f; pacc[r] = 0.0f; }
        // the staging loads go out between the matrix instructions
        static_assert(2 * CK::NPW <= D / 16 && CK::LOADS == CK::NPW * NW2, "whole staging loads");
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], __builtin_bit_cast(bf16x8, qw[s]), sacc, 0, 0, 0);
            constexpr int EVERY = D / 16 / (2 * CK::NPW);
            const int i = s / EVERY / 2;
            if (s % EVERY == 0)
                dma16_to_lds_saddr(s / EVERY % 2 ? yn : xn, goff[i], spn + (s / EVERY % 2 ? C::TILE : 0) + (wave + NW2 * i) * 1024);
        }
#pragma unroll
        for (int s = 0; s < D / 16; ++s) gw[s] = lds_load16((qa ^ (s << 5)) + C::TILE);
        __builtin_amdgcn_sched_barrier(0);
        __builtin_amdgcn_s_setprio(2);
        // part B: the chain of the logits (vector) beside dO.v and the back of subtile 0 (matrix)
        Chain ch;
        const bool fits = subtile_stage1<false>(ch, sacc, c2, n, hh);
#pragma unroll
        for (int s = 0; s < D / 16; ++s)
            pacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[s], __builtin_bit_cast(bf16x8, gw[s]), pacc, 0, 0, 0);
        back(ptile, scp, 0);
        __builtin_amdgcn_sched_barrier(0);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!fits) != 0, 0)) subtile_stage1_log<false>(ch, logits(qa), c2, n, hh);
        __builtin_amdgcn_s_setprio(1);
        // part C: A, G, dZ (vector) beside the back of subtile 1 (matrix)
        SubtileOut so;
        subtile_stage2<false, true>(so, ch, pacc, car, cbl, hh);
        back(ptile, scp, 1);
        const uint32_t w = sc + role * CK::W_BYTES + sw_off;
        lds_store16(w, so.pa[0]);
        lds_store16(w ^ 16, so.pa[1]);
        lds_store16(w + CK::M_BYTES, so.pz[0]);
        lds_store16((w ^ 16) + CK::M_BYTES, so.pz[1]);
        __builtin_amdgcn_s_setprio(0);
        __builtin_amdgcn_sched_barrier(0);
    };

    float cn0, cn1;                                          // ca, cb of this wave's subtile of the next tile
    const uint32_t* fg = nullptr;
    // rows past T: an infinite carry gives A = 0 and G = 0, and with cb = 0 also dZ = 0 (a dead
    // strip's rows lie outside the arrays; those of queries that do not reach the keys are not used)
    auto load_carries = [&](int jt, bool live) __attribute__((always_inline)) {
        const int j = jt * TK + 32 * role + n;
        cn0 = (j < T && live) ? cag[j] : INFINITY;
        cn1 = (j < T && live) ? cbg[j] : 0.0f;
    };
    // a head's first tile for block kb, into buffer b, and its carries
    auto first_tile = [&](int g, int kb, int b) __attribute__((always_inline)) {
        const int k0 = kb * CK::KEYS + strip * 32, jt0 = kb * CK::KEYS / TK;
        Qg = q + (qrow0 + g * qrow_step) * D;
        Gg = dout + (qrow0 + g * qrow_step) * D;
        cag = ca + cbase + g * cbase_step + (k0 >> 5) * cstride;
        cbg = cb + cbase + g * cbase_step + (k0 >> 5) * cstride;
        fg = first + (kh.qhead0 + g) * 2 * nqb_arg;
        load_carries(jt0, k0 < T);
        stage(jt0, smem + b * C::STAGE);
    };
    // All that block kb starts from: the first tile into buffer b, K into the one after it, V into half p of the
    // scratch; from there into registers: as whole rows and once, not as 32 bytes of 32 rows an instruction and by
    // both waves of a strip.  These 96 KB take a CU 6 us, a third of a short block's time.  A pair's second
    // block asks for them in the last interval of the first, which reads none of these three places, so that they
    // arrive under its back and its stores: B8 H16 T4096 all near 347 -> 318 us, a third far 634 -> 614, all far
    // 1290 -> 1268.
    static_assert(CK::KEYS * C::ROW <= C::STAGE && CK::KEYS * C::ROW <= CK::SCR_BUF, "the block's rows fit");
    int buf0 = 0, vhalf = 0;
    auto begin = [&](int kb, int b, int p) __attribute__((always_inline)) {
        buf0 = b;
        vhalf = p;
        first_tile(g0, kb, b);
        constexpr int KLOADS = CK::KEYS * C::ROW / 1024 / NW2;
        const int K0 = kb * CK::KEYS;
        char* const kp = smem + (b == 2 ? 0 : b + 1) * C::STAGE;
        char* const vp = smem + CK::T_OFF + p * CK::SCR_BUF;
#pragma unroll
        for (int i = 0; i < KLOADS; ++i) {
            const int row = (wave + NW2 * i) * C::BLK_ROWS + lane / C::CPR;
            const int off = (min(row, T - 1 - K0) * D + (((lane % C::CPR) ^ swz_perm<D>(row)) << 3)) * 2;
            dma16_to_lds_saddr(k + base + (long)K0 * D, off, kp + (wave + NW2 * i) * 1024);
            dma16_to_lds_saddr(v + base + (long)K0 * D, off, vp + (wave + NW2 * i) * 1024);
        }
    };
    begin(sh.i, 0, 0);
    for (int part = 0;; ++part) {
        const int kb = part == 0 ? sh.i : nkb - 1 - sh.i;    // small kb = most later queries = first
        const bool more = PAIRS && part == 0 && 2 * sh.i != nkb - 1;   // odd block count: the middle block is alone
        const int K0 = kb * CK::KEYS;
        const int k0 = K0 + strip * 32;                      // the strip's 32 keys
        const int kt32 = k0 >> 5;
        const bool live = k0 < T;
        const int jt0 = K0 / TK;
        const int nqb = (T + BQ - 1) / BQ;
        dma_wait<0>();
        barrier_lds();
        if (PARTS && part_of == 0 && __builtin_expect(in_parts(beyond, sh.i * KS), 0)) {
            alone = false;
            g1 = parts.heads;
        }
        {
            const uint32_t at = strip * 32 * C::ROW + tile_off_perm<D>(perm_row(n), hh);
            const uint32_t ka = smem0 + (buf0 == 2 ? 0 : buf0 + 1) * C::STAGE + at;
            const uint32_t va = smem0 + CK::T_OFF + vhalf * CK::SCR_BUF + at;
#pragma unroll
            for (int s = 0; s < D / 16; ++s) {
                kf[s] = __builtin_bit_cast(bf16x8, lds_load16(ka ^ (s << 5)));
                vf[s] = __builtin_bit_cast(bf16x8, lds_load16(va ^ (s << 5)));
            }
        }
#pragma unroll
        for (int b = 0; b < D / 32; ++b)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[b][r] = 0.0f;

        // the query heads of the group one after the other, into the same accumulators
        for (int g = g0; g < g1; ++g) {
        if (g > g0) {
            dma_wait<0>();                                   // the steady state's last staging, read by nobody
            barrier_lds();                                   // everyone is done with the LDS of the head before
            first_tile(g, kb, buf0);
        }

        // ---- sweep over 64-row query tiles, from the block's diagonal to the end.  Interval
        // `it` (between two barriers) holds the front of tile jt0 + it (buffer (buf0 + it) % 3, scratch
        // it & 1) and the back of tile jt0 + it - 1; the staging loads of tile jt0 + it + 1 are
        // issued at its start, after the carries of that tile (vector memory operations
        // complete in order, so the carries must not queue behind the staging loads).
        const Reach reach = reach_of(fg, start_words(fg, K0 / BQ, nqb, lane), K0 >> 5, (K0 >> 5) + KS - 1, nqb, lane);
        const int ntile = min((T + TK - 1) / TK, reach.end) - jt0;
        const int ndiag = min(ntile, CK::KEYS / TK);              // tiles that touch the diagonal band
        // steady state (the intervals hot_begin .. hot_end - 1): the strip is live, tile `it` is past
        // the diagonal band and complete, and the next tile is complete and reaches the block's keys,
        // or does not exist
        const int nfull = min(max(T / TK - jt0, 0), ntile);
        const int hot_begin = ndiag + 1;
        const int sure = reach.sure - jt0;
        const int hot_end = !live ? 0 : min(nfull == ntile ? ntile : nfull - 1, sure < ntile ? sure - 1 : ntile);
        // which strips of the queries reach this wave's keys: of tile it - 1, it, it + 1
        int there_prev = 0, there = 0;
        uint32_t word_next = start_word(fg, jt0, reach.sure);
        int it = 0;
        while (it <= ntile) {
            if (it == hot_begin && it < hot_end) {
                // LDS addresses of the tile buffers of tiles it, it - 1, it + 1 and of the scratch
                // of tiles it, it - 1; they rotate, nothing is recomputed.  The tile staged in an
                // interval is tile it + 1, or, after the last one, that tile once more (never read).
                uint32_t a_cur = smem0 + ((buf0 + it) % 3) * C::STAGE, a_prev = smem0 + ((buf0 + it + 2) % 3) * C::STAGE;
                uint32_t a_next = smem0 + ((buf0 + it + 1) % 3) * C::STAGE;
                uint32_t s_cur = scr + (it & 1) * CK::SCR_BUF, s_prev = scr + ((it + 1) & 1) * CK::SCR_BUF;
                const int tn = min(it + 1, ntile - 1);
                const uint16_t* xn = Qg + (long)(jt0 + tn) * TK * D;
                const uint16_t* yn = Gg + (long)(jt0 + tn) * TK * D;
                const float* cap = cag + (jt0 + tn) * TK + 32 * role + n;
                const float* cbp = cbg + (jt0 + tn) * TK + 32 * role + n;
                for (; it < hot_end; ++it) {
                    dma_wait<0>();
                    barrier_lds();
                    const float car = cn0, cbl = cn1;
                    cn0 = *cap;
                    cn1 = *cbp;
                    step(a_cur + role * 32 * C::ROW, s_cur, a_prev, s_prev, car, cbl, xn, yn, smem + (a_next - smem0));
                    const int adv = it + 2 < ntile ? TK : 0;
                    xn += adv * D;
                    yn += adv * D;
                    cap += adv;
                    cbp += adv;
                    const uint32_t t = a_prev;
                    a_prev = a_cur;
                    a_cur = a_next;
                    a_next = t;
                    const uint32_t u = s_prev;
                    s_prev = s_cur;
                    s_cur = u;
                }
                there = 3;                               // the tile before and, if there is one, this one
                word_next = 0;
                continue;
            }
            const int bcur = (buf0 + it) % 3, bprev = (buf0 + it + 2) % 3, bnext = (buf0 + it + 1) % 3;   // buffers of tiles it, it - 1, it + 1
            dma_wait<0>();
            barrier_lds();        // tile `it` has landed, the scratch of tile it-1 is complete, tile it-2 is free
            const float car = cn0, cbl = cn1;
            there_prev = there;
            there = reaching(word_next, kt32);
            if (it + 1 < ntile) {
                const int jt = jt0 + it + 1;
                load_carries(jt, live);
                word_next = start_word(fg, jt, reach.sure);
                stage(jt, smem + bnext * C::STAGE);
            } else if (it == ntile && more && g == g1 - 1) {
                begin(nkb - 1 - kb, bcur, it & 1);
            }
            const int jbase = (jt0 + it) * TK;
            const uint32_t qt = smem0 + bcur * C::STAGE + role * 32 * C::ROW;
            const uint32_t sc = scr + (it & 1) * CK::SCR_BUF;
            const uint32_t spp = smem0 + bprev * C::STAGE;
            const uint32_t scp = scr + ((it + 1) & 1) * CK::SCR_BUF;
            const int j0 = jbase + 32 * role;
            if (it < ntile && live && j0 < T && (there >> role & 1)) {
                if (it < ndiag) {
                    if (j0 == k0) front(bc<true>{}, qt, sc, car, cbl);
                    else if (j0 > k0) front(bc<false>{}, qt, sc, car, cbl);
                } else {
                    front(bc<false>{}, qt, sc, car, cbl);
                }
            }
            if (it >= 1 && live) {
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const int ju = jbase - TK + 32 * u;
                    if (ju >= k0 && ju < T && (there_prev >> u & 1)) back(spp, scp, u);
                }
            }
            ++it;
        }
        }

        if (PARTS && !alone) {
            const PartSums<D> sums(parts, sh.bh, VL != Packed::NO ? H / G : BH, VL != Packed::NO ? Ttot : T_arg);
            if (live) store_strip<D, true>((role == 0 ? sums.dv : sums.dk) + part_of * sums.step + base + (long)k0 * D, T - k0, acc, 1.0f, n, hh);
            add_parts<D, 64 * NW2>(sums, parts.n, smem, base + (long)K0 * D, kh.qhead0 / G * nt32 + (K0 >> 5), min(T - K0, CK::KEYS), dk, dv, scale, tid);
            return;
        }
        if (live) store_strip<D>((role == 0 ? dv : dk) + base + (long)k0 * D, T - k0, acc, role == 0 ? 1.0f : scale, n, hh);
        if (!more) break;
    }
}

// ------------------------------------------------------------------ small grids
// Where the 128-row blocks leave most of the chip idle, what counts is the length of one row's chain of
// subtiles.  Here a workgroup takes one strip of 32 rows, and its waves share the other side's subtiles, each
// staging its own, without a barrier for the tiles.  Still bound by the chain: B2 H4 T777 d32 takes 8 + 8 us,
// of which 4 to 5 each are a launch and its first loads.  Which grids: small_grid().
template <int D, int NW_ = D == 128 ? 4 : 8> struct SmallCfg {
    static constexpr int NWS = NW_;                     // waves (four at d <= 64: four_waves())
    static constexpr int ROW = D * 2;
    static constexpr int SUB = 32 * ROW;                // one 32-row subtile of one matrix
    static constexpr int WAVE = 4 * SUB;                // two matrices, double buffered
    static constexpr int MAXSUB = D == 64 && NWS == 4 ? 96 : 128;      // (two workgroups a CU) subtiles of a strip for whose carries there is room
    static constexpr int LOADS = SUB / 1024;            // of 16 bytes a lane, for a subtile
};

// byte offsets inside a 32-row subtile of what a lane fetches with its loads
template <int D, bool PERM>
__device__ __forceinline__ void subtile_offsets(int (&off)[SmallCfg<D>::LOADS], int lane)
{
    using C = SmallCfg<D>;
    constexpr int CPR = C::ROW / 16;
#pragma unroll
    for (int i = 0; i < C::LOADS; ++i) {
        const int row = i * (1024 / C::ROW) + lane / CPR;
        off[i] = PERM ? tile_off_perm<D>(row, lane % CPR) : tile_off_nat<D>(row, lane % CPR);
    }
}
// the subtile that begins at `src` (wave-uniform), by one wave, to LDS address `lds`; only `rows` of its rows exist: those past
// them are clamped
template <int D>
__device__ __forceinline__ void stage_rows(const uint16_t* src, int rows, uint32_t lds, const int (&off)[SmallCfg<D>::LOADS], int lane)
{
    using C = SmallCfg<D>;
    if (rows >= 32) {
        dma16_to_lds_run_at(scalar_base(src), off, lds);
        return;
    }
    int o[C::LOADS];
#pragma unroll
    for (int i = 0; i < C::LOADS; ++i) o[i] = off[i] - max(i * (1024 / C::ROW) + lane / (C::ROW / 16) - (rows - 1), 0) * C::ROW;
    dma16_to_lds_run_at(scalar_base(src), o, lds);
}

// The strip's own 32 rows of two matrices, into the places x_at and y_at in LDS: whole rows and once, every wave its share.  (As
// operands from memory, 32 bytes of 32 rows an instruction and all of it by every wave, the two took a CU 2000, 4800 and 7000 clocks
// at d = 32, 64 and 128: a tenth to a third of a near strip's time.)
template <int D, int NWS>
__device__ __forceinline__ void stage_strip(const uint16_t* X, const uint16_t* Y, int rows, uint32_t x_at, uint32_t y_at, int wave, int lane)
{
    using C = SmallCfg<D>;
    constexpr int CPR = C::ROW / 16;
    for (int i = wave; i < 2 * C::LOADS; i += NWS) {
        const bool x = i < C::LOADS;
        const int j = x ? i : i - C::LOADS, row = j * (1024 / C::ROW) + lane / CPR;
        dma16_to_lds_at(scalar_base(x ? X : Y), min(row, rows - 1) * C::ROW + (((lane % CPR) ^ swz_perm<D>(row)) << 4), (x ? x_at : y_at) + j * 1024);
    }
}

// by how much a row's carries are too large, `left` being the one of the diagonal's subtile: rounding, if it is that small
__device__ __forceinline__ float overshoot(float left) { return fabsf(left) < 16.0f ? left : 0.0f; }

// what a wave has staged has landed, and its reads of the buffer to be refilled have returned
__device__ __forceinline__ void own_landed() { asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory"); }

// Query-stationary pass: a sweep from the left to the diagonal, a round of one subtile per wave at a time: logits and chains;
// one barrier to add up the softplus totals; A and G; one barrier to add up the G of the subtiles further left; dZ.  What the
// carries start from is m.  Where m says that the rows are exhausted on the way, the totals are taken first, from the diagonal
// on, until they are: that is where the sweep starts, and the sums are its carries.
// Counting down from m, a row's carries are all off by what is left at the diagonal, where nothing should be: the roundings of m and
// of the sums on the way, of numbers as large as m, 2e-5 of a weight where m is near exhaustion.  Every weight, and all that is linear in them,
// is off by the same factor; overshoot() takes it out, here of dQ, in the key-stationary pass of A and dZ.  (Share of the bf16 weights above 2^-12 that
// are rounded otherwise than in fp64, rows with 80 to 130 bits of their stick used up, H8 T1000 d128: 1.5e-3 -> 9e-4, as with totals from the diagonal.
// Costs up to 1 % of a step, 2 % where the heads of a group of 8 share a kv head.)
// Against totals of all subtiles first, in every strip, and one wave adding them up one after the other, all heads far, then none, us:
// B2 H4 T777 d32 12.5 -> 9.1, 7.3 -> 6.7; B1 H4 T4000 d64 56 -> 38, 22.5 -> 13.3; B1 H8 T700 d128 21.3 -> 16.6, 14.2 -> 12.5.
template <int D, bool RB, int NWS>
__global__ void __launch_bounds__(64 * NWS)
bwd_dq_small_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                    const uint16_t* __restrict__ v, const uint16_t* __restrict__ rb,
                    const float* __restrict__ m,
                    const uint16_t* __restrict__ dout, float* __restrict__ dq,
                    float* __restrict__ ca, float* __restrict__ cb, uint16_t* __restrict__ first,
                    int T_arg, int BH, int H, int G, int n_arg, int nqb_arg, int nt32,       // n_arg: strips a head; packed batch: sequences
                    const int* __restrict__ cu, int Ttot, BiasGrad bias, int* __restrict__ arrived)
{
    using C = SmallCfg<D, NWS>;
    constexpr int NTHR = 64 * NWS;
    __shared__ __attribute__((aligned(1024))) char smem[NWS * C::WAVE];
    __shared__ __attribute__((aligned(1024))) float s_car[C::MAXSUB][32];      // carries per subtile, from the diagonal on, and row
    __shared__ float s_l[2][NWS][32], s_g[2][NWS][32];  // a round's softplus totals, and sums of G
    static_assert(NWS * 32 * D * 4 <= NWS * C::WAVE, "the partial gradients fit");

    asm volatile("" :: "s"(q), "s"(k), "s"(v), "s"(m), "s"(dout), "s"(T_arg), "s"(G));
    const int tid = threadIdx.x, lane = tid & 63;
    static_assert(NTHR * 8 / D * (D + 4) * 4 <= (int)sizeof(smem), "the partial sums fit");
    if (RB && (int)blockIdx.x >= bias.work) {
        bias_partial_at<D, NTHR>(reinterpret_cast<float*>(smem), blockIdx.x - bias.work, bias, m, dout, T_arg, cu, n_arg, Ttot, tid);
        return;
    }
    const Share sh = in_scalars(share_of(blockIdx.x, BH, -1));
    const int head = sh.bh % H;
    int bh = sh.bh, T = T_arg, nstrip = n_arg, i = sh.i;
    long row0 = bh * (long)T, kvrow0 = (long)(G == 1 ? bh : (int)((unsigned)bh / (unsigned)G)) * T;
    long cbase = (long)bh * nt32 * T, cstride = T;
    if (cu) {                                           // packed batch: sh.bh is the head alone, sh.i its place
        const Place at = place_of<32>(sh.i, cu, n_arg, Ttot, T_arg, lane);
        if (at.T == 0) return;
        T = at.T;
        nstrip = (T + 31) / 32;
        i = at.i;
        bh = at.seq * H + head;
        row0 = (long)head * Ttot + at.c0;
        kvrow0 = (long)(head / G) * Ttot + at.c0;
        cbase = (long)head * nt32 * Ttot + at.c0;
        cstride = Ttot;
    }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, hh = lane >> 5, gg = lane >> 4, li = lane & 15;
    const int strip = nstrip - 1 - i;
    const int q0 = strip * 32;
    const int nlast = min(T - q0, 32);                  // rows of the strip, and of the subtile on the diagonal
    const uint16_t* Kg = k + kvrow0 * D;
    const uint16_t* Vg = v + kvrow0 * D;
    const uint32_t base = lds_offset(smem) + wave * C::WAVE;
    const uint32_t ka = base + tile_off_perm<D>(perm_row(n), hh);       // A operands, ^ (s << 5)
    uint32_t ktr[2];                                                    // transposing reads, ^ (b << 6)
#pragma unroll
    for (int t = 0; t < 2; ++t)
        ktr[t] = base + tile_off_perm<D>(16 * (gg >> 1) + (li >> 2) + 4 * t, 2 * (gg & 1) + ((li & 3) >> 1)) + 8 * (li & 1);
    const float scale = 1.0f / sqrtf((float)D);
    const float c2 = SB_LOG2E * scale;
    int off[C::LOADS];
    subtile_offsets<D, true>(off, lane);
    auto stage_k = [&](int sub, int st) __attribute__((always_inline)) {
        stage_rows<D>(Kg + (long)sub * 32 * D, sub == strip ? nlast : 32, base + st * 2 * C::SUB, off, lane);
    };
    auto stage_v = [&](int sub, int st) __attribute__((always_inline)) {
        stage_rows<D>(Vg + (long)sub * 32 * D, sub == strip ? nlast : 32, base + st * 2 * C::SUB + C::SUB, off, lane);
    };

    // all that is needed whatever m says, at once; Q and dO pass through the place of the carries
    float a2 = -m[row0 + min(q0 + n, T - 1)] * SB_LOG2E;
    static_assert(2 * C::SUB <= (int)sizeof(s_car), "the strip's rows fit");
    const uint32_t x_at = lds_offset(reinterpret_cast<const char*>(s_car)), y_at = x_at + C::SUB;
    stage_strip<D, NWS>(q + (row0 + q0) * D, dout + (row0 + q0) * D, nlast, x_at, y_at, wave, lane);
    if (wave <= strip) stage_k(wave, 0);
    own_landed();
    barrier_nofence();
    bf16x8 qf[D / 16], gf[D / 16];
    {
        const uint32_t at = tile_off_perm<D>(n, hh);
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            qf[s] = __builtin_bit_cast(bf16x8, lds_load16((x_at + at) ^ (s << 5)));
            u32x4 x = lds_load16((y_at + at) ^ (s << 5));
            if (n >= nlast) x = u32x4{0u, 0u, 0u, 0u};   // rows past T contribute nothing
            gf[s] = __builtin_bit_cast(bf16x8, x);
        }
    }
    float bsum = 0.0f;                      // sum of G over the keys left of the round
    if constexpr (RB) {                     // remainder bias, as in bwd_dq_kernel
        const u32x4* rs = reinterpret_cast<const u32x4*>(rb + head * D + 8 * hh);
        float dot = 0.0f;
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            const bf16x8 rr = __builtin_bit_cast(bf16x8, rs[2 * s]);
#pragma unroll
            for (int e = 0; e < 8; ++e) dot += (float)gf[s][e] * (float)rr[e];
        }
        float d_lo, d_hi;
        both_halves(dot, d_lo, d_hi);
        bsum = fast_exp2(-a2) * (d_lo + d_hi);
    }
    asm volatile("" :: "v"(bsum));

    auto rows_by = [&](uint32_t rows, const bf16x8 (&f)[D / 16]) __attribute__((always_inline)) {
        u32x4 w[D / 16];
#pragma unroll
        for (int s = 0; s < D / 16; ++s) w[s] = lds_load16(rows ^ (s << 5));
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
        for (int s = 0; s < D / 16; ++s)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, w[s]), f[s], acc, 0, 0, 0);
        return acc;
    };
    auto sums_of = [&](const float (&a)[NWS][32], float (&x)[NWS]) __attribute__((always_inline)) {
#pragma unroll
        for (int w = 0; w < NWS; ++w) x[w] = a[w][n];
    };

    int start = 0;
    bool ends = __builtin_amdgcn_ballot_w64(!(a2 < CARRY_EXHAUSTED)) != 0;     // some row is exhausted on the way: all may be
    if (!ends) {
        if (wave <= strip) stage_v(wave, 0);
    } else {
        // ---- totals from the diagonal on.  A round takes subtiles lo .. lo + NWS - 1
        float right = 0.0f;
        bool more = true;
        int top = strip;
        for (int st = 0; more && top >= 0 && strip - top < C::MAXSUB; top -= NWS, st ^= 1) {
            const int lo = max(top - (NWS - 1), 0), sub = lo + wave;
            float l = 0.0f;
            if (sub <= top) {
                if (top == strip && lo > 0) stage_k(sub, 0);
                own_landed();
                if (lo > 0 && max(lo - NWS, 0) + wave < lo) stage_k(max(lo - NWS, 0) + wave, st ^ 1);
                const f32x16 s = rows_by(ka + st * 2 * C::SUB, qf);
                l = sub == strip ? sp2_total<true>(s, c2, n, hh) : sp2_total<false>(s, c2, n, hh);
            }
            float l_lo, l_hi, t[NWS];
            both_halves(l, l_lo, l_hi);
            if (hh == 0) s_l[st][wave][n] = l_lo + l_hi;
            barrier_lds();                               // (the first: Q and dO have been read)
            sums_of(s_l[st], t);
#pragma unroll
            for (int w = NWS - 1; w >= 0; --w) {
                if (lo + w > top) continue;
                if (more) {
                    if (wave == 0 && hh == 0) s_car[strip - (lo + w)][n] = right;
                    more = __builtin_amdgcn_ballot_w64(!(right >= CARRY_EXHAUSTED)) != 0;      // alike in all waves
                }
                if (more) {
                    start = lo + w;
                    right += t[w];
                }
            }
        }
        if (more && top >= 0) {                          // not among those there is room for: from the left and m, as the others
            ends = false;
            start = 0;
        }
        own_landed();                                    // a subtile asked for before the end was found
        if (start + wave <= strip) {
            stage_k(start + wave, 0);
            stage_v(start + wave, 0);
        }
        barrier_lds();                                   // the carries are there
    }
    // (where this pass takes strips the key-stationary one does too, so that nobody reads the places of strips that do not exist)
    if (tid == 0) {
        first[(long)bh * nqb_arg * 4 + strip] = (uint16_t)start;
        if (arrived && head % G == 0) arrived[(long)(bh / G) * nt32 + strip] = 0;
    }

    // ---- the sweep
    f32x16 dqacc[D / 32];
#pragma unroll
    for (int b = 0; b < D / 32; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) dqacc[b][r] = 0.0f;
    float* const cag = ca + cbase;
    float* const cbg = cb + cbase;
    for (int sub0 = start, st = 0; sub0 <= strip; sub0 += NWS, st ^= 1) {
        const int sub = sub0 + wave;
        const bool there = sub <= strip;
        Chain ch;
        SubtileOut so;
        so.g_tot = 0.0f;
        float car = 0.0f, l_tot = 0.0f;
        const uint32_t buf = st * 2 * C::SUB;
        if (there) {
            own_landed();
            if (sub + NWS <= strip) {
                stage_k(sub + NWS, st ^ 1);
                stage_v(sub + NWS, st ^ 1);
            }
            const f32x16 s = rows_by(ka + buf, qf);
            const bool fits = sub == strip ? subtile_stage1<true>(ch, s, c2, n, hh) : subtile_stage1<false>(ch, s, c2, n, hh);
            if (__builtin_expect(__builtin_amdgcn_ballot_w64(!fits) != 0, 0)) {
                const f32x16 again = rows_by(ka + buf, qf);
                if (sub == strip) subtile_stage1_log<true>(ch, again, c2, n, hh);
                else subtile_stage1_log<false>(ch, again, c2, n, hh);
            }
            float l_lo, l_hi;
            both_halves(ch.l, l_lo, l_hi);
            l_tot = l_lo + l_hi;
        }
        if (ends) {
            car = s_car[max(strip - sub, 0)][n];
        } else {
            float t[NWS];
            if (hh == 0) s_l[st][wave][n] = l_tot;
            barrier_lds();
            sums_of(s_l[st], t);
#pragma unroll
            for (int w = 0; w < NWS; ++w) {
                a2 -= t[w];
                if (w == wave) car = a2;
            }
        }
        bf16x8 kt[D / 16];
        if (there) {
            subtile_g<false, false>(so, ch, rows_by(ka + buf + C::SUB, gf), car, hh);
#pragma unroll
            for (int b = 0; b < D / 32; ++b)
#pragma unroll
                for (int s = 0; s < 2; ++s)
                    kt[2 * b + s] = tr_pair_at(((ktr[0] + buf) ^ (b << 6)) + 8 * s * C::ROW, ((ktr[1] + buf) ^ (b << 6)) + 8 * s * C::ROW);
        }
        if (hh == 0) s_g[st][wave][n] = so.g_tot;
        barrier_lds();
        float left = bsum, t[NWS];
        sums_of(s_g[st], t);
#pragma unroll
        for (int w = 0; w < NWS; ++w) {
            if (w == wave) left = bsum;
            bsum += t[w];
        }
        if (there) {
            if (hh == 0 && n < nlast) {
                const long ci = (long)sub * cstride + q0 + n;
                cag[ci] = car;
                cbg[ci] = left;
            }
            subtile_dz(so, ch, left, hh);
#pragma unroll
            for (int b = 0; b < D / 32; ++b)
#pragma unroll
                for (int s = 0; s < 2; ++s)
                    dqacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(so.pz[s], kt[2 * b + s], dqacc[b], 0, 0, 0);
        }
    }

    // ---- the waves' shares added up, in a fixed order.  dqacc[b][r] is query row 8*(r/4) + 4*hh + r%4, column 32b + n
    barrier_lds();                                       // everyone is done with the tiles
    float* const red = reinterpret_cast<float*>(smem);
    float* const right = s_l[0][0];                      // factor of a row
    if (wave == 0 && hh == 0) right[n] = ends ? 1.0f : fast_exp2(overshoot(a2));
#pragma unroll
    for (int b = 0; b < D / 32; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) red[(wave * 32 + 8 * (r >> 2) + 4 * hh + (r & 3)) * D + 32 * b + n] = dqacc[b][r];
    barrier_lds();
    for (int i = tid; i < 32 * D / 4; i += NTHR) {
        const int row = i / (D / 4), c = 4 * (i % (D / 4));
        f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < NWS; ++w) x += *reinterpret_cast<const f32x4*>(&red[(w * 32 + row) * D + c]);
        if (q0 + row < T) *reinterpret_cast<f32x4*>(dq + (row0 + q0 + row) * D + c) = x * (scale * right[row]);
    }
}

// Key-stationary pass: a strip of 32 keys a workgroup, whose waves take its query subtiles (of all
// query heads of the group) in turn and add their accumulators up at the end.
template <int D, bool DR, int NWS, bool PARTS>
__global__ void __launch_bounds__(64 * NWS, D == 32 && NWS == 4 ? 3 : 1)        // (three workgroups a CU: left alone it takes registers for two)
bwd_dkv_small_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                     const uint16_t* __restrict__ v, const uint16_t* __restrict__ dout,
                     const float* __restrict__ ca, const float* __restrict__ cb,
                     float* __restrict__ dk, float* __restrict__ dv, const uint16_t* __restrict__ first,
                     int T_arg, int BH, int H, int G_arg, int n_arg, int nqb_arg, int nt32,       // n_arg: strips a head; packed batch: sequences
                     const int* __restrict__ cu, int Ttot, bool strips_q, BiasGrad bias, Parts parts)       // strips_q: the carries are bwd_dq_small_kernel's
{
    using C = SmallCfg<D, NWS>;
    constexpr int NTHR = 64 * NWS;
    constexpr int WAVE = C::WAVE;                        // Q and dO subtiles, double buffered; A and dZ take their place in turn
    static_assert(2 * SCR_MAT <= 2 * C::SUB, "A and dZ fit");
    __shared__ __attribute__((aligned(1024))) char smem[NWS * WAVE];
    static_assert(NWS * WAVE <= 160 * 1024, "LDS budget");

    asm volatile("" :: "s"(q), "s"(k), "s"(v), "s"(dout), "s"(ca), "s"(cb), "s"(first), "s"(T_arg));
    const int tid = threadIdx.x, lane = tid & 63;
    if (DR && (int)blockIdx.x >= bias.work) {
        bias_sum<D, NTHR>(reinterpret_cast<float*>(smem), bias, blockIdx.x - bias.work, tid);
        return;
    }
    int wg = blockIdx.x;
    int part = 0;
    if constexpr (PARTS) part = take_part(wg, parts);
    const Share sh = in_scalars(share_of(wg, BH, -1));
    KvHead kh;
    int ks = sh.i;                                       // the strip; small ones have the most queries
    if (cu) {                                            // packed batch: sh.bh is the head alone, sh.i its place
        const Place at = place_of<32>(sh.i, cu, n_arg, Ttot, T_arg, lane);
        if (at.T == 0) return;
        packed_kv_head<D>(kh, at, sh.bh, 32, H, G_arg, nt32, Ttot);
        ks = at.i;
    } else {
        kv_head(kh, sh.bh, D, T_arg, n_arg, G_arg, nt32);
    }
    const int T = kh.T, nstrip = kh.nkb;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n = lane & 31, hh = lane >> 5, gg = lane >> 4, li = lane & 15;
    const int k0 = ks * 32;
    const int nq = nstrip - ks;                          // query strips from the keys' own on
    const int nlast = T - (nstrip - 1) * 32;             // rows of the last

    // Which of them reach the keys, as bits, 64 strips at a time of all heads' one after the other: `todo` holds those left of the
    // wave's share, every NWS-th.  The words to come are fetched one ahead.  (With head, strip and addresses worked out anew for
    // every strip, all heads far, us: B1 H8 Hkv1 T1000 d128 124 -> 103, T4096 d64 203 -> 185, near 34 -> 25; B1 H8 T700 d128 18.6 -> 17.0.
    // With a word for each head, a memory latency each, B2 H8 Hkv2 T90 d32 6.6 us in place of 5.7, B8 H32 Hkv4 T800 51 in place of 47, near 44 in place of 39.)
    constexpr unsigned long long EVERY = NWS == 8 ? 0x0101010101010101ull : 0x1111111111111111ull;
    static_assert(NWS == 4 || NWS == 8, "strips of a wave");
    bool alone = true;
    int G = G_arg;
    long qhead0 = kh.qhead0;
    int beyond = 0;
    if constexpr (PARTS) {
        beyond = start_beyond(parts, first, kh.qhead0, G, nqb_arg, ks, T, lane);
        if (__builtin_expect(part > 0, 0)) {
            if (!in_parts(beyond, ks)) return;
            alone = false;
            G = parts.heads;                             // the part's heads are the strip's
            qhead0 += part * G;
            kh.qrow0 += part * G * kh.qrow_step;
            kh.cbase += part * G * kh.cbase_step;
        }
    }
    int all = G * nq;
    int w0 = 0, wn = 0, g = 0, x0 = 0;                   // first strip of this word, and of the next one; head, and where its strips begin
    unsigned long long todo = 0;
    const uint16_t* const fg = first + qhead0 * nqb_arg * 4 + ks;
    auto word = [&](int x) __attribute__((always_inline)) {
        int head = 0, i = x;
        if (G > 1) {                                     // (from a quotient good to less than one)
            head = (int)((float)x * __builtin_amdgcn_rcpf((float)nq));
            i = x - head * nq;
            const int up = i >= nq ? 1 : i < 0 ? -1 : 0;
            head += up;
            i -= up * nq;
        }
        return x < all ? (int)fg[(long)head * (nqb_arg * 4) + i] : 0x7fffffff;
    };
    int fn = word(lane);
    const uint16_t *Qg, *Gg;                             // head g's rows from the keys' own strip on, and its carries
    const float *cag, *cbg;
    auto at_head = [&]() __attribute__((always_inline)) {
        const long r0 = (kh.qrow0 + g * kh.qrow_step + k0) * D, c0 = kh.cbase + g * kh.cbase_step + ks * kh.cstride + k0;
        Qg = q + r0;
        Gg = dout + r0;
        cag = ca + c0;
        cbg = cb + c0;
    };
    at_head();
    auto next = [&](int& r) __attribute__((always_inline)) {
        while (todo == 0) {
            if (wn >= all) return false;
            todo = __builtin_amdgcn_ballot_w64(fn <= ks) & (EVERY << wave);
            w0 = wn;
            wn += 64;
            if (wn < all) fn = word(wn + lane);
        }
        const int x = w0 + __builtin_ctzll(todo);
        todo &= todo - 1;
        if (x - x0 >= nq) {
            do { x0 += nq; ++g; } while (x - x0 >= nq);
            at_head();
        }
        r = x - x0;
        return true;
    };
    const uint32_t base = lds_offset(smem) + wave * WAVE;
    int off[C::LOADS];
    subtile_offsets<D, false>(off, lane);
    float cn0 = 0.0f, cn1 = 0.0f, cn2 = 0.0f;
    auto fetch = [&](int r, int st) __attribute__((always_inline)) {
        const int rows = r == nq - 1 ? nlast : 32;
        const unsigned at = r * 32 + min(n, rows - 1);
        cn0 = cag[at];
        cn1 = cbg[at];
        if (strips_q) cn2 = (cag + (long)r * kh.cstride)[at];          // of the diagonal's subtile (blocks do not always leave one)
        stage_rows<D>(Qg + (long)r * 32 * D, rows, base + st * 2 * C::SUB, off, lane);
        stage_rows<D>(Gg + (long)r * 32 * D, rows, base + st * 2 * C::SUB + C::SUB, off, lane);
    };
    // K and V pass through the second buffer of the first wave
    const uint32_t k_at = lds_offset(smem) + 2 * C::SUB, v_at = k_at + C::SUB;
    stage_strip<D, NWS>(k + kh.base + (long)k0 * D, v + kh.base + (long)k0 * D, min(T - k0, 32), k_at, v_at, wave, lane);
    // Behind them, before it is known whether it reaches the keys, the first strip of the first two waves' shares: the two nearest
    // ones nearly always do, and where they are all there is they are what bounds the strip.
    const bool ahead = wave < 2 && wave < nq;
    if (ahead) fetch(wave, 0);
    if (PARTS && part == 0 && __builtin_expect(in_parts(beyond, ks), 0)) {    // (the first part's heads are the first of all)
        alone = false;
        G = parts.heads;
        all = G * nq;
        if (lane >= all) fn = 0x7fffffff;
    }
    int r = 0;
    bool more = next(r);
    if (more && !(ahead && g == 0 && r == wave)) {
        own_landed();                                    // nothing is still on its way into the buffer
        fetch(r, 0);
    }
    own_landed();
    barrier_nofence();
    bf16x8 kf[D / 16], vf[D / 16];                       // A operands: MFMA row n <- key perm_row(n)
    {
        const uint32_t at = tile_off_perm<D>(perm_row(n), hh);
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            kf[s] = __builtin_bit_cast(bf16x8, lds_load16((k_at + at) ^ (s << 5)));
            vf[s] = __builtin_bit_cast(bf16x8, lds_load16((v_at + at) ^ (s << 5)));
        }
    }
    barrier_lds();                                       // the buffer is free
    const uint32_t qb = base + tile_off_nat<D>(n, hh);                  // B operands, ^ (s << 5)
    uint32_t qtr[2];                                                    // transposing reads, ^ (b << 6)
#pragma unroll
    for (int t = 0; t < 2; ++t)
        qtr[t] = base + tile_off_nat<D>(8 * (gg >> 1) + (li >> 2) + 4 * t, 2 * (gg & 1) + ((li & 3) >> 1)) + 8 * (li & 1);
    // A and dZ on their way to the second products' operands: in the place of the subtiles they come from, whose operands
    // have all been asked for by then (a wave's LDS accesses stay in order)
    const uint32_t scr = base;
    const uint32_t sw_off = scr + scr_off(n, 2 * hh);
    uint32_t st_off[2];
#pragma unroll
    for (int t = 0; t < 2; ++t)
        st_off[t] = scr + scr_off(8 * (gg >> 1) + (li >> 2) + 4 * t, 2 * (gg & 1) + ((li & 3) >> 1)) + 8 * (li & 1);
    const float scale = 1.0f / sqrtf((float)D);
    const float c2 = SB_LOG2E * scale;
    f32x16 dkacc[D / 32], dvacc[D / 32];
#pragma unroll
    for (int b = 0; b < D / 32; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) { dkacc[b][r] = 0.0f; dvacc[b][r] = 0.0f; }

    for (int st = 0; more; st ^= 1) {
        own_landed();
        const float over = overshoot(cn2);
        float car = cn0 - over, cbl = cn1 * fast_exp2(over);
        asm volatile("" : "+v"(car), "+v"(cbl));
        const uint32_t buf = st * 2 * C::SUB;
        const bool diag = r == 0;
        if (r == nq - 1 && n >= nlast) {                 // rows past T: A, G and dZ are zero
            car = INFINITY;
            cbl = 0.0f;
        }
        if (diag && n == 0) car = cbl = 0.0f;            // as in bwd_dkv_kernel
        u32x4 qw[D / 16], gw[D / 16];
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            qw[s] = lds_load16((qb + buf) ^ (s << 5));
            gw[s] = lds_load16(((qb + buf) ^ (s << 5)) + C::SUB);
        }
        more = next(r);                                  // while the operands are on their way
        if (more) fetch(r, st ^ 1);
        f32x16 sacc, pacc;
#pragma unroll
        for (int r = 0; r < 16; ++r) { sacc[r] = 0.0f; pacc[r] = 0.0f; }
#pragma unroll
        for (int s = 0; s < D / 16; ++s) {
            sacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], __builtin_bit_cast(bf16x8, qw[s]), sacc, 0, 0, 0);
            pacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[s], __builtin_bit_cast(bf16x8, gw[s]), pacc, 0, 0, 0);
        }
        // the second products' operands land during the element-wise work
        bf16x8 gop[D / 16], qop[D / 16];
#pragma unroll
        for (int b = 0; b < D / 32; ++b)
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                const uint32_t x0 = ((qtr[0] + buf) ^ (b << 6)) + 16 * s2 * C::ROW, x1 = ((qtr[1] + buf) ^ (b << 6)) + 16 * s2 * C::ROW;
                gop[2 * b + s2] = tr_pair_at(x0 + C::SUB, x1 + C::SUB);
                qop[2 * b + s2] = tr_pair_at(x0, x1);
            }
        Chain ch;
        const bool fits = diag ? subtile_stage1<true>(ch, sacc, c2, n, hh) : subtile_stage1<false>(ch, sacc, c2, n, hh);
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!fits) != 0, 0)) {
            f32x16 again;
#pragma unroll
            for (int r = 0; r < 16; ++r) again[r] = 0.0f;
#pragma unroll
            for (int s = 0; s < D / 16; ++s)
                again = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[s], __builtin_bit_cast(bf16x8, lds_load16((qb + buf) ^ (s << 5))), again, 0, 0, 0);
            if (diag) subtile_stage1_log<true>(ch, again, c2, n, hh);
            else subtile_stage1_log<false>(ch, again, c2, n, hh);
        }
        SubtileOut so;
        subtile_stage2<false, true>(so, ch, pacc, car, cbl, hh);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        lds_store16(sw_off + buf, so.pa[0]);
        lds_store16((sw_off ^ 16) + buf, so.pa[1]);
        lds_store16(sw_off + buf + SCR_MAT, so.pz[0]);
        lds_store16((sw_off ^ 16) + buf + SCR_MAT, so.pz[1]);
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        bf16x8 at[2], zt[2];
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            const uint32_t x0 = st_off[0] + buf + 16 * s2 * 64, x1 = st_off[1] + buf + 16 * s2 * 64;
            at[s2] = tr_pair_at(x0, x1);
            zt[s2] = tr_pair_at(x0 + SCR_MAT, x1 + SCR_MAT);
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
#pragma unroll
        for (int b = 0; b < D / 32; ++b)
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2) {
                dvacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(at[s2], gop[2 * b + s2], dvacc[b], 0, 0, 0);
                dkacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(zt[s2], qop[2 * b + s2], dkacc[b], 0, 0, 0);
            }
    }

    // ---- the waves' shares added up, in a fixed order
    float* const red = reinterpret_cast<float*>(smem);   // [matrix][wave][32][D]
    static_assert(2 * NWS * 32 * D * 4 <= NWS * WAVE, "the partial gradients fit");
    barrier_lds();                                       // everyone is done with the tiles
#pragma unroll
    for (int b = 0; b < D / 32; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int at = (wave * 32 + 8 * (r >> 2) + 4 * hh + (r & 3)) * D + 32 * b + n;
            red[at] = dvacc[b][r];
            red[NWS * 32 * D + at] = dkacc[b][r];
        }
    barrier_lds();
    auto store = [&](float* to_dk, float* to_dv, auto shared) __attribute__((always_inline)) {
#pragma unroll
        for (int mat = 0; mat < 2; ++mat)
            for (int i = tid; i < 32 * D / 4; i += NTHR) {
                const int row = i / (D / 4), c = 4 * (i % (D / 4));
                f32x4 x = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
                for (int w = 0; w < NWS; ++w) x += *reinterpret_cast<const f32x4*>(&red[((mat * NWS + w) * 32 + row) * D + c]);
                if (k0 + row >= T) continue;
                float* const to = (mat == 0 ? to_dv : to_dk) + kh.base + (long)(k0 + row) * D + c;
                if constexpr (decltype(shared)::value) store_shared4(to, x);
                else *reinterpret_cast<f32x4*>(to) = mat == 0 ? x : x * scale;
            }
    };
    if (PARTS && __builtin_expect(!alone, 0)) {          // (see in_parts())
        const PartSums<D> sums(parts, sh.bh, cu ? H / G_arg : BH, cu ? Ttot : T_arg);
        store(sums.dk + part * sums.step, sums.dv + part * sums.step, bc<true>());
        add_parts<D, NTHR>(sums, parts.n, smem, kh.base + (long)k0 * D, kh.qhead0 / G_arg * nt32 + ks, min(T - k0, 32), dk, dv, scale, tid);
        return;
    }
    store(dk, dv, bc<false>());
}

// workspace layout: ca[BH][nt32][T], cb[BH][nt32][T] (fp32; [H][nt32][Ttot] for a packed
// batch), then the start strips of the queries' 32-row strips (16 bits): [BH][nqb][4], then the
// partial sums of the remainder-bias gradient (fp32): [BH][nchunk][D], [H][nchunk][D] for a packed batch; then, 16-byte aligned, where there is
// `room` for them, what Parts says.  B, T: batch size and
// length, or for a packed batch the number of sequences and the longest length.
template <int D, Packed PK>
hipError_t launch_one(const uint16_t* q, const uint16_t* k, const uint16_t* v, const uint16_t* rb,
                      const float* m, const uint16_t* dout, float* dq, float* dk, float* dv,
                      float* drb, float* workspace, int B, int H, int Hkv, int T, int passes, hipStream_t stream,
                      const int* cu, int Ttot, bool room)
{
    constexpr bool VL = PK != Packed::NO;
    const int BH = B * H;
    const int BHkv = B * Hkv;
    const int G = H / Hkv;
    const int nt32 = (T + 31) / 32;
    const int nqb = (T + BQ - 1) / BQ;
    const int nkb = (T + BKW - 1) / BKW;
    const int nkb64 = (T + 63) / 64;
    const long ncarry = VL ? (long)H * nt32 * Ttot : (long)BH * nt32 * T;
    float* ca = workspace;
    float* cb = ca + ncarry;
    uint16_t* first = reinterpret_cast<uint16_t*>(cb + ncarry);
    const uint32_t* first2 = reinterpret_cast<const uint32_t*>(first);     // of a tile's two strips
    float* part = reinterpret_cast<float*>(first + (long)BH * nqb * 4);
    const int entries = VL ? 1 : B;                      // of the bias's gradient
    const int nchunk = bias_chunks(B, T, VL, Ttot);
    Keys keys = keys_of(B, H, Hkv, T, D, VL, Ttot);
    Parts parts = {nullptr, 1, 0, 0, G};
    int* arrived = nullptr;
    if (room) {
        const KeyPlan plan = key_plan(B, H, Hkv, T, D, VL, Ttot);
        keys = plan.keys;
        parts.n = plan.parts;
        parts.heads = G / plan.parts;
        parts.beyond = plan.beyond;
        if (parts.n > 1) {
            const size_t base = VL ? bwd_varlen_workspace_bytes(B, H, Ttot, T, D) : bwd_workspace_bytes(B, H, T, D);
            parts.sums = reinterpret_cast<float*>(reinterpret_cast<char*>(workspace) + (base + 15) / 16 * 16);
            parts.blocks = (int)(keys == Keys::STRIPS ? pieces(B, Hkv, T, 32, VL, Ttot) : block_grid(B, Hkv, T, BKW, PK, Ttot));
            arrived = reinterpret_cast<int*>(parts.sums + 2 * parts.n * (VL ? (long)Hkv * Ttot : (long)BHkv * T) * D);
        }
    }
    const int NP = parts.n;
    const int mean = mean_T(B, T, VL, Ttot);
    const long gq = block_grid(B, H, T, BQ, PK, Ttot), gk64 = block_grid(B, Hkv, T, 64, PK, Ttot);
    const long gk = keys == Keys::PAIRS ? share_grid(BHkv, nkb, true) : block_grid(B, Hkv, T, BKW, PK, Ttot);
    const int shared = VL ? B : BHkv;                    // what the key-stationary kernels' BH counts
    const long strips_q = pieces(B, H, T, 32, VL, Ttot), strips_k = pieces(B, Hkv, T, 32, VL, Ttot);
    const int run_q = VL || G > 1 ? -1 : query_run(BH, nqb, D, true), run_k = VL || G > 1 ? -1 : share_run(BHkv, nkb);
    // checked before the first launch, so that an error leaves nothing enqueued
    // workgroups of the bias's gradient behind those of the passes
    const long bias_q = drb ? (long)nchunk * entries * H : 0, bias_k = drb ? H : 0;
    if (gq + bias_q > 0x7fffffffL || gk * NP + bias_k > 0x7fffffffL) return hipErrorInvalidValue;
    auto bias = [&](long work) { return BiasGrad{part, drb, (int)work, entries, H, nchunk}; };
    hipError_t e = hipSuccess;
#define SB_LAUNCH(WGS, THREADS, KERNEL, ...)                                                                    \
    {                                                                                                           \
    e = launch_workgroups(WGS, THREADS, [&](unsigned n, int first_wg) {                                         \
        hipLaunchKernelGGL(KERNEL, dim3(n), dim3(THREADS), 0, stream, __VA_ARGS__, first_wg);                   \
    });                                                                                                         \
    if (e != hipSuccess) return e;                                                                              \
    }
#define SB_DQ(RBV)                                                                                              \
    if (query_strips(B, H, T, D, VL, Ttot)) {                                                                   \
        auto go = [&](auto waves) {                                                                             \
            constexpr int NW = decltype(waves)::value;                                                          \
            hipLaunchKernelGGL((bwd_dq_small_kernel<D, RBV, NW>), dim3((unsigned)(strips_q + bias_q)), dim3(64 * NW), 0, stream, \
                               q, k, v, rb, m, dout, dq, ca, cb, first, T, VL ? H : BH, H, G, VL ? B : nt32, nqb, nt32, cu, Ttot, bias(strips_q), arrived); \
        };                                                                                                      \
        if (four_waves(strips_q, 1, mean, D)) go(std::integral_constant<int, 4>());                                      \
        else go(std::integral_constant<int, SmallCfg<D>::NWS>());                                               \
        if ((e = hipGetLastError()) != hipSuccess) return e;                                                    \
    } else SB_LAUNCH(gq + bias_q, NTHREADS, (bwd_dq_kernel<D, RBV, PK>),                                        \
              q, k, v, rb, m, dout, dq, ca, cb, first, T, VL ? B : BH, H, G, nqb, nt32, cu, Ttot, run_q, bias(gq), arrived)
// d = 128 takes the paired-wave kernel (two waves per SIMD instead of one); smaller head
// dimensions leave room for two workgroups of the one-wave-per-strip kernel per CU, which
// is faster there (measured).
#define SB_DKV(GQAV, DRV, PARTS)                                                                                       \
    if (keys == Keys::STRIPS) {                                                                                 \
        auto go = [&](auto waves) {                                                                             \
            constexpr int NW = decltype(waves)::value;                                                          \
            hipLaunchKernelGGL((bwd_dkv_small_kernel<D, DRV, NW, PARTS>), dim3((unsigned)(strips_k * NP + bias_k)), dim3(64 * NW), 0, stream, \
                               q, k, v, dout, ca, cb, dk, dv, first, T, VL ? Hkv : BHkv, H, G, VL ? B : nt32, nqb, nt32, cu, Ttot, \
                               query_strips(B, H, T, D, VL, Ttot), bias(strips_k * NP), parts);                             \
        };                                                                                                      \
        if (four_waves(strips_k, G, mean, D)) go(std::integral_constant<int, 4>());                                      \
        else go(std::integral_constant<int, SmallCfg<D>::NWS>());                                               \
        if ((e = hipGetLastError()) != hipSuccess) return e;                                                    \
    } else if constexpr (D == 128) {                                                                            \
        constexpr bool CAN = !VL && !GQAV;                                                                      \
        if (!PARTS && keys == Keys::KEYS_64)                                                                              \
            SB_LAUNCH(gk64 + bias_k, 256, (bwd_dkv_pair_kernel<D, 2, GQAV, PK, false, DRV, false>),                    \
                      q, k, v, dout, ca, cb, dk, dv, first2, T, shared, H, G, nkb64, nqb, nt32, cu, Ttot, bias(gk64), parts) \
        else if (CAN && keys == Keys::PAIRS)                                                                    \
            SB_LAUNCH(gk * NP + bias_k, 512, (bwd_dkv_pair_kernel<D, 4, GQAV, PK, CAN, DRV, false>),                        \
                      q, k, v, dout, ca, cb, dk, dv, first2, T, shared, H, G, nkb, nqb, nt32, cu, Ttot, bias(gk * NP), parts) \
        else                                                                                                    \
            SB_LAUNCH(gk * NP + bias_k, 512, (bwd_dkv_pair_kernel<D, 4, GQAV, PK, false, DRV, PARTS>),                      \
                      q, k, v, dout, ca, cb, dk, dv, first2, T, shared, H, G, nkb, nqb, nt32, cu, Ttot, bias(gk * NP), parts) \
    } else if (!PARTS && keys == Keys::TWO_GROUPS) {                                                                      \
        SB_LAUNCH(gk * NP + bias_k, 2 * NTHREADS, (bwd_dkv_kernel<D, GQAV, PK, 2, DRV, false>),                             \
                  q, k, v, dout, ca, cb, dk, dv, first2, T, shared, H, G, nkb, nt32, cu, Ttot, run_k, bias(gk * NP), parts); \
    } else {                                                                                                    \
        SB_LAUNCH(gk * NP + bias_k, NTHREADS, (bwd_dkv_kernel<D, GQAV, PK, 1, DRV, PARTS>),                                 \
                  q, k, v, dout, ca, cb, dk, dv, first2, T, shared, H, G, nkb, nt32, cu, Ttot, run_k, bias(gk * NP), parts); \
    }
    if (passes & 1) {
        if (rb) { SB_DQ(true); }
        else    { SB_DQ(false); }
    }
    if (passes & 2) {
        if (NP > 1) {
            if (drb) { SB_DKV(true, true, true) }
            else     { SB_DKV(true, false, true) }
        } else if (G > 1) {
            if (drb) { SB_DKV(true, true, false) }
            else     { SB_DKV(true, false, false) }
        } else {
            if (drb) { SB_DKV(false, true, false) }
            else     { SB_DKV(false, false, false) }
        }
    }
#undef SB_LAUNCH
#undef SB_DQ
#undef SB_DKV
    return e;
}

}  // namespace

size_t bwd_workspace_bytes(int B, int H, int T, int d)
{
    const size_t nt32 = (size_t)(T + 31) / 32;
    const size_t nblk = (size_t)(T + BQ - 1) / BQ;
    const size_t nchunk = (size_t)(T + DR_ROWS - 1) / DR_ROWS;
    return (2 * sizeof(float) * nt32 * T + 4 * sizeof(uint16_t) * nblk + sizeof(float) * nchunk * d) * (size_t)B * H;
}

// Behind the bytes of one part those of Parts, 16 in any case: what is larger than the other size has room for the plan that key_plan() makes
static size_t gqa_bytes(size_t base, size_t parts) { return (base + 15) / 16 * 16 + std::max<size_t>(16, parts); }

size_t bwd_gqa_workspace_bytes(int B, int H, int Hkv, int T, int d)
{
    const size_t base = bwd_workspace_bytes(B, H, T, d), heads = (size_t)B * Hkv;
    return H == Hkv ? base : gqa_bytes(base, part_bytes(key_plan(B, H, Hkv, T, d, false, 0).parts, heads * T, heads, T, d));
}

size_t bwd_varlen_gqa_workspace_bytes(int nseq, int H, int Hkv, int Ttot, int max_T, int d)
{
    const size_t base = bwd_varlen_workspace_bytes(nseq, H, Ttot, max_T, d);
    return H == Hkv ? base : gqa_bytes(base, part_bytes(key_plan(nseq, H, Hkv, max_T, d, true, Ttot).parts, (size_t)Hkv * Ttot, (size_t)nseq * Hkv, max_T, d));
}

size_t bwd_varlen_workspace_bytes(int nseq, int H, int Ttot, int max_T, int d)
{
    const size_t nt32 = (size_t)(max_T + 31) / 32;
    const size_t nblk = (size_t)(max_T + BQ - 1) / BQ;
    const size_t nchunk = (size_t)(max_T + DR_ROWS - 1) / DR_ROWS;
    return 2 * sizeof(float) * nt32 * (size_t)Ttot * H +
           (4 * sizeof(uint16_t) * nblk + sizeof(float) * nchunk * d) * (size_t)nseq * H;
}

hipError_t launch_bwd_bf16(const uint16_t* q, const uint16_t* k, const uint16_t* v, const uint16_t* rb,
                           const float* m, const uint16_t* dout, float* dq, float* dk, float* dv,
                           float* drb, float* workspace,
                           int B, int H, int Hkv, int T, int d, int passes, hipStream_t stream, bool room)
{
#define SB_BWD(DD) launch_one<DD, Packed::NO>(q, k, v, rb, m, dout, dq, dk, dv, drb, workspace, B, H, Hkv, T, passes, stream, nullptr, 0, room)
    if (d == 32) return SB_BWD(32);
    if (d == 64) return SB_BWD(64);
    return SB_BWD(128);
#undef SB_BWD
}

hipError_t launch_bwd_bf16_varlen(const uint16_t* q, const uint16_t* k, const uint16_t* v, const uint16_t* rb,
                                  const float* m, const uint16_t* dout, float* dq, float* dk, float* dv,
                                  float* drb, float* workspace, const int* cu, int nseq, int H, int Hkv,
                                  int Ttot, int max_T, int d, hipStream_t stream, bool room)
{
#define SB_BWD(DD, PK) launch_one<DD, PK>(q, k, v, rb, m, dout, dq, dk, dv, drb, workspace, nseq, H, Hkv, max_T, 3, stream, cu, Ttot, room)
    if (packed_as(nseq, max_T, Ttot) == Packed::ALIKE) {
        if (d == 32) return SB_BWD(32, Packed::ALIKE);
        if (d == 64) return SB_BWD(64, Packed::ALIKE);
        return SB_BWD(128, Packed::ALIKE);
    }
    if (d == 32) return SB_BWD(32, Packed::BY_LENGTH);
    if (d == 64) return SB_BWD(64, Packed::BY_LENGTH);
    return SB_BWD(128, Packed::BY_LENGTH);
#undef SB_BWD
}

}  // namespace sb
