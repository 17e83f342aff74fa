// bf16 forward of causal stick-breaking attention on the gfx950 matrix cores.
//
// Work split.  A query block is 128 rows of one (batch, head); each of the 4
// wavefronts of a workgroup owns 32 of them and keeps their Q fragments in
// registers.  Every workgroup one block, the longest first (share_of()).  Two
// workgroups share a CU at d = 128 (two wavefronts per SIMD), three at d = 64, four
// at d = 32.
//
// Keys are swept in 64-row tiles (two 32-row subtiles each) from the diagonal
// towards key 0, the order Algorithm 1 prescribes: the weight of key i needs the
// total of softplus(z) over the keys between i and the query (Eq. 2), so that total
// is carried per query row from subtile to subtile (the vector `a` of Algorithm 1).
// K and V tiles are brought into LDS by direct global->LDS loads, double buffered,
// one workgroup barrier per tile; tiles above the diagonal are never touched.
//
// Layout inside a wavefront.  Logits are formed transposed, S^T = K Q^T, with the
// 32x32x16 bf16 MFMA: A operand = 32 key rows from LDS, B operand = the wave's 32
// query rows.  In the accumulator a lane owns ONE query column (lane % 32) and 16
// key rows; the LDS row fed to MFMA row rho is perm_row(rho), which makes those 16
// keys consecutive (lanes 0-31: keys 0..15 of the subtile, lanes 32-63: keys
// 16..31).  The running product along the keys is then a serial chain inside the
// lane plus one exchange with the partner lane.  The weights feed the second MFMA
// (O += A V) straight from registers: the accumulator's per-lane key order is a
// valid K-dimension order for the A operand, and V is read from LDS with the
// transposing load in that same key order.
//
// Arithmetic between the two MFMAs (fp32): Eq. 1's product is evaluated in the
// linear domain inside a lane's 16 keys and in the log domain across lanes,
// subtiles and tiles.  With x = z*log2(e) and e_r = 2^{x_r} = beta_r / (1 - beta_r):
//     A[r] = beta_r * prod_{r' > r} (1 - beta_r') * 2^{-carry}
//          = e_r * prod_{r' < r} (1 + e_r') / prod_{all r'} (1 + e_r') * 2^{-carry},
// carry = sum over all nearer keys of log2(1 + e) (the base-2 softplus, i.e. Eq. 2's
// running sum).  That costs one exponential and four multiply/adds per weight; the
// log form of Eq. 2/3 needs three transcendentals.  Where the in-lane product could
// overflow, the wave falls back to the log form for that subtile (see ew()).
//
// Exhausted rows (the paper's "conditional computation", section 4.1): the carry of a row
// is -log2 of the stick it has left, and no weight of a farther key can exceed 2^-carry.
// From CARRY_EXHAUSTED = 160 on every farther weight IS zero in this arithmetic (the smallest
// nonzero bf16 is 2^-133, the smallest nonzero fp32 2^-149), so once every row of a query
// block is there, the rest of the sweep cannot change a bit of o (for finite inputs: a NaN in V
// would come through a zero weight, and does not where its tile is left out).  Without m the
// block stops; with m, which needs the softplus total over all keys, it goes on with the logits
// alone (no V, no A V: sum_tail()).  Rows whose weights reach far never get there and pay, every
// two tiles, a ballot, an LDS write per wave and a read of four flags behind the barrier.
// sb_attn_fwd_halt is the same kernel with the caller's threshold -log2(eps) in place of 160;
// its error is at most eps * max|v|.
#include <type_traits>

#include "sb_kernels.h"
#include "sb_mma.h"
#include "sb_share.h"

namespace sb {
namespace {

constexpr int NW = 4;                                   // wavefronts per workgroup
constexpr int BQ = 32 * NW;                             // query rows per block
constexpr int NS = 2;                                   // staging buffers (tiles in LDS)

template <int D> struct FwdCfg {
    static constexpr int ROW = D * 2;                   // bytes per tile row (unpadded, swizzled)
    static constexpr int TK = 64;                       // keys per staged tile
    static constexpr int KT_BYTES = TK * ROW;           // one K (or V) tile
    static constexpr int STAGE = 2 * KT_BYTES;          // K tile then V tile
    static constexpr int CPR = ROW / 16;                // 16 B chunks per row
    static constexpr int BLK_ROWS = 1024 / ROW;         // rows moved by one wave-wide 16 B/lane load
    static constexpr int NPW = KT_BYTES / 1024 / NW;    // such loads per wave per K (or V) tile
};

// workgroups that share a CU (waves per SIMD)
constexpr int wgs_per_cu(int d) { return d == 128 ? 2 : (d == 64 ? 3 : 4); }

template <bool B> using bc = std::integral_constant<bool, B>;
template <int I> using ic = std::integral_constant<int, I>;

// Element-wise path of one 32x32 subtile: logits -> weights (as MFMA operands).
// Inside the lane the chain  t_r = W_r e_r,  W_{r+1} = W_r + t_r  runs over the 16
// keys in ascending order, so W_r = W_0 prod_{r' < r} (1 + e_r') and the weight of
// key r is t_r / W_16 * 2^-(carry from all nearer keys).  log2(W_16 / W_0) is this
// lane's contribution to the carry.  W_0 = 2^-60 keeps the chain inside fp32 for
// in-lane products up to 2^140; weights below 2^-66 are flushed to zero.  If a chain
// still gets beyond 2^80 (sharp logits: softplus summing to more than 97 nats over
// 16 keys) or overflows, the wave redoes the subtile in the log form of Eq. 2 with
// the overflow-proof base-2 softplus.
// With MASK (the subtile on the diagonal) key 16hh + r is visible to query n iff
// 16hh + r < n.
// chain_of(): what needs no carry, handed to then(linear, g, t_lo, t_hi).  g: the t_r, or in the log form
// x - (sum of sp2 over this lane's keys from r on); t_lo, t_hi: both halves' softplus totals.
template <bool MASK, class F>
__device__ __forceinline__ void chain_of(const f32x16& sin, float c2, int n, int hh, F then)
{
    float g[16], t_lo, t_hi;
    float W = 0x1p-60f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        float e = fast_exp2(sin[r] * c2);
        if constexpr (MASK) e = (16 * hh + r < n) ? e : 0.0f;
        g[r] = W * e;
        W += g[r];
    }
    const bool bad = !(W < 0x1p80f);
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(bad) == 0, 1)) {
        both_halves(fast_log2(W) + 60.0f, t_lo, t_hi);   // log2 of the lane's prod (1 + e)
        then(bc<true>{}, g, t_lo, t_hi);
        return;
    }
    float run = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        g[r] = sin[r] * c2;
        if constexpr (MASK) g[r] = (16 * hh + r < n) ? g[r] : -INFINITY;
    }
#pragma unroll
    for (int r = 15; r >= 0; --r) {
        run += sp2(g[r]);
        g[r] -= run;
    }
    both_halves(run, t_lo, t_hi);
    then(bc<false>{}, g, t_lo, t_hi);
}
// keys 16..31 (hh = 1) are nearer to the query than keys 0..15
template <bool LINEAR>
__device__ __forceinline__ void weights_of(const float (&g)[16], float t_lo, float t_hi, float a, int hh, bf16x8 (&pout)[2])
{
    if constexpr (LINEAR) {
        const float kf = fast_exp2(60.0f - (a + t_hi + (hh == 0 ? t_lo : 0.0f)));
#pragma unroll
        for (int r = 0; r < 16; ++r) pout[r >> 3][r & 7] = (__bf16)(g[r] * kf);
    } else {
        const float off = a + (hh == 0 ? t_hi : 0.0f);
#pragma unroll
        for (int r = 0; r < 16; ++r) pout[r >> 3][r & 7] = (__bf16)fast_exp2(g[r] - off);
    }
}

// VL: packed variable-length batch.  The tensors are [H][Ttot][D] ([H/G][Ttot][D] for k, v),
// sequence s occupies rows cu[s] .. cu[s+1]-1, T_arg is at least the longest sequence's length and BH the number of sequences.
// TRI: measurement variant of the element-wise path.  The in-tile reverse cumulative sum of
// Algorithm 1 is taken on the matrix pipe, as a product with a triangular matrix of ones,
// instead of the in-lane chain (see ew_tri()); everything else is the same kernel.
template <int D, bool WRITE_M, bool RB, Packed VL, bool TRI = false>
__global__ void __launch_bounds__(64 * NW, wgs_per_cu(D))
fwd_bf16_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                const uint16_t* __restrict__ v, const uint16_t* __restrict__ rb,
                uint16_t* __restrict__ o, float* __restrict__ m,
                int T_arg, int BH, int H, int G, int nqb_arg, float enough,
                unsigned long long* __restrict__ tile_counts, const int* __restrict__ cu, int Ttot, int run, int first_wg)
{
    using C = FwdCfg<D>;
    constexpr int NPW = C::NPW;
    __shared__ __attribute__((aligned(1024))) char smem[NS * C::STAGE];
    __shared__ __attribute__((aligned(16))) int s_done[NW];         // per wave: all rows exhausted
    __shared__ __attribute__((aligned(16))) char s_tri[TRI ? 2 * 64 * 16 : 16];   // triangular operand, per lane

    // workgroup -> (head, query block).  What the first loads need is fetched together with it, not behind
    // the branches of share_of(): a short prompt is a chain of such latencies.
    asm volatile("" :: "s"(q), "s"(k), "s"(v), "s"(T_arg), "s"(G));
    const int wg = first_wg + blockIdx.x;
    Share sh;
    int T = T_arg, nqb = nqb_arg;
    long row0, kvrow0;                                  // first row of this head's q / k rows
    int head;
    if constexpr (VL != Packed::NO) {
        const Place at = block_of<BQ, VL == Packed::BY_LENGTH>(head, wg, H, G, cu, BH, Ttot, T_arg, threadIdx.x & 63);
        if (at.T == 0) return;
        sh.i = at.i;
        T = at.T;
        nqb = (T + BQ - 1) / BQ;
        row0 = (long)head * Ttot + at.c0;
        kvrow0 = (long)(head / G) * Ttot + at.c0;
    } else {
        // grouped kv heads: G consecutive query heads read the same K and V
        sh = in_scalars(share_of(wg, BH, run));
        const int bh = sh.bh;
        head = bh % H;
        row0 = bh * (long)T;
        kvrow0 = (long)(G == 1 ? bh : (int)((unsigned)bh / (unsigned)G)) * T;
    }

    // a sweep's instructions go before those of another block's sum_tail(): a sweep waits for memory and
    // for its own chain, the tail only for the pipes (1-2 % of a launch where heads are near)
    if constexpr (WRITE_M) __builtin_amdgcn_s_setprio(1);
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if constexpr (WRITE_M) {
        // measurement aid: with a non-null tile_counts the first workgroup leaves the shader
        // clock counter and the 100 MHz reference counter at its start ([0], [1]) and at its end
        // ([2], [3]); their ratio is the clock the chip sustained while this kernel ran
        if (tile_counts && wg == 0 && tid == 0) {
            tile_counts[0] = (unsigned long long)clock64();
            tile_counts[1] = (unsigned long long)wall_clock64();
        }
    }
    const int n = lane & 31;          // query column inside the wave
    const int hh = lane >> 5;         // half-wave: keys 16*hh .. 16*hh+15 of a subtile
    const int gg = lane >> 4, li = lane & 15;
    if constexpr (TRI) {
        // A operand of C^T = U L^T, U[key][key'] = 1 for key' >= key (keys of one 32-key subtile).
        // MFMA row rho stands for key perm_row(rho) (the accumulator layout of the logits), and
        // K-dim element 8h + e of MFMA s stands for key 16h + 8s + e (the order in which a lane
        // holds its 16 values).  Every wave writes the same words: benign.
        const int key_out = perm_row(n);
#pragma unroll
        for (int s = 0; s < 2; ++s) {
            bf16x8 u;
#pragma unroll
            for (int e = 0; e < 8; ++e) u[e] = (16 * hh + 8 * s + e >= key_out) ? (__bf16)1.0f : (__bf16)0.0f;
            *reinterpret_cast<bf16x8*>(s_tri + (s * 64 + lane) * 16) = u;
        }
        __syncthreads();
    }

    const uint16_t* Qg = q + row0 * D;
    // in scalar registers: the compiler keeps them in vector ones otherwise, which costs the unrolled
    // sweep 22 of its 964 vector instructions
    const uint16_t* Kg = reinterpret_cast<const uint16_t*>(scalar_base(k + kvrow0 * D));
    const uint16_t* Vg = reinterpret_cast<const uint16_t*>(scalar_base(v + kvrow0 * D));

    // ---- per-lane LDS byte addresses inside the first 32-row subtile of the first staging
    // buffer; every other subtile, matrix and buffer is a compile-time constant further on
    const uint32_t smem0 = lds_offset(smem);
    uint32_t aoff[D / 16];                  // K rows as A operand: row perm_row(n), chunk 2s + hh
    {
        const int key_l = perm_row(n);
#pragma unroll
        for (int s = 0; s < D / 16; ++s) aoff[s] = smem0 + tile_off_perm<D>(key_l, 2 * s + hh);
    }
    uint32_t vtr[D / 32][2];                // V through the transposing load: rows 16hh + li/4 (+4t, +8s)
    {
        const int row_l = 16 * (gg >> 1) + (li >> 2);
        const int cl = 2 * (gg & 1) + ((li & 3) >> 1);
#pragma unroll
        for (int b = 0; b < D / 32; ++b)
#pragma unroll
            for (int t = 0; t < 2; ++t)
                vtr[b][t] = smem0 + tile_off_perm<D>(row_l + 4 * t, 4 * b + cl) + 8 * (li & 1);
    }

    // ---- direct global -> LDS staging of one 64-row tile of K and of V.
    // One instruction moves 16 B per lane to 1 KB of consecutive LDS; the swizzle is
    // applied on the global side: the lane whose LDS position is (row, physical chunk)
    // fetches the logical chunk that belongs there.  Instruction i of this wave covers
    // tile rows (wave*NPW + i)*BLK_ROWS + lane/CPR.
    int goff[NPW];
#pragma unroll
    for (int i = 0; i < NPW; ++i) {
        const int row = (wave * NPW + i) * C::BLK_ROWS + lane / C::CPR;
        goff[i] = (row * D + (((lane % C::CPR) ^ swz_perm<D>(row)) << 3)) * 2;
    }
    auto stage_tile = [&](int jt, int st) __attribute__((always_inline)) {
        char* sp = smem + st * C::STAGE;
        const uint16_t* kb = Kg + (long)jt * C::TK * D;
        const uint16_t* vb = Vg + (long)jt * C::TK * D;
        if ((jt + 1) * C::TK <= T) {                    // all 64 rows exist
            dma16_to_lds_run(kb, goff, sp + wave * NPW * 1024);
            dma16_to_lds_run(vb, goff, sp + C::KT_BYTES + wave * NPW * 1024);
        } else {                                        // rows past T are clamped (causality masks them)
            const int row0 = wave * NPW * C::BLK_ROWS + lane / C::CPR, last = T - 1 - jt * C::TK;
            dma16_to_lds_run_clamped<C::ROW, C::BLK_ROWS>(kb, goff, row0, last, sp + wave * NPW * 1024);
            dma16_to_lds_run_clamped<C::ROW, C::BLK_ROWS>(vb, goff, row0, last, sp + C::KT_BYTES + wave * NPW * 1024);
        }
    };

    f32x16 oacc[D / 32];
    float a = 0.0f;                   // carry: sum of log2(1 + e) over all keys already swept (nearer keys)
    bf16x8 qf[D / 16];                // B operand of S^T = K Q^T: Q[q0 + n][16s + 8hh .. +7]
    const float c2 = SB_LOG2E / sqrtf((float)D);

    // operand fetches from LDS, kept apart from the MFMAs that use them so that they
    // can be issued a phase ahead
    // kslot / vslot: byte offset of the subtile's K / V rows from the start of the LDS tile
    // array; a compile-time constant in the unrolled sweep (it then rides in the instruction's
    // offset field), a runtime value in the diagonal band
    auto k_fetch = [&](uint32_t kslot, u32x4 (&kop)[D / 16]) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < D / 16; ++s) kop[s] = lds_load16(aoff[s] + kslot);
    };
    auto v_fetch = [&](uint32_t vslot, bf16x8 (&vop)[D / 16]) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < D / 32; ++b)
#pragma unroll
            for (int s = 0; s < 2; ++s) {
                const uint32_t pp = vslot + (8 * s) * C::ROW;
                vop[2 * b + s] = tr_pair_at(vtr[b][0] + pp, vtr[b][1] + pp);
            }
    };
    // S^T = K Q^T
    auto s_mfma = [&](const u32x4 (&kop)[D / 16]) __attribute__((always_inline)) {
        f32x16 acc;
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
        for (int s = 0; s < D / 16; ++s)
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kop[s]), qf[s], acc, 0, 0, 0);
        return acc;
    };
    // O[q][dcol] += sum_keys A[q][key] V[key][dcol]; K-dim index 8h+e <-> key 16h + 8s + e
    auto pv_mfma = [&](const bf16x8 (&vop)[D / 16], const bf16x8 (&p)[2]) __attribute__((always_inline)) {
#pragma unroll
        for (int b = 0; b < D / 32; ++b)
#pragma unroll
            for (int s = 0; s < 2; ++s)
                oacc[b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[s], vop[2 * b + s], oacc[b], 0, 0, 0);
    };

    auto ew = [&](auto mask_c, const f32x16& sin, bf16x8 (&pout)[2]) __attribute__((always_inline)) {
        chain_of<decltype(mask_c)::value>(sin, c2, n, hh, [&](auto linear, const float (&g)[16], float t_lo, float t_hi) __attribute__((always_inline)) {
            weights_of<decltype(linear)::value>(g, t_lo, t_hi, a, hh, pout);
            a += t_lo + t_hi;
        });
    };

    // The same step in the log form of Eq. 2 with Algorithm 1's in-tile cumulative sum on the
    // matrix pipe (unmasked subtiles only).  L = sp2(x) per element (two transcendentals); the
    // inclusive sums over the keys from a lane's own key to the subtile's last key, both
    // half-waves at once, are C^T = U L^T with L split into a bf16 head and a bf16 remainder
    // (one bf16 alone would leave 2^-9 of up to 32 summands in the exponent): four MFMAs.  The
    // weight is 2^(x - C - carry), a third transcendental.
    auto ew_tri = [&](const f32x16& sin, bf16x8 (&pout)[2]) __attribute__((always_inline)) {
        float y[16];
        bf16x8 lh[2], ll[2];
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            y[r] = sin[r] * c2;
            const float L = sp2(y[r]);
            const __bf16 h = (__bf16)L;
            lh[r >> 3][r & 7] = h;
            ll[r >> 3][r & 7] = (__bf16)(L - (float)h);
        }
        const bf16x8 u0 = *reinterpret_cast<const bf16x8*>(s_tri + lane * 16);
        const bf16x8 u1 = *reinterpret_cast<const bf16x8*>(s_tri + (64 + lane) * 16);
        f32x16 c;
#pragma unroll
        for (int r = 0; r < 16; ++r) c[r] = 0.0f;
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u0, lh[0], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u1, lh[1], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u0, ll[0], c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(u1, ll[1], c, 0, 0, 0);
        float t_lo, t_hi;
        both_halves(c[0], t_lo, t_hi);                 // key 0's sum (lanes 0-31) is the subtile's total
#pragma unroll
        for (int r = 0; r < 16; ++r) pout[r >> 3][r & 7] = (__bf16)fast_exp2((y[r] - c[r]) - a);
        a += t_lo;
    };

    // one 32-key subtile, start to end (tiles that touch the diagonal band)
    auto subtile = [&](auto mask_c, uint32_t stage_off, int sub) __attribute__((always_inline)) {
        const uint32_t kslot = stage_off + sub * 32 * C::ROW;
        const uint32_t vslot = stage_off + C::KT_BYTES + sub * 32 * C::ROW;
        u32x4 kop[D / 16];
        bf16x8 vop[D / 16];
        k_fetch(kslot, kop);
        const f32x16 s = s_mfma(kop);
        v_fetch(vslot, vop);
        bf16x8 p[2];
        ew(mask_c, s, p);
        pv_mfma(vop, p);
    };
    // a full tile, upper subtile first, written so that the operand fetches of a phase
    // can be issued during the phase before it; kop: the K rows of the upper subtile, fetched by first_k()
    auto first_k = [&](uint32_t sp, u32x4 (&kop)[D / 16]) __attribute__((always_inline)) { k_fetch(sp + 32 * C::ROW, kop); };
    auto hot_tile = [&](uint32_t sp, u32x4 (&kop)[D / 16]) __attribute__((always_inline)) {
        bf16x8 vop[D / 16];
        bf16x8 p[2];
        f32x16 s = s_mfma(kop);
        v_fetch(sp + C::KT_BYTES + 32 * C::ROW, vop);
        if constexpr (TRI) ew_tri(s, p); else ew(bc<false>{}, s, p);
        k_fetch(sp, kop);
        pv_mfma(vop, p);
        s = s_mfma(kop);
        v_fetch(sp + C::KT_BYTES, vop);
        if constexpr (TRI) ew_tri(s, p); else ew(bc<false>{}, s, p);
        pv_mfma(vop, p);
    };

    const int Q0 = (nqb - 1 - sh.i) * BQ;
    const int q0 = Q0 + wave * 32;                   // this wave's first query row
    const bool wave_live = q0 < T;
    // The rest of a sweep whose weights are all zero, for m alone: adds log2(1 + e) over the keys of
    // tiles 0 .. ntail-1 to the carry.  Two K tiles fill a staging buffer (V is not needed), so a
    // barrier covers 128 keys.  The accumulators of the output are free by now: a wave takes one of
    // the two subtiles of every tile for its own rows and for those of its neighbour (wave ^ 1), which
    // halves the LDS reads of a product, and the exponentials of a subtile stand beside the products of
    // the next one in one block of code.  Bound by the matrix pipe and its power at d = 128 (1.1 PFLOP/s of
    // products at T = 16384, what a library GEMM reaches on this data is 1.2), by the three vector
    // instructions a logit below.  Against a wave's own rows alone, product and exponentials in turn, all
    // heads near, the whole forward, us: B8 H16 T4096 d128 409 -> 378, B1 H32 T16384 d128 1279 -> 1130, one
    // block's chain B1 H16 T4096 d128 73 -> 57, B1 H24 T16384 d64 565 -> 537, B8 H16 T2048 d64 76.6 -> 75.8.
    auto sum_tail = [&](int ntail) __attribute__((always_inline)) {
        __builtin_amdgcn_s_setprio(0);
        const uint32_t khalf = (wave & 1) * 32 * C::ROW;     // the wave's subtile of a tile
        const int npr = (ntail + 1) >> 1;
        auto stage_pair = [&](int i, int st) __attribute__((always_inline)) {
            char* sp = smem + st * C::STAGE;
#pragma unroll
            for (int x = 0; x < 2; ++x) {
                const uint16_t* kb = Kg + (long)min(2 * i + x, ntail - 1) * C::TK * D;
                dma16_to_lds_run(kb, goff, sp + x * C::KT_BYTES + wave * NPW * 1024);
            }
        };
        dma_wait<0>();
        barrier_lds();                                       // nobody reads the sweep's tiles any more
        stage_pair(0, 0);
        // the neighbour's rows, through the other buffer (read again from memory they cost a fifth of the
        // traffic of a block whose weights end early)
        static_assert(NW * (D / 16) * 1024 <= C::STAGE, "the rows of all waves fit a buffer");
        bf16x8 qn[D / 16];
        const uint32_t qswap = smem0 + C::STAGE + lane * 16;
#pragma unroll
        for (int s = 0; s < D / 16; ++s) lds_store16(qswap + (wave * (D / 16) + s) * 1024, qf[s]);
        barrier_lds();
#pragma unroll
        for (int s = 0; s < D / 16; ++s)
            qn[s] = __builtin_bit_cast(bf16x8, lds_load16(qswap + ((wave ^ 1) * (D / 16) + s) * 1024));
        float l = 0.0f, ln = 0.0f;                           // this lane's keys only: the halves are added at the end
        struct Logits { f32x16 own, nbr; };
        // logits of the subtile in `slot`, beside the totals of the one before
        auto logits = [&](uint32_t slot, Logits& x) __attribute__((always_inline)) {
            u32x4 kop[D / 16];
            k_fetch(khalf + slot, kop);
#pragma unroll
            for (int r = 0; r < 16; ++r) { x.own[r] = 0.0f; x.nbr[r] = 0.0f; }
#pragma unroll
            for (int s = 0; s < D / 16; ++s) {
                x.own = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kop[s]), qf[s], x.own, 0, 0, 0);
                x.nbr = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kop[s]), qn[s], x.nbr, 0, 0, 0);
            }
        };
        auto add = [&](const Logits& x) __attribute__((always_inline)) { sp2_total_of_two(x.own, x.nbr, c2, l, ln); };
        Logits x0, x1;
#pragma unroll
        for (int r = 0; r < 16; ++r) { x1.own[r] = -INFINITY; x1.nbr[r] = -INFINITY; }     // adds nothing
        auto pair_tile = [&](int i, auto buf_c) __attribute__((always_inline)) {
            constexpr int BUF = decltype(buf_c)::value;
            constexpr uint32_t sp = BUF * C::STAGE;
            dma_wait<0>();
            barrier_lds();
            if (i + 1 < npr) stage_pair(i + 1, BUF ^ 1);
            logits(sp, x0);
            add(x1);
            logits(sp + C::KT_BYTES, x1);
            add(x0);
        };
        for (int i = 0; i < npr; i += 2) {
            pair_tile(i, ic<0>{});
            if (i + 1 < npr) pair_tile(i + 1, ic<1>{});
        }
        if (!(ntail & 1)) add(x1);                           // else the last tile was staged twice
        // (the lane index once more, so that it is not kept across the loop: d = 32 has no register to spare)
        const int at = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        const int n = at & 31, hh = at >> 5;
        float lo, hi;
        both_halves(ln, lo, hi);
        barrier_lds();                                       // the tiles have been read
        float* const swap = reinterpret_cast<float*>(smem);
        if (hh == 0) swap[(wave ^ 1) * 32 + n] = lo + hi;
        barrier_lds();
        both_halves(l, lo, hi);
        a += (lo + hi) + swap[wave * 32 + n];
    };

    const int kmax = min(T, Q0 + BQ) - 1;                // keys 0 .. kmax-1 are visible to some row
    const int ntile = (kmax + C::TK - 1) / C::TK;
    const int ndiag = min(ntile, ntile - Q0 / C::TK);    // leading tiles that touch the diagonal band
    // iteration `it` handles tile ntile-1-it, staged in buffer it % NS.  The first tile and Q are
    // fetched together: one memory latency in front of a block, not two.
    if (ntile > 0) stage_tile(ntile - 1, 0);
    {
        const int jq = min(q0 + n, T - 1);
        const u32x4* src = reinterpret_cast<const u32x4*>(Qg + (long)jq * D + 8 * hh);
#pragma unroll
        for (int s = 0; s < D / 16; ++s) qf[s] = __builtin_bit_cast(bf16x8, src[2 * s]);
    }
    // Wait for the Q loads here, once: the staging
    // loads are issued behind the compiler's back, and a wait for "all my
    // loads" placed inside the loop would also wait for those.
#pragma unroll
    for (int s = 0; s < D / 16; ++s) asm volatile("" :: "v"(qf[s]));
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
    for (int b = 0; b < D / 32; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[b][r] = 0.0f;
    a = 0.0f;

    // ---- the sweep over 64-key tiles, from the diagonal down to key 0
    auto begin_iter = [&](int it) __attribute__((always_inline)) {
        dma_wait<0>();                                   // this wave's share of tile `it` has landed
        // ... everyone's has, and tile it-1 is no longer read.  The waves' exhaustion flags go
        // through LDS here: their writes must have completed first, or the waves of a
        // workgroup could disagree about leaving the loop.
        barrier_lds();
        if (it + 1 < ntile) stage_tile(ntile - 2 - it, (it + 1) % NS);
        return (uint32_t)((it % NS) * C::STAGE);
    };
    int it = 0;
    for (; it < ndiag; ++it) {                           // tiles that touch the diagonal band
        const uint32_t sp = begin_iter(it);
        const int jt = ntile - 1 - it;
        if (wave_live) {
#pragma unroll
            for (int sub = 1; sub >= 0; --sub) {
                const int k0 = jt * C::TK + 32 * sub;    // subtiles and wave rows are both 32-aligned
                if (k0 == q0) subtile(bc<true>{}, sp, sub);
                else if (k0 < q0) subtile(bc<false>{}, sp, sub);
            }
        }
    }
    // A wave leaves in s_done whether all its rows are exhausted (both half-waves hold the same carry;
    // rows past T repeat row T-1).  The flags are read after the next barrier, by all waves alike, and
    // written again only after the one behind that.
    auto publish = [&]() __attribute__((always_inline)) {
        if (!TRI && lane == 0) s_done[wave] = !wave_live || __builtin_amdgcn_ballot_w64(!(a >= enough)) == 0;
    };
    // Tiles fully visible to every row.  The first row of a block has no key in the diagonal band, so the
    // tile behind the band is the first after which a block can stop, and a halting one usually does.
    // From there on two tiles per trip with the staging buffer a compile-time constant, so that every LDS
    // read of the sweep is a precomputed register plus an immediate: no address arithmetic in the
    // loop.  The barrier in front of a trip is taken at the end of the one before, where the flags
    // decide whether there is another: the loop has this one exit.  (With a second one in its middle the
    // compiler copies the accumulators, which spills.  The band is two tiles, or one or none in a ragged
    // last block.)
    // The K rows of the next tile are asked for together with the flags: their latency is one.
    // Against flags read in the middle of a trip and acted on at its end, us: B8 H16 T4096 d128 near heads
    // 168 -> 149, with halt 134 -> 122; B1 H24 T16384 d64 66 -> 55, 52 -> 42; one block's chain, all far,
    // B1 H9 T4096 d128 89 -> 87, B2 H5 T3490 d64 52.1 -> 52.7 (with the runs of sb_share.h in the first two).
    static_assert(NS == 2, "the unrolled sweep alternates two buffers");
    int stop = 0;
    u32x4 kop[D / 16];
    const bool lead = !(it & 1) && it < ntile;
    if (lead) {
        begin_iter(it);
        first_k(0u, kop);
        hot_tile(0u, kop);
        ++it;
        publish();
    }
    if (it < ntile) {
        begin_iter(it);
        if (!TRI && lead) stop = waves_done(s_done);
        first_k((uint32_t)C::STAGE, kop);
    }
    while (it + 1 < ntile && !stop) {
        hot_tile((uint32_t)C::STAGE, kop);
        begin_iter(it + 1);
        first_k(0u, kop);
        hot_tile(0u, kop);
        it += 2;
        publish();
        begin_iter(it);
        if (!TRI) stop = waves_done(s_done);
        first_k((uint32_t)C::STAGE, kop);                    // past the last tile: read and not used
    }
    if (it < ntile && !stop) { hot_tile((uint32_t)C::STAGE, kop); ++it; }
    if constexpr (!WRITE_M) {
        if (tile_counts && tid == 0) {
            atomicAdd(&tile_counts[0], (unsigned long long)it);        // tiles swept
            atomicAdd(&tile_counts[1], (unsigned long long)ntile);     // tiles of the full sweep
        }
    }
    dma_wait<0>();                                       // a tile staged before the sweep stopped

    // ---- store.  oacc[b][r] is query row 8*(r/4) + 4*hh + r%4, column 32b + n.
    if (wave_live) {
        if constexpr (RB) {
            // remainder bias (Appendix C): o_j += (stick left of row j) * r_head.  The
            // lanes n of both half-waves hold the carry of row q0 + n.
            const float rem = fast_exp2(-a);
            const uint16_t* rh = rb + head * D;
            float rc[D / 32];
#pragma unroll
            for (int b = 0; b < D / 32; ++b)
                rc[b] = __builtin_bit_cast(float, (uint32_t)rh[32 * b + n] << 16);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float rr = __shfl(rem, 8 * (r >> 2) + 4 * hh + (r & 3));
#pragma unroll
                for (int b = 0; b < D / 32; ++b) oacc[b][r] += rr * rc[b];
            }
        }
        uint16_t* const Og = reinterpret_cast<uint16_t*>(scalar_base(o + (row0 + q0) * D));
        if (q0 + 32 <= T) {
            // whole strips: without a test per element, and two columns a store.  A lane holds one column
            // of rows r and r + 1; with its neighbour's it makes two columns of row r (n even) or r + 1.
            const uint32_t pick = (n & 1) ? 0x03020706u : 0x05040100u;
            const int at = (4 * hh + (n & 1)) * D + (n & ~1);
#pragma unroll
            for (int r = 0; r < 16; r += 2)
#pragma unroll
                for (int b = 0; b < D / 32; ++b) {
                    typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
                    const bf16x2 two = {(__bf16)oacc[b][r], (__bf16)oacc[b][r + 1]};
                    const uint32_t x = __builtin_bit_cast(uint32_t, two);
                    const uint32_t y = __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true);      // of lane n ^ 1
                    *reinterpret_cast<uint32_t*>(Og + (8 * (r >> 2) + (r & 3)) * D + 32 * b + at) = __builtin_amdgcn_perm(y, x, pick);
                }
        } else {
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int row = 8 * (r >> 2) + 4 * hh + (r & 3);
                if (q0 + row < T)
#pragma unroll
                    for (int b = 0; b < D / 32; ++b) {
                        const __bf16 val = (__bf16)oacc[b][r];
                        Og[row * D + 32 * b + n] = __builtin_bit_cast(uint16_t, val);
                    }
            }
        }
    }
    if constexpr (WRITE_M) {
        if (it < ntile) sum_tail(ntile - it);
        const int at = __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
        if (wave_live && at < 32 && q0 + at < T) m[row0 + q0 + at] = -a * SB_LN2;
    }
    if constexpr (WRITE_M) {
        if (tile_counts && wg == 0 && tid == 0) {
            tile_counts[2] = (unsigned long long)clock64();
            tile_counts[3] = (unsigned long long)wall_clock64();
        }
    }
}

// ------------------------------------------------------------------ small grids
// Where the 128-row blocks leave most of the chip idle, what counts is the length of one row's chain of
// subtiles.  Here a workgroup takes one strip of 32 query rows, and its waves take the strip's subtiles from
// the diagonal on in rounds of one each: logits and chains, which need no carry, side by side; one barrier
// for the carries; weights, into LDS; one barrier; then O += A V, over the round's subtiles in order, by waves
// of their own, one per 32 columns, beside the logits and chains of the next round.  Every sum is taken in the order of
// fwd_bf16_kernel: o is the same, bit for bit (m too, unless the rows are exhausted on the way).  Which grids: small_fwd_grid().
// Against O += A V by the first of the waves between two rounds, and Q read by all of them, all heads far, then none, us: B2 H4 T777 d32
// 8.4 -> 7.3, 6.0 -> 5.2; B1 H4 T4000 d64 36 -> 30, 18.7 -> 16.1; B1 H8 T700 d128 13.0 -> 10.9, 10.1 -> 8.3; B1 H16 T100 d64 5.0 -> 4.5.
template <int D, int NWS> struct FwdSmallCfg {          // NWS: waves that take subtiles
    static constexpr int NWO = D / 32;                  // and waves that take O += A V
    static constexpr int NTHR = 64 * (NWS + NWO);
    static constexpr int ROW = D * 2;
    static constexpr int SUB = 32 * ROW;                // one 32-row subtile of K (or V)
    static constexpr int LOADS = SUB / 1024;            // of 16 bytes a lane, for a subtile
    static constexpr int Q_OFF = 3 * SUB;               // Q passes through a buffer of V that the second round is the first to fill
    static constexpr int W_OFF = NWS * 4 * SUB;         // after the waves' K and V, double buffered: weights
    static constexpr int W_SUB = 2 * 1024;              // of a subtile: two operands of 16 bytes a lane
};

// 32 columns of a strip of `rows` rows, to `out` (wave-uniform): oacc[r] is row 8*(r/4) + 4*hh + r%4, column n.  Two columns a store, as in fwd_bf16_kernel
template <int D>
__device__ __forceinline__ void store_strip_rows(uint16_t* out, const f32x16& oacc, int rows, int n, int hh)
{
    const uint32_t pick = (n & 1) ? 0x03020706u : 0x05040100u;
    const int at = (4 * hh + (n & 1)) * D + (n & ~1);
    auto store = [&](auto whole) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
            const bf16x2 two = {(__bf16)oacc[r], (__bf16)oacc[r + 1]};
            const uint32_t x = __builtin_bit_cast(uint32_t, two);
            const uint32_t y = __builtin_amdgcn_mov_dpp(x, 0xB1, 0xF, 0xF, true);      // of lane n ^ 1
            const int row = 8 * (r >> 2) + (r & 3);
            if (decltype(whole)::value || row + 4 * hh + (n & 1) < rows)
                *reinterpret_cast<uint32_t*>(out + row * D + at) = __builtin_amdgcn_perm(y, x, pick);
        }
    };
    if (rows == 32) store(bc<true>{});
    else store(bc<false>{});
}

template <int D, int NWS>
__global__ void __launch_bounds__((FwdSmallCfg<D, NWS>::NTHR))
fwd_small_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
                 const uint16_t* __restrict__ v, const uint16_t* __restrict__ rb,
                 uint16_t* __restrict__ o, float* __restrict__ m,
                 int T_arg, int BH, int H, int G, int n_arg, float enough,       // n_arg: strips a head; packed batch: sequences
                 unsigned long long* __restrict__ clocks, const int* __restrict__ cu, int Ttot)
{
    using C = FwdSmallCfg<D, NWS>;
    __shared__ __attribute__((aligned(1024))) char smem[C::W_OFF + NWS * C::W_SUB];
    __shared__ float s_tot[2][NWS][32];                 // per round parity: softplus totals of its subtiles (base 2), per row

    asm volatile("" :: "s"(q), "s"(k), "s"(v), "s"(T_arg), "s"(G));
    const int tid = threadIdx.x, lane = tid & 63;
    const Share sh = in_scalars(share_of(blockIdx.x, BH, -1));
    const int bh = sh.bh, head = bh % H;
    int T = T_arg, nstrip = n_arg, i = sh.i;
    long row0 = bh * (long)T, kvrow0 = (long)(G == 1 ? bh : (int)((unsigned)bh / (unsigned)G)) * T;
    if (cu) {                                           // packed batch: bh is the head alone, sh.i its place
        const Place at = place_of<32>(sh.i, cu, n_arg, Ttot, T_arg, lane);
        if (at.T == 0) return;
        T = at.T;
        nstrip = (T + 31) / 32;
        i = at.i;
        row0 = (long)head * Ttot + at.c0;
        kvrow0 = (long)(head / G) * Ttot + at.c0;
    }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool sums = wave >= NWS;                      // one of the waves that take O += A V
    const int cols = wave - NWS;                        // its columns, 32 cols ..
    const bool clock = clocks && blockIdx.x == 0 && tid == 0;
    if (clock) {                                        // as in fwd_bf16_kernel
        clocks[0] = (unsigned long long)clock64();
        clocks[1] = (unsigned long long)wall_clock64();
    }
    const int n = lane & 31, hh = lane >> 5, gg = lane >> 4, li = lane & 15;
    const int strip = nstrip - 1 - i;
    const int q0 = strip * 32;
    const int nlast = min(T - q0, 32);                  // rows of the strip, and of the subtile on the diagonal
    const uint16_t* Kg = reinterpret_cast<const uint16_t*>(scalar_base(k + kvrow0 * D));
    const uint16_t* Vg = reinterpret_cast<const uint16_t*>(scalar_base(v + kvrow0 * D));
    const uint32_t smem0 = lds_offset(smem);

    // a wave's buffers: K, K, V, V
    const uint32_t mine = smem0 + wave * 4 * C::SUB;
    constexpr int CPR = C::ROW / 16;
    int off[C::LOADS];
#pragma unroll
    for (int i = 0; i < C::LOADS; ++i) off[i] = tile_off_perm<D>(i * (1024 / C::ROW) + lane / CPR, lane % CPR);
    auto stage = [&](const uint16_t* X, int sub, uint32_t dst) __attribute__((always_inline)) {
        const uint64_t xb = scalar_base(X + (long)sub * 32 * D);
        if (sub < strip || nlast == 32) {
            dma16_to_lds_run_at(xb, off, dst);
        } else {                                        // rows past T are clamped (causality masks them)
            int o[C::LOADS];
#pragma unroll
            for (int i = 0; i < C::LOADS; ++i) o[i] = off[i] - max(i * (1024 / C::ROW) + lane / CPR - (nlast - 1), 0) * C::ROW;
            dma16_to_lds_run_at(xb, o, dst);
        }
    };
    // Q by whole rows and once, every wave its share.  (As operands from
    // memory, 32 bytes of 32 rows an instruction, all of it by every wave: 1700, 2200 and 4500 clocks at d = 32, 64 and 128.)
    for (int i = wave; i < C::LOADS; i += C::NTHR / 64) {
        const int row = i * (1024 / C::ROW) + lane / CPR;
        dma16_to_lds_at(scalar_base(q + (row0 + q0) * D), min(row, nlast - 1) * C::ROW + (((lane % CPR) ^ swz_perm<D>(row)) << 4),
                        smem0 + C::Q_OFF + i * 1024);
    }
    if (!sums && strip - wave >= 0) {
        stage(Kg, strip - wave, mine);
        stage(Vg, strip - wave, mine + 2 * C::SUB);
        dma_wait<C::LOADS>();                           // all but V
    } else {
        dma_wait<0>();
    }
    barrier_nofence();
    const float c2 = SB_LOG2E / sqrtf((float)D);
    f32x16 oacc;                                        // columns 32 cols ..
    float a = 0.0f;                                     // carry of the round
    bool done = false;                                  // every row exhausted: the weights are zero from here on
    int st = 0, top = strip;
    auto totals = [&](float (&t)[NWS]) __attribute__((always_inline)) {
#pragma unroll
        for (int w = 0; w < NWS; ++w) t[w] = s_tot[st][w][n];
    };
    auto ended = [&]() __attribute__((always_inline)) {          // alike in all waves
        done = __builtin_amdgcn_ballot_w64(!(a >= enough)) == 0;
        return done || top < NWS;
    };
    // Both kinds of waves pass the same barriers.
    if (sums) {
        uint32_t vtr[2];                                // V of wave 0, this wave's columns, through the transposing load
#pragma unroll
        for (int t = 0; t < 2; ++t)
            vtr[t] = smem0 + 2 * C::SUB + tile_off_perm<D>(16 * (gg >> 1) + (li >> 2) + 4 * t, 4 * cols + 2 * (gg & 1) + ((li & 3) >> 1)) + 8 * (li & 1);
        const uint32_t wts = smem0 + C::W_OFF + lane * 16;
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[r] = 0.0f;
        // operands of a round's subtiles, all asked for before the first product
        bf16x8 p[2 * NWS], x[2 * NWS];
        auto ask = [&](int st, int count) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 2 * NWS; ++i) {
                const int w = min(i >> 1, count - 1), s = i & 1;
                const uint32_t vs = w * 4 * C::SUB + st * C::SUB + 8 * s * C::ROW;
                p[i] = __builtin_bit_cast(bf16x8, lds_load16(wts + w * C::W_SUB + s * 1024));
                x[i] = tr_pair_at(vtr[0] + vs, vtr[1] + vs);
            }
            __builtin_amdgcn_sched_barrier(0);
        };
        auto multiply = [&](int from, int to) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < 2 * NWS; ++i)
                if (i >= from && i < to) oacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[i], x[i], oacc, 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        };
        for (;; top -= NWS, st ^= 1) {
            if (top != strip) {                         // the round before: half of it beside the logits of this one
                ask(st ^ 1, NWS);
                multiply(0, NWS);
            }
            barrier_lds();
            if (top != strip) multiply(NWS, 2 * NWS);
            float t[NWS];
            totals(t);
#pragma unroll
            for (int w = 0; w < NWS; ++w) a += t[w];
            barrier_lds();
            if (ended()) break;
        }
        const int count = min(NWS, top + 1);            // the last round
        ask(st, count);
        multiply(0, 2 * count);
        if (m && done) barrier_lds();
    } else {
        bf16x8 qf[D / 16];
        {
            const uint32_t at = smem0 + C::Q_OFF + tile_off_perm<D>(n, hh);
#pragma unroll
            for (int s = 0; s < D / 16; ++s) qf[s] = __builtin_bit_cast(bf16x8, lds_load16(at ^ (s << 5)));
        }
        const uint32_t ka = mine + tile_off_perm<D>(perm_row(n), hh);               // K as A operand, ^ (s << 5)
        const uint32_t wts = smem0 + C::W_OFF + wave * C::W_SUB + lane * 16;
        auto logits = [&](int st) __attribute__((always_inline)) {
            u32x4 kop[D / 16];
#pragma unroll
            for (int s = 0; s < D / 16; ++s) kop[s] = lds_load16((ka + st * C::SUB) ^ (s << 5));
            f32x16 acc;
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
            for (int s = 0; s < D / 16; ++s)
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kop[s]), qf[s], acc, 0, 0, 0);
            return acc;
        };
        for (;; top -= NWS, st ^= 1) {
            const int sub = top - wave;
            float g[16], t_lo = 0.0f, t_hi = 0.0f;
            bool linear = true;
            if (sub >= 0) {
                // this subtile's K has landed, V was asked for behind it; the K buffer to be refilled was read a round ago, by this wave
                asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" :: "n"(C::LOADS) : "memory");
                if (sub - NWS >= 0) stage(Kg, sub - NWS, mine + (st ^ 1) * C::SUB);
                const f32x16 acc = logits(st);
                auto keep = [&](auto lin, const float (&x)[16], float x_lo, float x_hi) __attribute__((always_inline)) {
                    linear = decltype(lin)::value;
                    t_lo = x_lo;
                    t_hi = x_hi;
#pragma unroll
                    for (int r = 0; r < 16; ++r) g[r] = x[r];
                };
                if (sub == strip) chain_of<true>(acc, c2, n, hh, keep);
                else chain_of<false>(acc, c2, n, hh, keep);
                if (sub - NWS >= 0) dma_wait<C::LOADS>();    // V has landed
                else dma_wait<0>();
            }
            if (hh == 0) s_tot[st][wave][n] = t_lo + t_hi;
            barrier_lds();                               // totals and V have landed, the weights before have been used
            float mine_a = a, t[NWS];
            totals(t);
#pragma unroll
            for (int w = 0; w < NWS; ++w) {
                if (w == wave) mine_a = a;
                a += t[w];
            }
            if (sub >= 0) {
                if (sub - NWS >= 0) stage(Vg, sub - NWS, mine + (2 + (st ^ 1)) * C::SUB);
                bf16x8 p[2];
                if (linear) weights_of<true>(g, t_lo, t_hi, mine_a, hh, p);
                else weights_of<false>(g, t_lo, t_hi, mine_a, hh, p);
                lds_store16(wts, p[0]);
                lds_store16(wts + 1024, p[1]);
            }
            barrier_lds();
            if (ended()) break;
        }
        if (m && done) {
            // the logits alone, as in sum_tail(), every wave on its own (in rounds with the others, us: B1 H4 T4000 d64 near
            // 21.7 -> 16.7, B2 H4 T777 d32 near 6.2 -> 5.4, all far 8.0 -> 7.8, with no test for it in the rounds)
            float l = 0.0f;
            int b = st ^ 1;
            for (int sub = top - NWS - wave; sub >= 0; sub -= NWS, b ^= 1) {
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
                if (sub - NWS >= 0) stage(Kg, sub - NWS, mine + (b ^ 1) * C::SUB);
                l += sp2_total<false>(logits(b), c2, n, hh);
            }
            float l_lo, l_hi;
            both_halves(l, l_lo, l_hi);
            if (hh == 0) s_tot[st][wave][n] = l_lo + l_hi;   // this round's totals have been read
            barrier_lds();
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");     // subtiles staged before the sweep stopped
    }
    if (m && done) {
        float t[NWS], rest = 0.0f;
        totals(t);
#pragma unroll
        for (int w = 0; w < NWS; ++w) rest += t[w];
        a += rest;
    }

    // ---- store.  oacc[r] is query row 8*(r/4) + 4*hh + r%4, column 32 cols + n.
    if (sums) {
        if (rb) {                                        // remainder bias, as in fwd_bf16_kernel
            const float rem = fast_exp2(-a);
            const float rc = __builtin_bit_cast(float, (uint32_t)rb[head * D + 32 * cols + n] << 16);
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[r] += __shfl(rem, 8 * (r >> 2) + 4 * hh + (r & 3)) * rc;
        }
        store_strip_rows<D>(reinterpret_cast<uint16_t*>(scalar_base(o + (row0 + q0) * D + 32 * cols)), oacc, nlast, n, hh);
    }
    if (m && tid < 32 && n < nlast) m[row0 + q0 + n] = -a * SB_LN2;
    if (clock) {
        clocks[2] = (unsigned long long)clock64();
        clocks[3] = (unsigned long long)wall_clock64();
    }
}

// Two adjacent strips a workgroup, without m: both sweep the same subtiles, from the diagonal of the second one on, NWS to a round, each with waves
// of its own for the logits, chains and weights and for O += A V, as above: sixteen waves in all, the most there can be.  The first strip's waves stage K,
// the second's V; what one stages others read, so that K too lands before a barrier.  The sums are the same in the same order: o is the same, bit for bit.
// Bound by the rounds' latencies as fwd_small_kernel is, with half as many workgroups for near heads to wait for.  Which grids, and what it measured: two_strips().
template <int D> struct FwdTwoCfg {
    static constexpr int NWS = D == 64 ? 6 : 4;         // subtiles of a round, and a strip's waves for them
    static constexpr int NWO = D / 32;                  // and its waves for O += A V
    static constexpr int NTHR = 64 * 2 * (NWS + NWO);
    static constexpr int ROW = D * 2;
    static constexpr int SUB = 32 * ROW;
    static constexpr int LOADS = SUB / 1024;
    static constexpr int V_OFF = 2 * NWS * SUB;         // K and V by round parity, subtile
    static constexpr int Q_OFF = V_OFF + NWS * SUB;     // Q of both strips passes through V of the second round
    static constexpr int W_OFF = 4 * NWS * SUB;         // weights by strip, subtile
    static constexpr int W_SUB = 2 * 1024;
    static constexpr int LDS_BYTES = W_OFF + 2 * NWS * W_SUB;
};

template <int D>
__global__ void __launch_bounds__(FwdTwoCfg<D>::NTHR)
fwd_two_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k,
               const uint16_t* __restrict__ v, const uint16_t* __restrict__ rb, uint16_t* __restrict__ o,
               int T_arg, int BH, int H, int G, int n_arg,         // n_arg: pairs of strips a head; packed batch: sequences
               const int* __restrict__ cu, int Ttot)
{
    using C = FwdTwoCfg<D>;
    constexpr int NWS = C::NWS;
    __shared__ __attribute__((aligned(1024))) char smem[C::LDS_BYTES];
    __shared__ float s_tot[2][2][NWS][32];              // per round parity and strip: softplus totals of the subtiles (base 2), per row

    asm volatile("" :: "s"(q), "s"(k), "s"(v), "s"(T_arg), "s"(G));
    const int tid = threadIdx.x, lane = tid & 63;
    const Share sh = in_scalars(share_of(blockIdx.x, BH, -1));
    const int bh = sh.bh, head = bh % H;
    int T = T_arg, npair = n_arg, i = sh.i;
    long row0 = bh * (long)T, kvrow0 = (long)(G == 1 ? bh : (int)((unsigned)bh / (unsigned)G)) * T;
    if (cu) {                                           // packed batch: bh is the head alone, sh.i its place
        const Place at = place_of<64>(sh.i, cu, n_arg, Ttot, T_arg, lane);
        if (at.T == 0) return;
        T = at.T;
        npair = (T + 63) / 64;
        i = at.i;
        row0 = (long)head * Ttot + at.c0;
        kvrow0 = (long)(head / G) * Ttot + at.c0;
    }
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const bool sums = wave >= 2 * NWS;                  // one of the waves that take O += A V
    const bool second = sums ? wave >= 2 * NWS + C::NWO : wave >= NWS;
    const int w = wave - (second ? NWS : 0);            // subtile of a round
    const int cols = wave - 2 * NWS - (second ? C::NWO : 0);         // columns 32 cols ..
    const int n = lane & 31, hh = lane >> 5, gg = lane >> 4, li = lane & 15;
    const int q0 = (npair - 1 - i) * 64;
    const int rows = min(T - q0, 64);                   // of both strips
    const int last = (q0 + rows - 1) >> 5;              // the last subtile there is
    const int nlast = min(T - 32 * last, 32);           // and its rows
    const int strip = (q0 >> 5) + (second ? 1 : 0);
    const bool live = strip <= last;                    // (a second strip may have no rows)
    const uint16_t* Kg = reinterpret_cast<const uint16_t*>(scalar_base(k + kvrow0 * D));
    const uint16_t* Vg = reinterpret_cast<const uint16_t*>(scalar_base(v + kvrow0 * D));
    const uint32_t smem0 = lds_offset(smem);

    constexpr int CPR = C::ROW / 16;
    int off[C::LOADS];
#pragma unroll
    for (int i = 0; i < C::LOADS; ++i) off[i] = tile_off_perm<D>(i * (1024 / C::ROW) + lane / CPR, lane % CPR);
    auto stage = [&](const uint16_t* X, int sub, uint32_t dst) __attribute__((always_inline)) {
        const uint64_t xb = scalar_base(X + (long)sub * 32 * D);
        if (sub < last || nlast == 32) {
            dma16_to_lds_run_at(xb, off, dst);
        } else {                                        // rows past T are clamped (causality masks them)
            int o[C::LOADS];
#pragma unroll
            for (int i = 0; i < C::LOADS; ++i) o[i] = off[i] - max(i * (1024 / C::ROW) + lane / CPR - (nlast - 1), 0) * C::ROW;
            dma16_to_lds_run_at(xb, o, dst);
        }
    };
    for (int i = wave; i < 2 * C::LOADS; i += C::NTHR / 64) {
        const int r = i * (1024 / C::ROW) + lane / CPR;              // of both strips' 64
        dma16_to_lds_at(scalar_base(q + (row0 + q0) * D), min(r, rows - 1) * C::ROW + (((lane % CPR) ^ swz_perm<D>(r & 31)) << 4),
                        smem0 + C::Q_OFF + i * 1024);
    }
    const uint16_t* const Xg = second ? Vg : Kg;        // what this wave stages, and where: by parity NWS * SUB apart
    const uint32_t mine = smem0 + (second ? C::V_OFF : 0) + w * C::SUB;
    if (!sums && w <= last) {
        stage(Xg, last - w, mine);
        if (second) dma_wait<C::LOADS>();               // all but V
        else dma_wait<0>();
    } else {
        dma_wait<0>();
    }
    barrier_nofence();
    const float c2 = SB_LOG2E / sqrtf((float)D);
    float a[2] = {0.0f, last > (q0 >> 5) ? 0.0f : INFINITY};         // carries of the round, of both strips in all waves
    int st = 0, top = last;
    auto add_up = [&](float& mine_a) __attribute__((always_inline)) {
        float t[2][NWS];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int x = 0; x < NWS; ++x) t[s][x] = s_tot[st][s][x][n];
#pragma unroll
        for (int s = 0; s < 2; ++s)
#pragma unroll
            for (int x = 0; x < NWS; ++x) {
                if (x == w && (s == 1) == second) mine_a = a[s];
                a[s] += t[s][x];
            }
    };
    auto ended = [&]() __attribute__((always_inline)) {              // alike in all waves
        return top < NWS || __builtin_amdgcn_ballot_w64(!(a[0] >= CARRY_EXHAUSTED && a[1] >= CARRY_EXHAUSTED)) == 0;
    };
    // Both kinds of waves pass the same barriers.
    if (!sums) {
        bf16x8 qf[D / 16];
        {
            const uint32_t at = smem0 + C::Q_OFF + (second ? C::SUB : 0) + tile_off_perm<D>(n, hh);
#pragma unroll
            for (int s = 0; s < D / 16; ++s) qf[s] = __builtin_bit_cast(bf16x8, lds_load16(at ^ (s << 5)));
        }
        const uint32_t ka = smem0 + w * C::SUB + tile_off_perm<D>(perm_row(n), hh);          // K as A operand, ^ (s << 5)
        const uint32_t wts = smem0 + C::W_OFF + wave * C::W_SUB + lane * 16;
        for (;; top -= NWS, st ^= 1) {
            const int sub = top - w;
            float g[16], t_lo = 0.0f, t_hi = 0.0f;
            bool linear = true;
            // K(sub) has landed.  Where the next one goes was read before the last round's first barrier
            if (!second && sub >= NWS) stage(Xg, sub - NWS, mine + (st ^ 1) * NWS * C::SUB);
            const bool work = sub >= 0 && sub <= strip && live;
            if (work) {
                u32x4 kop[D / 16];
#pragma unroll
                for (int s = 0; s < D / 16; ++s) kop[s] = lds_load16((ka + st * NWS * C::SUB) ^ (s << 5));
                f32x16 acc;
#pragma unroll
                for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
#pragma unroll
                for (int s = 0; s < D / 16; ++s)
                    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, kop[s]), qf[s], acc, 0, 0, 0);
                auto keep = [&](auto lin, const float (&x)[16], float x_lo, float x_hi) __attribute__((always_inline)) {
                    linear = decltype(lin)::value;
                    t_lo = x_lo;
                    t_hi = x_hi;
#pragma unroll
                    for (int r = 0; r < 16; ++r) g[r] = x[r];
                };
                if (sub == strip) chain_of<true>(acc, c2, n, hh, keep);
                else chain_of<false>(acc, c2, n, hh, keep);
            }
            if (second) dma_wait<0>();                   // V(sub) has landed
            if (hh == 0) s_tot[st][second ? 1 : 0][w][n] = t_lo + t_hi;
            barrier_lds();                               // totals and V have landed, the weights before have been used
            float mine_a = 0.0f;
            add_up(mine_a);
            if (second && sub >= NWS) stage(Xg, sub - NWS, mine + (st ^ 1) * NWS * C::SUB);
            if (work) {
                bf16x8 p[2];
                if (linear) weights_of<true>(g, t_lo, t_hi, mine_a, hh, p);
                else weights_of<false>(g, t_lo, t_hi, mine_a, hh, p);
                lds_store16(wts, p[0]);
                lds_store16(wts + 1024, p[1]);
            }
            if (!second) dma_wait<0>();                  // the next K has landed
            barrier_lds();
            if (ended()) break;
        }
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // subtiles staged before the sweep stopped
        return;
    }
    uint32_t vtr[2];                                     // V of the first subtile, this wave's columns, through the transposing load
#pragma unroll
    for (int t = 0; t < 2; ++t)
        vtr[t] = smem0 + C::V_OFF + tile_off_perm<D>(16 * (gg >> 1) + (li >> 2) + 4 * t, 4 * cols + 2 * (gg & 1) + ((li & 3) >> 1)) + 8 * (li & 1);
    const uint32_t wts = smem0 + C::W_OFF + (second ? NWS * C::W_SUB : 0) + lane * 16;
    f32x16 oacc;                                         // columns 32 cols ..
#pragma unroll
    for (int r = 0; r < 16; ++r) oacc[r] = 0.0f;
    bf16x8 p[2 * NWS], x[2 * NWS];
    auto ask = [&](int st, int count) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2 * NWS; ++i) {
            const int w = min(i >> 1, count - 1), s = i & 1;
            const uint32_t vs = (st * NWS + w) * C::SUB + 8 * s * C::ROW;
            p[i] = __builtin_bit_cast(bf16x8, lds_load16(wts + w * C::W_SUB + s * 1024));
            x[i] = tr_pair_at(vtr[0] + vs, vtr[1] + vs);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    auto multiply = [&](int from, int to) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < 2 * NWS; ++i)
            if (i >= from && i < to) oacc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(p[i], x[i], oacc, 0, 0, 0);
        __builtin_amdgcn_sched_barrier(0);
    };
    int from = last > strip ? 2 : 0;                     // (the first strip has no weights for the subtile on the second one's diagonal)
    for (;; top -= NWS, st ^= 1) {
        if (top != last && live) {                       // the round before: half of it beside the logits of this one
            ask(st ^ 1, NWS);
            multiply(from, NWS);
        }
        barrier_lds();
        if (top != last && live) {
            multiply(NWS, 2 * NWS);
            from = 0;
        }
        float none = 0.0f;
        add_up(none);
        barrier_lds();
        if (ended()) break;
    }
    if (!live) return;
    const int count = min(NWS, top + 1);                 // the last round
    ask(st, count);
    multiply(from, 2 * count);

    // ---- store.  oacc[r] is query row 8*(r/4) + 4*hh + r%4, column 32 cols + n.
    const int own = second ? rows - 32 : min(rows, 32);  // rows of the strip
    if (rb) {                                            // remainder bias, as in fwd_bf16_kernel
        const float rem = fast_exp2(-(second ? a[1] : a[0]));
        const float rc = __builtin_bit_cast(float, (uint32_t)rb[head * D + 32 * cols + n] << 16);
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[r] += __shfl(rem, 8 * (r >> 2) + 4 * hh + (r & 3)) * rc;
    }
    store_strip_rows<D>(reinterpret_cast<uint16_t*>(scalar_base(o + (row0 + 32 * strip) * D + 32 * cols)), oacc, own, n, hh);
}

template <int D, bool WRITE_M, bool RB, Packed PK = Packed::NO, bool TRI = false>
hipError_t launch_one(const uint16_t* q, const uint16_t* k, const uint16_t* v, const uint16_t* rb,
                      uint16_t* o, float* m, int BH, int H, int G, int T, float enough,
                      unsigned long long* tile_counts, hipStream_t stream,
                      const int* cu = nullptr, int Ttot = 0)
{
    constexpr bool VL = PK != Packed::NO;
    const long strips = pieces(BH / H, H, T, 32, VL, Ttot);
    // A halting sweep: strips where every one has a CU to itself, whatever the heads' reach: blocks /
    // strips, us, eps 1e-9, a third of the heads far, then none: B1 H8 T1000 d64 17.4 / 8.3, 6.5 / 5.2; B1 H2 T4000 d64 6.6 / 5.2 (none); B2 H3 T1300 d128 29 / 16,
    // 8.8 / 5.3; B1 H3 T2700 d32 35 / 14.5, 5.4 / 4.7; with more, near heads lose: B1 H4 T4000 d64 57 / 23.5, 6.6 / 9.0; B1 H10 T3000 d32 39 / 23, 5.6 / 14.3.
    const bool fits = !TRI && small_fwd_grid(strips, T, D) && (enough == CARRY_EXHAUSTED || strips <= 256);
    // What tile_counts counts (without m) are the blocks' tiles.  Where strips are taken the blocks sweep for the counts alone: how far o's sweep goes
    // does not depend on whether anyone counts.
    if (!fits || (!WRITE_M && tile_counts)) {
        const int nqb = (T + BQ - 1) / BQ;
        const long grid = block_grid(BH / H, H, T, BQ, PK, Ttot);
        if (grid > 0x7fffffffL) return hipErrorInvalidValue;
        const hipError_t e = launch_workgroups(grid, 64 * NW, [&](unsigned n, int first_wg) {
            hipLaunchKernelGGL((fwd_bf16_kernel<D, WRITE_M, RB, PK, TRI>), dim3(n), dim3(64 * NW), 0, stream,
                               q, k, v, rb, o, m, T, VL ? BH / H : BH, H, G, nqb, enough, tile_counts, cu, Ttot, VL || G > 1 ? -1 : query_run(BH, nqb, D, false), first_wg);
        });
        if (!fits || e != hipSuccess) return e;
    }
    const int heads = VL ? H : BH, n = VL ? BH / H : (T + 31) / 32;
    if constexpr (!WRITE_M && D >= 64) {
        if (enough == CARRY_EXHAUSTED && two_strips(strips, T, D)) {
            const long pairs = pieces(BH / H, H, T, 64, VL, Ttot);
            hipLaunchKernelGGL((fwd_two_kernel<D>), dim3((unsigned)pairs), dim3(FwdTwoCfg<D>::NTHR), 0, stream,
                               q, k, v, rb, o, T, heads, H, G, VL ? BH / H : (T + 63) / 64, cu, Ttot);
            return hipGetLastError();
        }
    }
    auto go = [&](auto waves) {
        constexpr int NWS = decltype(waves)::value;
        hipLaunchKernelGGL((fwd_small_kernel<D, NWS>), dim3((unsigned)strips), dim3(FwdSmallCfg<D, NWS>::NTHR), 0, stream,
                           q, k, v, rb, o, m, T, heads, H, G, n, enough, WRITE_M ? tile_counts : nullptr, cu, Ttot);
    };
    if constexpr (D == 32) {
        if (four_fwd_waves(strips, T)) {
            go(ic<4>());
            return hipGetLastError();
        }
    }
    go(ic<D == 128 ? 4 : 8>());
    return hipGetLastError();
}

}  // namespace

hipError_t launch_fwd_bf16(const uint16_t* q, const uint16_t* k, const uint16_t* v, const uint16_t* rb,
                           uint16_t* o, float* m, int B, int H, int Hkv, int T, int d, hipStream_t stream,
                           unsigned long long* clocks)
{
    const int BH = B * H;
    const int G = H / Hkv;
#define SB_FWD(DD, WM, RBV) launch_one<DD, WM, RBV>(q, k, v, rb, o, m, BH, H, G, T, CARRY_EXHAUSTED, m ? clocks : nullptr, stream)
    if (d == 32) {
        if (rb) return m ? SB_FWD(32, true, true) : SB_FWD(32, false, true);
        return m ? SB_FWD(32, true, false) : SB_FWD(32, false, false);
    }
    if (d == 64) {
        if (rb) return m ? SB_FWD(64, true, true) : SB_FWD(64, false, true);
        return m ? SB_FWD(64, true, false) : SB_FWD(64, false, false);
    }
    if (rb) return m ? SB_FWD(128, true, true) : SB_FWD(128, false, true);
    return m ? SB_FWD(128, true, false) : SB_FWD(128, false, false);
#undef SB_FWD
}

hipError_t launch_fwd_bf16_tri(const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* o, float* m,
                               int B, int H, int T, hipStream_t stream)
{
    return launch_one<128, true, false, Packed::NO, true>(q, k, v, nullptr, o, m, B * H, H, 1, T, CARRY_EXHAUSTED, nullptr, stream);
}

hipError_t launch_fwd_bf16_varlen(const uint16_t* q, const uint16_t* k, const uint16_t* v, const uint16_t* rb,
                                  uint16_t* o, float* m, const int* cu, int nseq, int H, int Hkv,
                                  int Ttot, int max_T, int d, hipStream_t stream)
{
    const int BH = nseq * H;
    const int G = H / Hkv;
#define SB_FWD(DD, WM, RBV)                                                                                     \
    (packed_as(nseq, max_T, Ttot) == Packed::ALIKE                                                              \
         ? launch_one<DD, WM, RBV, Packed::ALIKE>(q, k, v, rb, o, m, BH, H, G, max_T, CARRY_EXHAUSTED, nullptr, stream, cu, Ttot) \
         : launch_one<DD, WM, RBV, Packed::BY_LENGTH>(q, k, v, rb, o, m, BH, H, G, max_T, CARRY_EXHAUSTED, nullptr, stream, cu, Ttot))
    if (d == 32) {
        if (rb) return m ? SB_FWD(32, true, true) : SB_FWD(32, false, true);
        return m ? SB_FWD(32, true, false) : SB_FWD(32, false, false);
    }
    if (d == 64) {
        if (rb) return m ? SB_FWD(64, true, true) : SB_FWD(64, false, true);
        return m ? SB_FWD(64, true, false) : SB_FWD(64, false, false);
    }
    if (rb) return m ? SB_FWD(128, true, true) : SB_FWD(128, false, true);
    return m ? SB_FWD(128, true, false) : SB_FWD(128, false, false);
#undef SB_FWD
}

hipError_t launch_fwd_bf16_halt(const uint16_t* q, const uint16_t* k, const uint16_t* v, uint16_t* o,
                                float eps, unsigned long long* tile_counts,
                                int B, int H, int T, int d, hipStream_t stream)
{
    const int BH = B * H;
    const float enough = fminf(-log2f(eps), CARRY_EXHAUSTED);   // carry = -log2(stick left)
    if (d == 32)
        return launch_one<32, false, false>(q, k, v, nullptr, o, nullptr, BH, H, 1, T, enough, tile_counts, stream);
    if (d == 64)
        return launch_one<64, false, false>(q, k, v, nullptr, o, nullptr, BH, H, 1, T, enough, tile_counts, stream);
    return launch_one<128, false, false>(q, k, v, nullptr, o, nullptr, BH, H, 1, T, enough, tile_counts, stream);
}

}  // namespace sb
