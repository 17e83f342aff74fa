// Single-token decode: one new query per (batch entry, head) against a cache of T keys
// and values, all of them visible (the last row of Eq. 1 on the extended sequence).
//
// The work is one pass over K and V (2*T*d*2 bytes per kv head), a few FLOP per byte: bound by
// HBM bandwidth as long as the vector ALU stays out of the way.  Both contractions are matrix
// instructions with the query heads of a group as the 16 columns (see decode_kernel), split over
// the keys to fill the chip ("split-KV").  Stick-breaking partial results
// combine without any rescaling by a maximum: a chunk of keys processed on its own gives
//     O_s = sum_i A_s[i] v_i   with the chunk-local weights A_s (Eq. 2 inside the chunk),
//     a_s = sum_i softplus(z_i)                      (minus the log of what the chunk leaves),
// and the exact output is  sum_s exp(-sum_{s' nearer than s} a_s') O_s  (the farther
// chunk's log-weights are shifted by what the nearer chunks took; Eq. 2).
//
// In a large cache the nearest keys come first, in a launch of their own: they take most of the stick,
// and where they take all of it (CARRY_EXHAUSTED: every farther weight is zero in fp32) the
// rest of the cache is not read at all.  A small one is read whole by the second launch (split_of()).
//   decode_kernel<.., false, ..>  grid (kv head, block of query heads): the nearest keys, all of a
//       short cache.  Finishes the heads that are exhausted, or all if that was all.
//   decode_kernel<.., true, ..>   grid (chunk, kv head, block of query heads): the keys before
//       those.  Returns at once where the heads are finished.
//   decode_combine_kernel     one workgroup per query head that is not finished: adds the
//       chunks up, in a fixed order.  (Done by the last workgroup of the second launch to arrive
//       instead, it cost more: 14 % of B8 H16 T16384 d128 in stores and counters each workgroup
//       waits for, 10 us at B1 H8 Hkv1 T30000 d64 for one workgroup to add what eight can.)
// Exhaustion does not end a pass that has to return m, the log of the stick left over all keys: the second
// launch then takes the nearest keys as well.
//
// Measured without m, a third of the kv heads reaching far / all of them / all keys in one pass over the
// chip, whatever they take (the first form of this kernel), us: B8 H16 T16384 d128 63 / 164 / 180 (all keys at
// 6.5 TB/s), B1 H32 Hkv8 T65000 d128 25.6 / 51 / 47, B32 H16 T1800 d64 27.6 / 43 / 37, B16 H32 Hkv8 T4096 d128
// 26 / 52 / 45: where every head reaches far the launch in front is 4 to 10 us lost.
#include <mutex>
#include <type_traits>

#include "../../include/sb_attn.h"
#include "sb_kernels.h"
#include "sb_mma.h"
#include "sb_split.h"

namespace sb {
namespace {

constexpr int GMAX = 16;               // query heads of a group per workgroup: the columns of the MFMA
constexpr int COMBINE_THREADS = 256;


// sum of v over the lanes below this one, and over all lanes in `total` (by DPP: the same through LDS shuffles took 800 clocks)
template <int CTRL, int ROWS> __device__ __forceinline__ float dpp_or_zero(float x)
{
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, x), CTRL, ROWS, 0xF, false));
}
__device__ __forceinline__ float wave_prefix_excl(float v, float& total)
{
    float inc = v;
    inc += dpp_or_zero<0x111, 0xF>(inc);                  // row_shr:1, 2, 4, 8
    inc += dpp_or_zero<0x112, 0xF>(inc);
    inc += dpp_or_zero<0x114, 0xF>(inc);
    inc += dpp_or_zero<0x118, 0xF>(inc);
    inc += dpp_or_zero<0x142, 0xA>(inc);                  // row_bcast:15 into rows 1 and 3
    inc += dpp_or_zero<0x143, 0xC>(inc);                  // row_bcast:31 into rows 2 and 3
    total = __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, inc), 63));
    return inc - v;
}

// The far keys are read once and by one workgroup: kept out of the way of the caches (B8 H16 T16384
// d128, every chunk read: 191 -> 168 us; the first launch, whose reads are few, is faster without).
template <bool NT, typename V> __device__ __forceinline__ V stream_load(const V* p)
{
    if constexpr (NT) return __builtin_nontemporal_load(p);
    return *p;
}

// element c of a head's output r and, with c = 0, its m; total: sp2 over all keys.  Remainder bias
// (Appendix C): what no key took goes to the head's embedding.
__device__ __forceinline__ void store_out(const uint16_t* rb, uint16_t* o, float* m, int c, float r, float total)
{
    if (rb) r += fast_exp2(-total) * __builtin_bit_cast(float, (uint32_t)rb[c] << 16);
    const __bf16 val = (__bf16)r;
    o[c] = __builtin_bit_cast(uint16_t, val);
    if (m && c == 0) *m = -total * SB_LN2;
}

// the same of columns c .. c + 3, their embedding e in hand
typedef __attribute__((ext_vector_type(4))) uint16_t u16x4;
__device__ __forceinline__ void store_out4(bool rb, u16x4 e, uint16_t* o, float* m, int c, f32x4 r, float total)
{
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
    if (rb) {
        const float left = fast_exp2(-total);
#pragma unroll
        for (int i = 0; i < 4; ++i) r[i] += left * __builtin_bit_cast(float, (uint32_t)e[i] << 16);
    }
    const bf16x4 v = {(__bf16)r[0], (__bf16)r[1], (__bf16)r[2], (__bf16)r[3]};
    *reinterpret_cast<bf16x4*>(o + c) = v;
    if (m && c == 0) *m = -total * SB_LN2;
}

// A workgroup takes its keys from the nearest down in passes of KEYS, 32 keys per wave.
//   logits   z[key][head] = K q: 16x16x32 bf16 MFMA, A = 16 rows of K (lane: row lane%16, 16-byte chunk
//            4s + lane/16), B = the query heads of the group.  A lane gets four consecutive keys of one head.
//   weights  through LDS: wave g takes head g (and g + NW), NW/2 consecutive keys per lane, lane 0 the nearest.
//   output   O^T[c][head] += V^T w: a lane loads D/16 columns of the 8 rows 8*(lane/16) + i, and an
//            in-register transposition (one v_perm per packed pair) makes them the A operand of
//            D/16 MFMAs, rows = columns of V, 32 keys deep.  B = the weights, each split exactly
//            into three bf16 (8 + 8 + 8 bits of mantissa), so that nothing of the fp32 weight is lost.
// On the vector ALU the same two products cost 35 instructions per 16-byte word and head, which
// bound groups of 4 heads (B1 H32 Hkv8 T65000 d128: 78 us against 48 us of memory time; this way 55).
// K comes through LDS, whole rows at a time, every wave its own: a CU takes in 55 bytes a clock where a load's lanes lie
// side by side, and 15 where they are the rows of an operand, which bound a CU that has the cache's keys to itself
// (pass of 256 keys, d = 128: 5200 of 8000 clocks).  K's place and V's registers (two sets) are asked for again as soon as a
// pass has its logits, one pass ahead.  At d = 128 two far workgroups a CU read faster than three (all heads far, B8 H16 T16384 174 / 167 us,
// B1 H32 Hkv8 T65000 55 / 51).
template <int D, bool FAR, bool SKIP>
__global__ void __launch_bounds__(64 * (FAR ? FAR_NW : NEAR_NW), FAR && D < 128 ? 3 : 2)
decode_kernel(const uint16_t* __restrict__ q, const uint16_t* __restrict__ k, const uint16_t* __restrict__ v,
              const uint16_t* __restrict__ rb, uint16_t* __restrict__ o, float* __restrict__ m,
              float* __restrict__ part_o, float* __restrict__ part_a,
              int T, int Tcap, int Hkv, int G, int near, int C, int nfar)
{
    constexpr int NW = FAR ? FAR_NW : NEAR_NW;
    constexpr int NTHR = 64 * NW;
    constexpr int KEYS = KW * NW;          // keys per pass
    constexpr int ZS = KEYS + 4;           // row stride of the logits in LDS (heads apart by 4 banks)
    constexpr int CW = D / 16;             // columns of V per lane
    constexpr int ROW = 2 * D, CPR = ROW / 16;
    constexpr int NK = KW * ROW / 1024;    // loads of K per wave and pass
    constexpr int NV = 8;                  // and of V
    typedef __attribute__((ext_vector_type(CW / 2))) unsigned int vword;
    constexpr int CH = D / 4;              // 16-byte chunks of a head's columns
    __shared__ __attribute__((aligned(1024))) char kbuf[KEYS * ROW];
    __shared__ __attribute__((aligned(16))) float zs[2][GMAX][ZS];   // per pass parity: logits (base 2), then weights
    __shared__ float s_carry[GMAX];
    __shared__ int s_left[2];              // per pass parity: heads not exhausted
    f32x4* const ored = reinterpret_cast<f32x4*>(kbuf);              // once the keys are done
    static_assert(NW * GMAX * D * 4 <= KEYS * ROW, "the waves' shares fit");

    asm volatile("" :: "s"(q), "s"(k), "s"(v), "s"(T), "s"(Tcap), "s"(G), "s"(near), "s"(C));
    const int bkv = FAR ? blockIdx.y : blockIdx.x;     // batch entry * Hkv + kv head
    const int g0 = blockIdx.z * GMAX;      // first query head (inside the group) of this workgroup
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l16 = lane & 15, lq = lane >> 4;
    const int nch = nfar + (near > 0);     // chunk nfar: the nearest keys, where they have a launch of their own
    const int chunk = FAR ? blockIdx.x : nfar;
    const int kend = FAR ? min(T - near, (chunk + 1) * C) : T;
    const int k0 = FAR ? chunk * C : T - near;
    const long hq0 = (long)bkv * G + g0;   // first query head of this workgroup
    const int live = min(GMAX, G - g0);    // and how many there are
    const float c2 = SB_LOG2E / sqrtf((float)D);

    if constexpr (FAR) {
        if (!m && near > 0) {
            const float a = part_a[(hq0 + min(lane, live - 1)) * nch + nfar];
            if (__builtin_amdgcn_ballot_w64(!(a >= CARRY_EXHAUSTED)) == 0) return;
        }
    }

    // rows hi - KEYS + 32 wave .. + 31; those before k0 are loaded as k0 and masked, with SKIP not at all where they are all a wave has (skip_rows())
    const int r0 = wave * KW - KEYS;
    const char* const kg = reinterpret_cast<const char*>(k) + (long)bkv * Tcap * ROW;
    const char* const vg = reinterpret_cast<const char*>(v) + (long)bkv * Tcap * ROW;
    const uint32_t mine = lds_offset(kbuf) + wave * KW * ROW;
    auto fetch_k = [&](int hi) __attribute__((always_inline)) {
        const uint64_t base = scalar_base(kg + (long)(hi + r0) * ROW);
        const int lo = k0 - (hi + r0);
        if (SKIP && lo >= KW) return;
#pragma unroll
        for (int i = 0; i < NK; ++i) {
            const int row = i * (1024 / ROW) + lane / CPR;
            const int off = max(row, lo) * ROW + (((lane % CPR) ^ swz_nat<D>(row)) << 4);
            if constexpr (FAR) dma16_to_lds_at_nt(base, off, mine + i * 1024);
            else dma16_to_lds_at(base, off, mine + i * 1024);
        }
    };
    auto fetch_v = [&](int hi, vword (&vw)[NV]) __attribute__((always_inline)) {
        const char* const base = vg + (long)(hi + r0) * ROW;
        const int lo = k0 - (hi + r0);
        if (SKIP && lo >= KW) {                                              // (their weights are zero)
#pragma unroll
            for (int i = 0; i < NV; ++i) vw[i] = vword(0u);
            return;
        }
#pragma unroll
        for (int i = 0; i < NV; ++i)
            vw[i] = stream_load<FAR>(reinterpret_cast<const vword*>(base + (unsigned)(max(8 * lq + i, lo) * ROW + l16 * 2 * CW)));
    };
    bf16x8 qw[D / 32];                     // B operand: head l16 (columns past `live` repeat the last one)
    {
        const uint16_t* row = q + (hq0 + min(l16, live - 1)) * D + 8 * lq;
#pragma unroll
        for (int s = 0; s < D / 32; ++s) qw[s] = *reinterpret_cast<const bf16x8*>(row + 32 * s);
    }
    vword va[NV], vb[NV];
    fetch_k(kend);
    fetch_v(kend, va);
    f32x4 acc[CW];                         // O^T: row 4 lq + r of MFMA e is column CW * (4 lq + r) + e, head l16
#pragma unroll
    for (int e = 0; e < CW; ++e) acc[e] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    if (tid < GMAX) s_carry[tid] = 0.0f;   // sp2 of the keys already passed, per head
    if (tid == 0) s_left[0] = 0;
    const uint32_t ka = mine + tile_off_nat<D>(l16, lq);             // A operand: rows 16t + l16, chunks 4s + lq: + 16t ROW, ^ (s << 6)
    int par = 0, hi = kend;
    // one pass; whether another follows.  vw: this pass's V, vn: the next one's
    auto pass = [&](vword (&vw)[NV], vword (&vn)[NV]) __attribute__((always_inline)) {
        const bool more = hi - KEYS > k0;
        // ---- logits
        dma_wait<NV>();                    // K has landed, V was asked for behind it
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            f32x4 z = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int s = 0; s < D / 32; ++s)
                z = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, lds_load16((ka + 16 * t * ROW) ^ (s << 6))), qw[s], z, 0, 0, 0);
            const int i = wave * KW + 16 * t + 4 * lq;
#pragma unroll
            for (int r = 0; r < 4; ++r) z[r] = hi - KEYS + i + r >= k0 ? z[r] * c2 : -INFINITY;
            if (l16 < live) *reinterpret_cast<f32x4*>(&zs[par][l16][i]) = z;
        }
        barrier_lds();
        // V has landed (nothing is asked for between it and here that the compiler does not count)
#pragma unroll
        for (int i = 0; i < NV; ++i)
#pragma unroll
            for (int e = 0; e < CW / 2; ++e) {
                unsigned int x = vw[i][e];
                asm volatile("" : "+v"(x));
                vw[i][e] = x;
            }
        if (more) {
            fetch_k(hi - KEYS);
            fetch_v(hi - KEYS, vn);
        }
        if (tid == 0) s_left[par ^ 1] = 0;                   // everyone has read it, in the pass before
        // ---- weights: w[i] = 2^(x_i - carry - sum_{i' >= i} sp2(x_i'))  (Eq. 2)
        for (int g = wave; g < live; g += NW) {
            constexpr int EPL = KEYS / 64;
            typedef __attribute__((ext_vector_type(EPL))) float zvec;
            zvec* z = reinterpret_cast<zvec*>(&zs[par][g][EPL * (63 - lane)]);
            zvec x = *z;
            float sp[EPL], own = 0.0f;
#pragma unroll
            for (int e = 0; e < EPL; ++e) { sp[e] = sp2(x[e]); own += sp[e]; }
            float total;
            const float carry = s_carry[g];
            float run = wave_prefix_excl(own, total) + carry;
#pragma unroll
            for (int e = EPL - 1; e >= 0; --e) {
                run += sp[e];
                x[e] = fast_exp2(x[e] - run);
            }
            *z = x;
            if (lane == 0) {
                s_carry[g] = carry + total;
                if (!(carry + total >= CARRY_EXHAUSTED)) atomicAdd(&s_left[par], 1);
            }
        }
        barrier_lds();
        // ---- output
        {
            float w[8];
            const float* wrow = &zs[par][min(l16, live - 1)][wave * KW + 8 * lq];
#pragma unroll
            for (int i = 0; i < 8; ++i) w[i] = wrow[i];
            bf16x8 w0, w1, w2;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                w0[i] = (__bf16)w[i];
                const float r1 = w[i] - (float)w0[i];
                w1[i] = (__bf16)r1;
                w2[i] = (__bf16)(r1 - (float)w1[i]);
            }
#pragma unroll
            for (int e = 0; e < CW; ++e) {
                // column e of the 8 rows: bytes 0,1 (e even) or 2,3 (e odd) of word e/2 of each
                u32x4 x;
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    x[i] = __builtin_amdgcn_perm(vw[2 * i + 1][e >> 1], vw[2 * i][e >> 1], (e & 1) ? 0x07060302u : 0x05040100u);
                const bf16x8 a = __builtin_bit_cast(bf16x8, x);
                acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w2, acc[e], 0, 0, 0);
                acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w1, acc[e], 0, 0, 0);
                acc[e] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, w0, acc[e], 0, 0, 0);
            }
        }
        const bool on = more && (m || s_left[par] != 0);
        hi -= KEYS;
        par ^= 1;
        return on;
    };
    barrier_lds();
    while (pass(va, vb) && pass(vb, va)) {}
    dma_wait<0>();                         // keys asked for before the end was known
    barrier_lds();                         // (theirs is the place of the shares)

    // the thread's columns of the embeddings, asked for ahead of the waves' shares, which take as long as the load.  (Asked for ahead of the keys they held two registers
    // through the sweep, with a bias or without: at d = 32 82 in place of 79, two workgroups a CU in place of three.  With the output in hand / ahead of the keys / here, us, with
    // bias, then without: B32 H24 T300 d32 6.4 / 8.2 / 6.2, 6.2 / 8.2 / 6.1;  B24 H64 Hkv32 T500 d32 9.7 / 10.4 / 9.5, 10.2 / 10.7 / 10.2;  B16 H22 Hkv11 T491 d64 5.9 / 5.8 / 5.7,
    // 5.6 / 5.7 / 5.6;  B1 H12 Hkv4 T333 d128 6.4 / 6.3 / 6.2, 6.2 in all three.)
    static_assert(FAR || GMAX * CH <= NTHR, "one round of the loop that stores the output");
    u16x4 bias = u16x4(0);
    if (!FAR && rb && tid < live * CH)
        bias = *reinterpret_cast<const u16x4*>(rb + ((bkv % Hkv) * G + g0 + tid / CH) * D + 4 * (tid % CH));
    // ---- the waves' shares, all heads at once: a lane holds 4 CW columns of its head, CW chunks of 16 bytes.  The chunk's place is xor-ed with
    // the head, so that heads, whose rows begin in the same bank, do not meet in one.  (Float by float, four heads at a time with two barriers each, this took
    // 2300 clocks of 9600 for up to four heads and 5200 for eight, d = 128; now 2000.  With the loads of waves that have no keys left out, us: B9 H24 Hkv3 T476
    // d128 8.9 -> 7.7, B1 H12 Hkv4 T333 d128 6.8 -> 6.2, B1 H64 Hkv8 T3000 d128 9.0 -> 8.5, B2 H16 Hkv2 T70 d128 6.6 -> 5.3.)
    if (l16 < live) {
        f32x4* const r = ored + (wave * live + l16) * CH;
#pragma unroll
        for (int j = 0; j < CW; ++j) {
            f32x4 x;
#pragma unroll
            for (int i = 0; i < 4; ++i) x[i] = acc[(4 * j + i) % CW][(4 * j + i) / CW];
            r[(CW * lq + j) ^ (l16 & 7)] = x;
        }
    }
    barrier_lds();
    for (int i = tid; i < live * CH; i += NTHR) {
        const int g = i / CH, c = i % CH;
        f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < NW; ++w) s += ored[(w * live + g) * CH + (c ^ (g & 7))];
        const float a = s_carry[g];
        if (!FAR && (nfar == 0 || (!m && a >= CARRY_EXHAUSTED)))
            store_out4(rb != nullptr, bias, o + (hq0 + g) * D, m ? m + hq0 + g : nullptr, 4 * c, s, a);
        if (nfar > 0) {
            *reinterpret_cast<f32x4*>(&part_o[((hq0 + g) * nch + chunk) * D + 4 * c]) = s;
            if (c == 0) part_a[(hq0 + g) * nch + chunk] = a;
        }
    }
}

template <int D>
__global__ void __launch_bounds__(COMBINE_THREADS)
decode_combine_kernel(const float* __restrict__ part_o, const float* __restrict__ part_a,
                      const uint16_t* __restrict__ rb, uint16_t* __restrict__ o, float* __restrict__ m, int H, int nch, bool near)
{
    constexpr int NV = D / 4;              // a thread adds four columns of every NG-th chunk
    constexpr int NG = COMBINE_THREADS / NV;
    __shared__ __attribute__((aligned(16))) float ored[NG][D];
    __shared__ float ws[MAXFAR + 1];
    const long bh = blockIdx.x;
    const int tid = threadIdx.x, lane = tid & 63;
    const int c4 = tid % NV, grp = tid / NV;
    const float* pa = part_a + bh * nch;
    // chunk i is shifted by everything the nearer (higher) chunks took; lane l holds chunks 2(63 - l), 2(63 - l) + 1
    const int ch = 2 * (63 - lane);
    if (!m && near && pa[nch - 1] >= CARRY_EXHAUSTED) return;      // finished by the first launch
    float a[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) a[e] = ch + e < nch ? pa[ch + e] : 0.0f;
    const f32x4* po = reinterpret_cast<const f32x4*>(part_o + bh * (long)nch * D) + c4;
    // all of a thread's share is in flight at once
    constexpr int N = (MAXFAR + NG) / NG;
    f32x4 x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = po[(long)min(grp + i * NG, nch - 1) * NV];
    float total;
    float above = wave_prefix_excl(a[0] + a[1], total);
    if (tid < 64)
#pragma unroll
        for (int e = 1; e >= 0; --e) {
            ws[ch + e] = ch + e < nch ? fast_exp2(-above) : 0.0f;
            above += a[e];
        }
    __syncthreads();
    f32x4 s = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int i = 0; i < N; ++i) s += ws[grp + i * NG] * x[i];
    *reinterpret_cast<f32x4*>(&ored[grp][4 * c4]) = s;
    __syncthreads();
    if (tid < D) {
        float r = 0.0f;
#pragma unroll
        for (int g = 0; g < NG; ++g) r += ored[g][tid];
        store_out(rb ? rb + (bh % H) * D : nullptr, o + bh * D, m ? m + bh : nullptr, tid, r, total);
    }
}

// Whether waves without keys of their own in the last pass of the first launch leave their loads out.  Where the launch is one round of workgroups they are what the others
// wait for; in later passes and rounds, and in the far launch, the branch costs more than the loads.  Loads / left out, us: d = 128 B1 H12 Hkv4 T333 6.8 / 6.3, B2 H16 Hkv2 T70 5.1 / 4.5;  d = 64 B2 H16
// Hkv4 T333 5.4 / 5.1;  d = 32 B32 H24 T300 6.4 / 6.1;  not d = 128 B14 H50 Hkv25 T495 17.5 / 18.1, B16 H64 Hkv32 T400 19.7 / 20.2;  far launch B2 H28 Hkv7 T6248 11.0 / 11.8;  d = 64 B5 H8 T36294 24.7 / 25.3;
// d = 32 B27 H8 Hkv4 T2893 10.5 / 10.8;  but d = 128 B8 H16 T16384 61.5 / 61.1
inline bool skip_rows(long wgs, int keys, int d)
{
    constexpr int KEYS = KW * NEAR_NW;
    return wgs <= (d == 32 ? 768 : d == 64 ? 512 : 256) && (keys - 1) % KEYS < KEYS - KW;
}

template <int D>
hipError_t launch_d(const uint16_t* q, const uint16_t* k, const uint16_t* v, const uint16_t* rb,
                    uint16_t* o, float* m, float* workspace, int B, int H, int Hkv, int T, int Tcap, hipStream_t stream)
{
    const int G = H / Hkv;
    const int nz = (G + GMAX - 1) / GMAX;
    const Split s = split_of((long)B * Hkv * nz, 4.0 * B * Hkv * T * D, T, D, m != nullptr);
    const long heads = (long)B * H;
    float* part_o = workspace;                                            // [heads][chunks][D]
    float* part_a = part_o + heads * s.chunks() * D;                      // [heads][chunks]
    hipError_t e = hipSuccess;
    if (s.near > 0) {
        auto go = [&](auto skip) {
            hipLaunchKernelGGL((decode_kernel<D, false, decltype(skip)::value>), dim3((unsigned)(B * Hkv), 1u, (unsigned)nz), dim3(64 * NEAR_NW), 0, stream,
                               q, k, v, rb, o, m, part_o, part_a, T, Tcap, Hkv, G, s.near, s.C, s.nfar);
        };
        if (skip_rows((long)B * Hkv * nz, s.near, D)) go(std::true_type());
        else go(std::false_type());
        e = hipGetLastError();
    }
    if (e != hipSuccess || s.nfar == 0) return e;
    hipLaunchKernelGGL((decode_kernel<D, true, false>), dim3((unsigned)s.nfar, (unsigned)(B * Hkv), (unsigned)nz), dim3(64 * FAR_NW), 0, stream,
                       q, k, v, rb, o, m, part_o, part_a, T, Tcap, Hkv, G, s.near, s.C, s.nfar);
    e = hipGetLastError();
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((decode_combine_kernel<D>), dim3((unsigned)heads), dim3(COMBINE_THREADS), 0, stream,
                       part_o, part_a, rb, o, m, H, s.chunks(), s.near > 0);
    return hipGetLastError();
}

// Scratch of the entry point that allocates nothing: every GPU the library runs on holds its
// own copy of this array, at its own address, until the process ends.  Host code never uses
// the array's name as a pointer: the device address is looked up once per device.
constexpr size_t DEC_STATIC_BYTES = SB_DECODE_STATIC_BYTES;
static __device__ __align__(256) unsigned char scratch[DEC_STATIC_BYTES];

constexpr int DEC_MAX_DEVICES = 64;
std::mutex scratch_lock;
void* scratch_ptr[DEC_MAX_DEVICES];        // device address of `scratch`, per device, once known

}  // namespace

int decode_max_T() { return 524288; }

size_t decode_static_bytes() { return DEC_STATIC_BYTES; }

hipError_t decode_static_scratch(float** out)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) return e;
    if (dev < 0 || dev >= DEC_MAX_DEVICES) return hipErrorInvalidDevice;
    std::lock_guard<std::mutex> guard(scratch_lock);
    if (!scratch_ptr[dev]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return e;
        if (!p) return hipErrorInvalidSymbol;
        scratch_ptr[dev] = p;
    }
    *out = static_cast<float*>(scratch_ptr[dev]);
    return hipSuccess;
}

size_t decode_workspace_bytes(int B, int H, int T, int d)
{
    const size_t nchunk = room(T);
    return sizeof(float) * ((((size_t)B * H * nchunk + 3) & ~(size_t)3) + (size_t)B * H * nchunk * d);
}

hipError_t launch_decode(const uint16_t* q, const uint16_t* k, const uint16_t* v, const uint16_t* rb,
                         uint16_t* o, float* m, float* workspace,
                         int B, int H, int Hkv, int T, int Tcap, int d, hipStream_t stream)
{
    if (B * Hkv > 65535) return hipErrorInvalidValue;
    if (d == 32) return launch_d<32>(q, k, v, rb, o, m, workspace, B, H, Hkv, T, Tcap, stream);
    if (d == 64) return launch_d<64>(q, k, v, rb, o, m, workspace, B, H, Hkv, T, Tcap, stream);
    return launch_d<128>(q, k, v, rb, o, m, workspace, B, H, Hkv, T, Tcap, stream);
}

}  // namespace sb
