// Which blocks a workgroup works on.
#pragma once
#include <hip/hip_runtime.h>

#include <algorithm>

namespace sb {

// Block i of a head (i = 0 the longest) and block n-1-i form pair i, of the same causal cost for
// every i; but how much of that cost a block is depends on how far its head's weights reach.
// Workgroup ids go round the 8 XCDs and start in order as places come free.
//
// Longest first: every workgroup one block, block 0 of all heads, then block 1, ...  What runs last is
// short.  The heads turn with i, so that no XCD is left with more of the costly heads than another: with
// every block, or with every run of 2^run blocks.  Inside a run a head stays on one XCD, and its
// blocks, which sweep the same tiles at the same time, find them in that XCD's L2.
// Longest first against pairs (below), a third of the heads reaching far, us: forward B1 H32 T16384 d128
// 940 / 1217, B8 H16 T4096 d128 331 / 615, query-stationary backward B8 H16 T2048 d64 142 / 170.
//
// In pairs: every workgroup a pair, every head on one XCD, slot s of the XCDs takes heads 8s .. 8s+7,
// turned by s(s+1)/2.  Only the key-stationary kernel of d = 128, one workgroup per CU and nothing else
// to hide a tile's latency, still takes it (take_pairs()): its second block is fetched under the end of the first.
// Pairs / longest first there, us, all heads far, then a third: B8 H16 T4096 1270 / 1345, 612 / 650; T8000 4706 / 5219,
// 1849 / 2035; B4 H32 T6144 2700 / 2930, 1155 / 1260; B16 H32 T512 171 / 177, 157 / 172; B8 H20 T4096 1592 / 1753,
// 818 / 771; B8 H24 T2048 549 / 578, 372 / 340.  From 128 heads on: with fewer it still wins where all reach far, but
// too little evens out where a third does: B7 H16 T4096 1112 / 1184, 557 / 564; B4 H24 T4096 955 / 990, 607 / 500;
// B2 H32 T8192 2355 / 2470, 1130 / 1035.  And where whole octets of heads fill whole rounds of the chip, as pairs cost all
// the same: B10 H20 T1000 (3.1 rounds) 227 / 199, 168 / 146; B3 H48 T2048 (4.5) 449 / 440, 271 / 259; B8 H22
// T2048 (5.5) 544 / 540, 328 / 319; B10 H13 T3000 834 / 810, 507 / 406; B8 H17 T4096 1434 / 1500, 746 / 663.
// Not for heads that share a kv head or a packed batch, whose pairs keep more than the registers hold: whole
// backward B16 H32 Hkv8 T4096 9430 / 9620, 5130 / 4945; B32 H32 Hkv4 T1024 1500 / 1455, 1290 / 1095; B6 H48 Hkv24 T3000
// 3130 / 3050, 1708 / 1564.
struct Share {
    int bh;                   // head
    int i;                    // block, or with pairs pair
};
inline long share_grid(long heads, int nblk, bool pairs)
{
    return pairs ? 8L * ((heads + 7) / 8) * ((nblk + 1) / 2) : heads * nblk;
}
inline bool take_pairs(long heads, int nblk)
{
    if (heads < 128 || heads % 8 != 0) return false;
    const long n = share_grid(heads, nblk, true), idle = (256 - n % 256) % 256;      // places in the last round
    return 32 * idle <= n;
}

// Grids of the backward that take one strip of 32 rows a workgroup, its waves sharing the strip's other side
// (bwd_dq_small_kernel, bwd_dkv_small_kernel), in place of 128-row blocks whose every wave has the
// whole other side to itself.  What bounds the blocks there is one chain, what bounds the strips from a round or two of the
// chip on is their tiles, which no other wave shares: the longer the chain, the more strips are still worth it.
// Blocks / strips, us, query-stationary, then key-stationary (the better of its block kernels), all heads far, then a third, then none:
//   d = 32   B1 H16 T500 (256) 14 / 6, 14 / 7;  T2048 H14 (896) 46 / 32, 45 / 25, 12 / 20 and 44 / 31, 44 / 22, 12 / 17 (eight waves; four_waves());  T4096 H12 (1536)
//            89 / 83, 88 / 51, 16 / 31 and 84 / 81, 84 / 45, 17 / 27
//   d = 64   T8192 H1 (256) 200 / 56 and 189 / 52
//   d = 128  T500 H16 (256) 22 / 13, 22 / 13, 18 / 11 and 19 / 14, 19 / 14, 15 / 11;  T2000 H8 (504) 70 / 43, 69 / 37, 19 / 23 and 50 / 43, 48 / 34,
//            18 / 23;  T8192 H1 (256) 263 / 130 and 162 / 108
// and not    d = 32 T500 H48 (768) 14.5 / 13.5, 14 / 15, 13 / 15 and 14 / 14.5, 14 / 14, 12 / 13;  T4096 H16 (2048) 89 / 109, 89 / 67, 17 / 40 and 92 / 105,
//            84 / 60, 18 / 36;  d = 64 T1000 H32 (1024) 30 / 31, 30 / 27, 15 / 26 and 31 / 35, 31 / 27, 17 / 25;  d = 128 T500 H32 (512) 23 / 20, 22 / 22,
//            19 / 22 and 21 / 24, 21 / 22, 18 / 22;  T1000 H24 (768) 39 / 42, 39 / 38, 20 / 33 and 35 / 46, 31 / 37, 22 / 32;  T3000 H10 (940) 101 / 106,
//            100 / 71, 21 / 42 and 82 / 102, 68 / 64, 23 / 41
// and, just beyond the line, not  d = 64 T3000 H16 (1504) 77 / 80, 77 / 53, 20 / 37 and 77 / 85, 75 / 50, 22 / 37;  d = 128 T3000 H8 (752) 101 / 91, 100 / 61, 20 / 33
//            and 73 / 85, 67 / 57, 22 / 33;  nor what would gain by it:  d = 32 T1000 H24 (768) 25 / 18, 25 / 17, 13 / 16 and 24 / 18, 24 / 16, 12 / 13;  T320 H26 (260)
//            9.4 / 7.7 and 10 / 8;  d = 64 T500 H32 (512) 17 / 11, 17 / 12, 14 / 13 and 18 / 13, 18 / 13, 15 / 12;  T1000 H24 30 / 22, 29 / 21, 15 / 20 and 30 / 26,
//            30 / 22, 16 / 20
// The limits are where a mix gains more by strips than near heads, and beyond them far ones, lose.  From 256 strips on at d = 128 and from 768 on below,
// near heads alone do lose: whole backward, blocks / strips, none far, then a third, B1 H8 T2000 d128 37 / 45, 117 / 72;  H5 T4096 44 / 61, 218 / 131;  H2 T8192 37 / 46;
// H14 T2500 d64 40 / 45, 131 / 69;  H12 T2600 d64 32 / 38, 134 / 68;  H12 T4096 d32 35 / 31, 169 / 77.
// One line serves both passes and, below d = 128, both head sizes.  What is due to long chains goes by the mean length of
// a packed batch's sequences: one long one among many short ones leaves the rest of the strips short.  Beyond 8192 rows not measured.
constexpr int SMALL_T = 4096, LONG_T = 8192;
inline bool small_grid(long strips, int T, int mean, int d)
{
    long limit = T > 64 && T <= SMALL_T ? (d == 128 ? 256 : T >= 1024 ? 768 : T > 341 ? 3L * T / 4 : 256) : 0;
    if (mean >= 1536 && T <= LONG_T) limit = std::max(limit, d == 128 ? std::clamp(mean / 4L, 512L, 768L) : std::clamp(mean / 2L, 768L, 1536L));
    return strips <= limit;
}
// The key-stationary pass of G query heads to a kv head: G times as long a chain for every strip of keys, and the strip's first loads, K, V and
// stores are shared by as many.  Whole backward with blocks / strips of keys, us, all heads far, then a third, then none:
//   d = 32   B1 H32 Hkv8 T3870 (968 strips) 421 / 278, 388 / 182, 64 / 62;  B8 H32 Hkv4 T800 (800) 181 / 119, 180 / 96, 103 / 77;  B4 H32 Hkv4 T3672 (1840)
//            942 / 953, 805 / 541, 186 / 172;  B1 H16 Hkv4 T8192 (1024) 881 / 594, 875 / 562, 64 / 69
//   d = 64   B1 H24 Hkv12 T3000 (1128) 228 / 196, 224 / 135, 68 / 63;  B8 H16 Hkv4 T1500 (1504) 242 / 268, 211 / 149, 120 / 108;  B16 H32 Hkv4 T300 (640)
//            108 / 79 in all three;  B16 H32 Hkv8 T100 (512) 33 / 28 in all three;  B2 H24 Hkv12 T2048 (1536) 176 / 189, 159 / 124, 71 / 73
//   d = 128  B1 H32 Hkv8 T2048 (512) 258 / 231, 251 / 184, 81 / 74;  B3 H16 Hkv4 T1600 (600) 217 / 207, 203 / 148, 103 / 90;  B2 H6 Hkv3 T2000 (378) 164 / 129,
//            162 / 127, 49 / 46;  B12 H12 Hkv4 T256 (384) 49 / 43 in all three;  B1 H8 Hkv2 T8192 (512) 937 / 743, 81 / 77, 81 / 77
// and not    d = 32 B11 H20 Hkv5 T2770 (4785) 876 / 989, 437 / 377, 197 / 240;  B8 H32 Hkv16 T400 (1664) 49 / 60, 49 / 59, 47 / 59;  d = 64 B4 H24 Hkv8 T2048
//            (2048) 296 / 364, 217 / 173, 109 / 118;  B12 H9 Hkv3 T1500 (1692) 202 / 232, 166 / 158, 102 / 102;  d = 128 B4 H12 Hkv4 T2048 (1024) 276 / 317,
//            212 / 204, 117 / 108;  B16 H8 Hkv1 T1500 (752) 428 / 485, 260 / 178, 260 / 178
inline bool grouped_strips(long strips, int G, int T, int mean, int d)
{
    if (G == 1 || mean <= 64 || T > LONG_T) return false;
    if (d == 128) return strips <= (G == 2 ? std::clamp(2L * mean / 7, 328L, 576L) : 640L);
    return strips <= std::clamp(3L * G * mean / 8, 512L, d == 64 ? 1536L : 1920L);
}

// How many strips or blocks of `rows` rows there are: exactly, or in a packed batch of nseq sequences, whose
// lengths the host does not know, at most (and as many as in the batched call where they are all equal).
inline long pieces(int B, int H, int T, int rows, bool packed, int Ttot)
{
    const long all = (long)B * H * ((T + rows - 1) / rows);
    return packed ? std::min(all, (long)H * (Ttot / rows + B)) : all;
}

// Gradient of the remainder bias: chunks of DR_ROWS rows, of one batch entry or of all of a packed batch's sequences
constexpr int DR_ROWS = 128;
inline int bias_chunks(int B, int T, bool packed, int Ttot) { return (int)pieces(packed ? B : 1, 1, T, DR_ROWS, packed, Ttot); }

// The 128-row blocks of a packed batch.  ALIKE: every sequence gets as many workgroups as the longest may need, and those beyond its end
// have nothing to do; block 0 of all sequences and heads, then block 1, ... is longest first as long as the lengths are much the same.
// BY_LENGTH: as many as pieces() counts, a workgroup looking up its block among all sequences' (longest_first(), below).  With
// lengths that differ it is the order that counts, and by some heads the empty workgroups.  ALIKE / BY_LENGTH, a third of the heads far, us, forward,
// backward (`of` the workgroups that ALIKE takes for one of pieces()):
//   d = 64   H24, 19 of 26 to 4096 rows (4.1) 160 / 150, 430 / 363;  H32 Hkv4, 15 up to 5931 (4.6) 262 / 238, 1920 / 1700;  H2, 5000 and 300 of 16 (32) 46 / 37, 75 / 35;
//            H16, 2000 and 20 of 700 to 900 (2.1) 68 / 59, 227 / 192;  H16, 8 up to 3341 (1.8) 93 / 79, 269 / 234;  H16, 16 up to 1881 (1.5) 76 / 71, 221 / 213
//   d = 128  H16, 31 up to 2048 (3.1) 118 / 108, 386 / 340;  H32 Hkv8, 16 up to 2000 (2.7) 130 / 129, 511 / 391;  H12, 8 up to 8000 (2.6) 548 / 425, 1203 / 910;
//            H16, 40 up to 991 (1.7) 100 / 101, 378 / 346
//   d = 32   H12, 24 up to 1500 (2.4) 32 / 27, 102 / 87;  H12 Hkv6, 22 up to 8192 (5.1) 185 / 143, 805 / 616;  H16, 40 up to 977 (1.7) 39 / 36, 119 / 107
// The look-up is 0.3 to 0.9 us ahead of a block's first load.  Not worth it for short sequences, unless they differ much, less so for many:
//   H24      d64 60 of 300, one of 600 (1.5) 60 / 59, 233 / 239;  d32 60 of 16 to 299 (1.3) 24.2 / 24.5, 78 / 83;  d64 200 of 16 to 399 (1.6) 127 / 138, 481 / 505;  240
//            of 16 to 200, one of 600 (2.8) 82 / 87, 316 / 323;  but 60 of 16 to 99, one of 260 (2.1) 17.4 / 15.2, 60 / 51;  100 of 16 to 300, one of 800
//            (3.2) 53 / 48, 208 / 197
enum class Packed { NO, ALIKE, BY_LENGTH };
inline Packed packed_as(int nseq, int T, int Ttot)
{
    const int least = nseq > 64 ? 15 : Ttot < 512L * nseq ? 10 : 6;
    return 5L * nseq * ((T + 127) / 128) > least * pieces(nseq, 1, T, 128, true, Ttot) ? Packed::BY_LENGTH : Packed::ALIKE;
}
inline long block_grid(int B, int H, int T, int rows, Packed as, int Ttot)
{
    return as == Packed::BY_LENGTH ? pieces(B, H, T, rows, true, Ttot) : (long)B * H * ((T + rows - 1) / rows);
}

// Rows of a sequence, in the mean
inline int mean_T(int B, int T, bool packed, int Ttot) { return packed ? Ttot / B : T; }

// A packed batch's strips are launched as pieces() counts them, T (max_T) being at least the longest sequence's length and perhaps far
// more; place_of() finds a workgroup's.  Each that T leaves room for, in every sequence, cost 2 us a thousand: 64 sequences of 32 rows,
// H4 d64, T 2048, forward 34.6 -> 5.7 us, backward 85 -> 15.8.  The rules above hold for packed batches as well, though the host
// cannot tell a long chain from many short ones.  Blocks / strips, us, forward, then backward: that batch 4.9 / 5.7, 12.9 / 15.8; T 200
// with 32 of them 5.3 / 5.1, 11.0 / 14.2; H2 d128, T 512 5.5 / 5.3, 12.8 / 17.4; 100 of 70 rows, H1 d64, T 400 5.3 / 8.3, 15.2 / 15.1 (blocks);
// but with one long one, all heads far, then none: 250 and 20 of 16 rows, H4 d64 7.5 / 5.7, 23 / 15.7 and 7.5 / 5.9, 23 / 15.6; 500 and
// 40 of 60, H2 d32 9.3 / 6.1, 28 / 15 and 9.0 / 5.4, 24 / 12; 1000 and 30 of 20, H4 d64 18 / 10.4, 66 / 28 and 13.7 / 7.4, 33 / 18; 2000
// and 44 of 16, H2 d64 31 / 16.7, 119 / 44 and 19.5 / 9.0, 32 / 20.
struct Place {
    int seq, i;               // sequence, strip
    int c0, T;                // the sequence's first row and length; none: T = 0
};
__device__ __forceinline__ int sum_up_to_lane(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, false);       // row_shr:1, 2, 4, 8
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, false);
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);       // row_bcast:15 into rows 1 and 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);       // row_bcast:31 into rows 2 and 3
    return x;
}
// The strips (or blocks, of ROWS rows) of sequence 0, then of sequence 1, ...: what has nothing to do comes last.  (Among the others, with the
// offsets alone to say where a sequence's places begin, it takes a CU's turn: the batch above 8.2 and 25.9 us.)
template <int ROWS>
__device__ __forceinline__ Place place_of(int place, const int* __restrict__ cu, int nseq, int Ttot, int T_arg, int lane)
{
    int s = min(lane, nseq - 1), n0 = cu[s], n1 = cu[s + 1];
    for (int b = 0; b < nseq; b += 64) {
        const int c0 = n0, c1 = min(n1, Ttot);
        s = min(b + 64 + lane, nseq - 1);                                     // the next 64, one step ahead
        n0 = cu[s];
        n1 = cu[s + 1];
        const int T = b + lane < nseq && c0 >= 0 && c1 > c0 ? min(c1 - c0, T_arg) : 0;     // never past the packed rows or the stated maximum
        const int n = (T + ROWS - 1) / ROWS;
        const int upto = sum_up_to_lane(n);
        const unsigned long long beyond = __builtin_amdgcn_ballot_w64(upto > place);
        if (beyond) {
            const int at = __builtin_ctzll(beyond);
            return {b + at, place - __builtin_amdgcn_readlane(upto - n, at), __builtin_amdgcn_readlane(c0, at), __builtin_amdgcn_readlane(T, at)};
        }
        place -= __builtin_amdgcn_readlane(upto, 63);
    }
    return {0, 0, 0, 0};
}
// Grids of the forward that take one strip of 32 rows a workgroup, its waves taking the strip's subtiles in rounds
// (fwd_small_kernel), in place of 128-row blocks whose every wave has its rows' chain to itself.  Blocks / strips, us, without m (with it,
// where it matters, in brackets), all heads far, then a third, then none:
//   d = 32   T3000 H10 (940) 39 / 34, 38 / 23, 7 / 14 (22 / 20) (eight waves; four_fwd_waves());  T8192 H1 100 / 37
//   d = 64   H64 T100 (256) 5.7 / 5.0;  H24 T500 (384) 10.6 / 8.5, 10.5 / 8.0, 8.2 / 8.0;  T3000 H10 (940) 45 / 41, 44 / 28, 9 / 18 (26 / 25) (one to a
//            workgroup; two_strips());  T8192 H1 114 / 44;  T16384 H1 225 / 92, none 8.5 / 9.7
//   d = 128  H24 T500 (384) 14.6 / 11.1, 14.5 / 10.5, 11.3 / 10.5;  T1000 H12 (384) 24.5 / 15.3, 24 / 15, 11.4 / 11.9;
//            T2048 H10 (640) 45 / 38, 44 / 26, 13 / 18 (26 / 26);  T8192 H1 161 / 82;  T16384 H1 318 / 175, none 12 / 16
// and not, d = 32 H37 T200 (259) 5.7 / 6.4;  T2048 H18 (1152) 28 / 32, 27 / 23, 8 / 17 (17 / 22);  d = 64 H96 T100 (384) 5.8 / 7.1;  T500 H48 (768) 11.1 / 14.8,
//            10.8 / 13.9, 8.6 / 13.4;  T2000 H16 (1008) 32 / 33, 32 / 24, 9 / 18 (20 / 22.5);  T4096 H12 (1536) 62 / 78, 60 / 45, 12 / 25 (34 / 44);
//            d = 128 T500 H48 (768) 16 / 21, 16 / 19, 13 / 19;  T1000 H24 (768) 25 / 30, 25 / 23, 13 / 19;  T4096 H9 (1152) 87 / 109, 86 / 55, 18 / 29 (44 / 63)
// nor, just beyond the line, what would gain by it:  d = 32 H32 T500 (512) 9.2 / 8.2, 8.9 / 8.1, 7.1 / 7.5 (9.0 / 7.7);  d = 64 T2000 H12 (756) 32 / 26, 31 / 19, 9 / 14
//            (20 / 17.5);  d = 128 H37 T200 (259) 8.4 / 6.9
// At d = 32 a chain of 10 subtiles is not worth the rounds' barriers.
inline bool small_fwd_grid(long strips, int T, int d)
{
    if (T <= (d == 32 ? 320 : 64)) return false;
    const long least = T < 256 ? 256 : T < 512 || d == 128 ? 384 : 512;
    return strips <= std::max(least, d == 128 ? std::min(2L * T / 5, 704L) : std::min(3L * T / 8, 1000L));
}

// Its strips at d = 32 whose workgroups have four waves for the subtiles in place of eight, three of them to a CU in place of one: as four_waves().
// Blocks / eight / four waves, us, without m, none far, then a third, then all:
//            B1 H10 T2500 (790 strips) 7.1 / 13.1 / 7.9, 33 / 18.2 / 19.0, 33 / 26 / 20;  H10 T3000 (940) 7.0 / 14.3 / 10.5, 39 / 23.3 / 22.3, 39 / 34 / 27
// and not    H9 T2753 (783) none 13.0 / 7.6 of the strips, a third 17.4 / 20.5, all 27 / 21;  H7 T3000 (658) 6.9 / 10.5 / 7.3, 39 / 15.7 / 22.2, 39 / 26 / 22;  H7 T4096 (896) 7.0 / 14.3 / 10.2, 52 / 22 / 29, 52 / 40 / 33;  H5 T6000 (940) 7.1 / 14.6 /
//            10.5, 74 / 28 / 41, 75 / 57 / 47;  H1 T16384 (512) all 196 / 77 / 107
// At d = 64, two workgroups to a CU, and d = 128 (of two waves in place of four) far heads lose as much as near ones gain, or more: H10 T3000 d64 9.0 / 18.4 / 15.3,
// 45 / 27.9 / 29.2, 45 / 41 / 49;  H10 T2048 d128 12.8 / 17.5 / 16.0, 45 / 25 / 36, 45 / 38 / 53 (two_strips()).  Nor does the backward gain by two waves at d = 128: B1 H8
// T2000 37 / 45 / 34, 117 / 72 / 119, 118 / 88 / 122.
inline bool four_fwd_waves(long strips, int T) { return strips > std::max(768, 3 * (T / 10)); }

// Grids without m whose strips go two to a workgroup (fwd_two_kernel): near heads are bound by how many rounds of workgroups the chip takes, a CU having room for
// one, and were slower in strips than in blocks; a lone far strip's rounds take 10 to 15 % longer beside another's at d = 128, a third longer at d = 64, with
// six subtiles to a round in place of eight.  Blocks / one strip / two, us, none far, then a third, then all:
//   d = 64   B1 H12 T2080 (780 strips) 8.8 / 15.9 / 11.6, 32 / 19.5 / 19.2, 32 / 27 / 20;  H10 T2500 (790) 8.7 / 16.1 / 12.1, 38 / 22.4 / 22.4, 38 / 31 / 23;  H9 T2752 (774)
//            8.7 / 15.8 / 12.3, 41 / 21.3 / 24.3, 41 / 32 / 25;  H10 T3000 (940) 9.0 / 18.4 / 13.4, 45 / 27.8 / 26.3, 45 / 41 / 30;  H9 T3500 (990) 9.1 / 19.2 / 13.6,
//            52 / 28.3 / 29.8, 52 / 48 / 35
//   d = 128  H12 T1200 (456) 12.0 / 12.7 / 8.2, 28 / 16.7 / 18.5, 28 / 19 / 18;  H8 T2000 (504) 12.0 / 14.6 / 10.1, 43 / 24.4 / 27.7, 43 / 29 / 28;  H6 T2500 (474) 11.8 / 13.2 /
//            8.4, 53 / 28.4 / 32.4, 53 / 32 / 32;  H2 T8192 (512) 12.1 / 16.0 / 10.5, all 162 / 92 / 100
// and not    d = 64 H7 T3000 (658) 8.5 / 14.6 / 11.2, 44 / 19.9 / 25.8, 44 / 31 / 26;  H7 T3500 (770) 8.7 / 16.0 / 12.4, 51 / 23 / 30, 51 / 39 / 30;  H5 T6000 (940) 9.1 / 19.5 / 13.3,
//            85 / 35 / 47, 86 / 69 / 52;  d = 128 beyond two rounds of single strips, where near heads gain less: H9 T2000 (567) 12.3 / 16.5 / 14.9, 43 / 24.7 / 28.2, 44 / 36 / 30;
//            nor where strips were always faster than blocks, H12 T1000 (384) 14.0 / 11.3 / 7.6, 16.9 / 14.2 / 15.3, 17.7 / 14.5 / 15.7;  d = 32 (four subtiles to a round)
//            H7 T3000 6.9 / 10.4 / 8.0, 39 / 15.7 / 24.9, 39 / 26 / 25
inline bool two_strips(long strips, int T, int d)
{
    return d == 128 ? strips > 384 && strips <= 512 : d == 64 && strips > std::max(768, T / 4);
}

// Grids of the key-stationary pass at d <= 64 whose blocks are taken by two groups of four waves (bwd_dkv_kernel<.., 2>): where a
// block has a CU to itself anyway (one wave per SIMD issues an instruction every five clocks at best, two keep it busy), and
// for some more blocks, of which few are left once some heads turn out near: what counts then is the longest block's chain.
// The limits lie where neither far heads nor near ones lose more by it than a mix gains.  One group / two, the whole backward, us,
// all heads far, then a third drawn at random (five times, mean), then none:
//   d = 64  B2 H16 T2048 (512 blocks) 130 / 121, 125 / 111, 46 / 51; B1 H36 T2011 (576) 139 / 139, 127 / 111, 52 / 61; B4 H8 T2500 (640)
//           169 / 176, 157 / 136, 59 / 67; B1 H24 T4096 (768) 331 / 345, 261 / 221, 63 / 71; B1 H27 T4096 (864) 338 / 347, 267 / 229, 74 / 87;
//           B1 H20 T6000 (940) 520 / 523, 393 / 352, 75 / 88; B1 H16 T8000 (1008) 706 / 723, 548 / 463, 78 / 90; B1 H32 T4096 (1024)
//           402 / 401, 289 / 270, 77 / 91; the least: B1 H30 T3500 (840) 284 / 308, 234 / 215, 71 / 85
//     not   B8 H16 T512 (512, 4 a head) this pass 25 / 29, 24 / 29, 23 / 28; B1 H48 T1499 (576, 12) 106 / 111, 99 / 93, 52 / 60; B1 H50 T1600 (650, 13)
//           116 / 124, 106 / 100, 56 / 64; B1 H40 T2048 (640, 16) 148 / 154, 131 / 120, 58 / 66
//   d = 32  B1 H16 T4096 (512) this pass 115 / 92, 114 / 84, 17 / 20; B1 H24 T4096 (768) 236 / 253, 225 / 187, 45 / 51; B5 H5 T4500 (900)
//           292 / 309, 240 / 207, 53 / 62; B1 H16 T8000 (1008) 523 / 563, 488 / 397, 55 / 64;  not B1 H43 T3035 (1032) 225 / 251, 194 / 175, 55 / 64
// Grouped heads, whose blocks are G times as long, up to 512:
//   d = 64  B1 H48 Hkv24 T2011 (384) 227 / 202, 195 / 164, 67 / 74; B8 H16 Hkv4 T1500 (384) 292 / 246, 264 / 211, 114 / 121; B12 H9 Hkv3
//           T1500 (432) 233 / 205, 207 / 168, 95 / 102; B1 H32 Hkv8 T8000 (504) 1602 / 1407, 1242 / 951, 139 / 142; B16 H16 Hkv2 T1200 (320)
//           442 / 362, 176 / 183, 177 / 185;  not B12 H9 Hkv3 T3256 (936) 832 / 832, 490 / 559, 177 / 200
//   d = 32  B2 H24 Hkv12 T2048 (384) 168 / 144, 158 / 132, 54 / 56; B4 H12 Hkv4 T4000 (512) 487 / 430, 423 / 343, 83 / 86
// A packed batch's blocks are counted by its rows (in brackets; every third head far):
//   d = 64  4500 and 30 of 50 rows, H8 (375) 343 / 279, 261 / 226, 62 / 81; four of 2000, H8 (500) 128 / 119, 126 / 110, 46 / 53; 2500 to 100, H12
//           (562) 192 / 172, 165 / 142, 60 / 72; 6000 and three of 200, H12 (618) 418 / 414, 386 / 330, 60 / 70; two of 4000, H12 (750) 282 / 301,
//           248 / 212, 61 / 72; six of 100 to 3000, H24 Hkv6 (248) 500 / 401, 477 / 377, 110 / 115; the worst: 4200 and three of 800, H8 (412)
//           246 / 304, 244 / 210, 51 / 69;  not four of 2000, H12 (750) 158 / 169, 138 / 129, 62 / 71; six of 1500, H9 (632) 110 / 122, 101 / 97, 59 / 69
//   d = 32  4500 and 30 of 50 rows, H8 (375) 297 / 233, 218 / 190, 50 / 69; two of 4000, H12 (750) 227 / 244, 213 / 180, 45 / 54
// and not for many short ones (64 of 32 rows, H4 d64, T 511, this pass 9.9 / 12.9) nor very many, whose empty places cost two groups
// more (5000 and 300 of 16, H2 d64, 77 / 117 with none far).
constexpr long ONE_PER_CU = 256;          // workgroups of a launch that leaves none waiting for a CU
inline bool take_in_turn(int B, int H, int Hkv, int T, bool packed, int Ttot)
{
    const long heads = (long)B * Hkv, nkb = (T + 127) / 128;
    if (packed) {
        if (heads > 256) return false;
        if (pieces(B, Hkv, T, 128, true, Ttot) <= ONE_PER_CU) return true;
        if (Ttot <= 64L * B) return false;
    }
    const long blocks = packed ? ((long)Hkv * Ttot + 127) / 128 : heads * nkb;
    const long limit = std::max(ONE_PER_CU, std::min(48 * nkb, 512L));
    return blocks <= (H == Hkv ? std::max(limit, std::min(36 * nkb, 1024L)) : limit);
}

// Grids of the key-stationary pass at d = 128 that take 64 keys a block in place of 128: what bounds a launch there is one
// block's chain of intervals, and with one wave per SIMD in place of two an interval is shorter.  Where the 128-key blocks
// outnumber the CUs this costs more rounds than it saves, except with long chains and heads of mixed
// reach.  Key-stationary pass with 128 / 64 keys a block, us, all heads far, then a third:
//   up to 256 blocks   B1 H20 T1024 (160) 40 / 31, 40 / 31; B1 H16 T2048 (256) 69 / 64, 67 / 50;
//                      B8 H16 T256 (256) 33 / 28, 33 / 27; B1 H8 T4096 (256) 123 / 108, 120 / 88
//   more, short heads  B2 H20 T1024 (320) 44 / 56, 42 / 46; B2 H16 T1280 (320) 50 / 62, 48 / 47;
//                      B3 H32 T512 (384) 39 / 48, 39 / 47; B1 H24 T2048 (384) 78 / 97, 68 / 70
//   more, long heads   B1 H20 T2048 (320) 71 / 83, 68 / 58; B1 H16 T3072 (384) 105 / 128, 94 / 79;
//                      B1 H12 T4096 (384) 138 / 164, 121 / 89; B1 H3 T16384 (384) 499 / 579, 439 / 318
//   beyond             B1 H14 T4096 (448) 152 / 185, 121 / 105; B1 H16 T4096 (512) 172 / 209, 121 / 116
constexpr long small_kv_grid(int nkb) { return std::clamp(64L + 16L * nkb, 256L, 384L); }

// Strips of the backward at d <= 64 whose workgroups have four waves in place of eight: two (d = 64) or three (d = 32) share a CU.  A near
// strip has two or three tiles and keeps no more waves busy, whatever there are; a far one's chain takes twice the rounds, which counts until
// there are two of them for every CU.  Whole step, eight / four waves, us, none far, then a third, then all:
//   d = 32   B1 H21 T993 (672 strips) 41 / 29, 45 / 40, 49 / 41;  B1 H12 T4096 (1536) 85 / 60, 148 / 127, 212 / 189 (two a CU, as all figures of all heads far but the first);  B5 H2 T3480 (1090) 70 / 51, - , 150 / 137;
//            B1 H9 T4096 (1152) 75 / 59 (two a CU), 124 / 125, 176 / 163
//   d = 64   B1 H21 T993 51 / 45, 55 / 52, 64 / 57;  B1 H14 T2500 (1106) 83 / 69, 122 / 108, 156 / 142
// and not    d = 32 B1 H10 T2100 (660) 43 / 34, 56 / 63, 71 / 67;  B1 H8 T2000 (504) all 51 / 58;  d = 64 B1 H12 T900 (348) all 35 / 41
// From 768 to 1024 strips, where there was one block kernel before there were strips so long, which near heads alone are faster in, the backward
// with blocks / eight / four waves:
//   d = 32   B1 H14 T2048 (896) 25 / 37 / 25, 88 / 46 / 43, 89 / 63 / 49;  B1 H10 T2500 (790) 24 / 34 / 20, 107 / 46 / 50, 108 / 64 / 55;  B1 H10 T2800 (880)
//            25 / 37 / 24, 119 / 53 / 54, 119 / 75 / 63
//   d = 64   B1 H14 T2048 32 / 48 / 35, 107 / 58 / 56, 108 / 84 / 78;  B1 H10 T2500 31 / 45 / 34, 130 / 59 / 64, 130 / 85 / 81;  B1 H12 T2600 (984) 32 / 49 / 38,
//            134 / 68 / 68, 135 / 108 / 99
// and not    d = 32 B1 H9 T2900 (819) 24 / 35 / 23, 122 / 46 / 56, 123 / 72 / 63;  d = 64 32 / 46 / 36, 148 / 58 / 73, 148 / 95 / 91:  the more of a strip's subtiles to
// a wave of eight, the more a lone far head's longest chain counts
// The key-stationary pass of grouped heads, whose chains are G times as long: B2 H36 Hkv12 T1750 d64 (1320) 120 / 116, 180 / 175;  B8 H16 Hkv4 T1500 d32
// (1504) 113 / 108 (two a CU), 184 / 171, d64 all 333 / 310;  not B1 H33 Hkv11 T3870 d32 (1331) 114 / 108, 278 / 307;  B1 H24 Hkv12 T3000 d64 (1128) 96 / 89, 185 / 194;  B4 H32
// Hkv4 T800 d32 (800) all 82 / 104
inline bool four_waves(long strips, int G, int mean, int d)
{
    if (d == 128) return false;
    return strips > (G > 1 ? std::max(1280, 5 * (mean / 8)) : mean > 1024 ? std::clamp(3 * (mean / 10), 768, 1024) : 640);
}

// The kernels of the backward's passes.
inline bool query_strips(int B, int H, int T, int d, bool packed, int Ttot)
{
    return small_grid(pieces(B, H, T, 32, packed, Ttot), T, mean_T(B, T, packed, Ttot), d);
}
enum class Keys {
    STRIPS,                               // bwd_dkv_small_kernel
    ONE_GROUP, TWO_GROUPS,                // bwd_dkv_kernel, d <= 64
    KEYS_64, KEYS_128, PAIRS,             // bwd_dkv_pair_kernel, d = 128
};
inline Keys keys_of(int B, int H, int Hkv, int T, int d, bool packed, int Ttot)
{
    const long heads = (long)B * Hkv;
    const int nkb = (T + 127) / 128;
    const long blocks = pieces(B, Hkv, T, 128, packed, Ttot);
    const long strips = pieces(B, Hkv, T, 32, packed, Ttot);
    const int mean = mean_T(B, T, packed, Ttot);
    if (small_grid(strips, T, mean, d) || grouped_strips(strips, H / Hkv, T, mean, d)) return Keys::STRIPS;
    if (d < 128) return take_in_turn(B, H, Hkv, T, packed, Ttot) ? Keys::TWO_GROUPS : Keys::ONE_GROUP;
    if (blocks <= small_kv_grid(nkb)) return Keys::KEYS_64;
    return !packed && H == Hkv && take_pairs(heads, nkb) ? Keys::PAIRS : Keys::KEYS_128;
}

// The key-stationary pass of grouped heads where the workspace has room for parts (Parts in sb_bwd_bf16.hip): the query heads of a block of keys over `parts`
// workgroups, if the queries `beyond` strips further on attend to it.  One block's G heads are one chain, and where some kv heads reach far their blocks' chains are what the
// launch waits for.  A part costs its K, V and sums (4 to 5 us of a launch), and a workgroup that finds nothing to do next to nothing: what near heads lose is the question, and is lost where it
// takes them for far ones (16 strips, not 8, beyond a block of four; rows of N(0,1) reach 5 to 8: B6 H4 Hkv2 T5496 d64, none far, the pass 43 us in one part, 50 with parts from 8
// strips on, 43 with none taken).  So a part has to have a long chain, of 13 rounds of its workgroup's waves in blocks, 5 or 7 in strips, and there have to be few of them; where blocks fill the chip by
// themselves, parts only add traffic.  Drawn from 3000 shapes, each with up to twelve plans; 465 more that the rule changes are 34 % faster
// in the mean with a third of the kv heads far, 22 % with all, 8 % with none, at worst 3 %, 10 % and 8 % slower (B12 H6 Hkv2 T1638 d128 all 269 / 299, B4 H18 Hkv9 T486 d128 none 51 / 56).
// Whole backward in one part with the kernel that keys_of() names / as here, us, all heads far, then a third, then none (one kv head: all, none):
//   strips   d = 128 B1 H16 Hkv2 T2087 (132 strips) 290 / 200, 288 / 197, 68 / 56;  B1 H16 Hkv2 T1228 (78) 176 / 96, 175 / 93, 65 / 53;  B3 H4 Hkv1 T506 (48) 46 / 40, 30 / 31
//            d = 64 B1 H4 Hkv1 T1778 (56) 61 / 36, 18 / 19;  B2 H8 Hkv2 T1173 (148) 53 / 45, 51 / 42, 29 / 30;  packed H8 Hkv1, 5 up to 1402 (92) 93 / 67, 35 / 37
//            d = 32 B1 H2 Hkv1 T3942 (124) 68 / 54, 14 / 14;  B6 H8 Hkv1 T562 (108) 43 / 36, 32 / 29;  B1 H24 Hkv3 T1532 (144) 100 / 77, 99 / 76, 34 / 30
//     not    more strips, d = 128 B3 H4 Hkv2 T1010 (192) 72 / 72, 72 / 69, 37 / 39;  packed H3 Hkv1, 18 up to 884 (148) 76 / 70, 42 / 52;  H2 Hkv1, 24 up to 978 (229) 72 / 77, 39 / 46;  B12 H8 Hkv2 T445 (336) 58 / 65, 57 / 63, 53 / 60;
//            d = 64 B5 H16 Hkv4 T426 (280) 35 / 39, 34 / 38, 31 / 35;  B2 H4 Hkv2 T2964 (372) 87 / 98, 83 / 93, 36 / 38;  d = 32 B11 H4 Hkv2 T382 (264) 20 / 24 in all three;  B5 H16 Hkv2 T1116
//            (350) 81 / 88, 79 / 71, 45 / 49;  but packed H8 Hkv1 d64, 5 up to 4989 (314) 369 / 298, 66 / 63
//   blocks   d = 128 B4 H12 Hkv4 T2048 (256 blocks) 274 / 260, 212 / 188, 115 / 113;  B3 H6 Hkv3 T2068 (153) 170 / 158, 170 / 153, 70 / 62;  B1 H15 Hkv5 T7819 (310) 1194 / 1033, 763 / 533, 147 / 141;  packed H32 Hkv4, 17
//            up to 3498 (476) 1269 / 1031, 1036 / 668, 452 / 451
//            d = 64 B3 H12 Hkv3 T6024 (432) 980 / 886, 795 / 512, 126 / 122;  B5 H8 Hkv4 T3497 (560) 398 / 358, 338 / 258, 88 / 90;  packed H32 Hkv8, 18 up to 2778 (776) 615 / 506, 469 / 310, 174 / 180
//            d = 32 B2 H14 Hkv7 T5822 (644) 550 / 493, 481 / 375, 74 / 73
//     not    d = 128 of one length beyond 320, B15 H8 Hkv2 T1651 (390) 405 / 470, 340 / 329, 205 / 200;  B3 H24 Hkv12 T2658 (756) 619 / 686, 388 / 413, 196 / 193;  but B2 H32 Hkv8 T3741 (480) 994 / 1070,
//            625 / 473, 234 / 225;  shorter ones, B8 H22 Hkv11 T786 194 / 224, 148 / 154, 145 / 147
//            d = 64 and 32 where parts are more than 2300, packed H14 Hkv7 d64, 23 up to 3688 (1477) 633 / 698, 392 / 321, 181 / 184;  B13 H22 Hkv11 T1364 d64 (1573) 435 / 511, 246 / 268, 186 / 188;  shorter ones, B3
//            H20 Hkv10 T928 d64 80 / 90, 80 / 89, 48 / 53;  at d = 32 blocks that are all on the chip at once, or nearly, B7 H4 Hkv2 T4514 (504) 341 / 354, 298 / 322, 61 / 63;
//            B5 H6 Hkv2 T6568 (520) 818 / 664, 774 / 559, 82 / 90
// Strips in one part where keys_of(), whose rule was made for batches of one length, takes blocks, packed ones going by their mean:
//            d = 32 H18 Hkv6, 13 up to 584 (480 strips) 61 / 34, 60 / 34, 43 / 29;  H32 Hkv4, 36 up to 3601 (2320) 990 / 477, 876 / 370, 203 / 170;  H32 Hkv16, 10 up to 4234 (4352) 425 / 375, 348 / 234, 101 / 94
//            d = 64 H8 Hkv4, 22 up to 632 (524) 61 / 44, 61 / 43, 44 / 35;  H24 Hkv6, 12 up to 4443 (1704) 614 / 459, 547 / 359, 136 / 108;  H21 Hkv7, 28 up to 1028 (1897) 157 / 122, 151 / 110, 92 / 94
//            d = 128 H14 Hkv7, 5 up to 474 (336) 57 / 47, 57 / 47, 50 / 44;  H12 Hkv3, 4 up to 3798 (720) 470 / 412, 457 / 339, 139 / 108
//            of one length, d = 128 B3 H18 Hkv9 T462 (405) 57 / 49, 57 / 48, 48 / 46;  B3 H14 Hkv7 T940 (630) 93 / 96, 92 / 80, 63 / 60;  not B13 H18 Hkv9 T169 (702) 44 / 47 in all three
// The first parts' workgroups come behind those that may have nothing to do: before them, packed H14 Hkv7 d64, 33 up to 1942 164 / 186, 144 / 170, 93 / 107.
struct KeyPlan {
    Keys keys;
    int parts, beyond;
};
// bytes of `parts` sums of `rows` rows (of all kv heads) and of the counts of `heads` kv heads of up to T rows
inline size_t part_bytes(int parts, size_t rows, size_t heads, int T, int d)
{
    return parts > 1 ? 2 * sizeof(float) * parts * rows * d + sizeof(int) * heads * ((T + 31) / 32) : 0;
}
constexpr size_t MOST_PART_BYTES = 210u * 1000 * 1000 - 16;      // (with what rounds the rest up to 16, what the header says)
inline KeyPlan key_plan(int B, int H, int Hkv, int T, int d, bool packed, int Ttot)
{
    const int G = H / Hkv, mean = mean_T(B, T, packed, Ttot);
    const long strips = pieces(B, Hkv, T, 32, packed, Ttot), blocks = pieces(B, Hkv, T, 128, packed, Ttot);
    KeyPlan p = {keys_of(B, H, Hkv, T, d, packed, Ttot), 1, 0};
    if (G == 1) return p;
    // the most parts of which each has a chain of `rounds` rounds of its waves
    const size_t rows = packed ? (size_t)Hkv * Ttot : (size_t)B * Hkv * T;
    auto most = [&](long pieces, long limit, int rounds) {
        const long chain = (long)G * ((T + 31) / 32), waves = d == 128 ? 4 : 8;
        int n = 1;
        for (int x = 2; x <= std::min(G, 8); ++x)
            if (G % x == 0 && pieces * x <= limit && chain >= rounds * waves * x && part_bytes(x, rows, (size_t)B * Hkv, T, d) <= MOST_PART_BYTES) n = x;
        return n;
    };
    const bool lengths = packed && packed_as(B, T, Ttot) == Packed::BY_LENGTH, fit = mean > 64 && T <= LONG_T;
    if (p.keys != Keys::STRIPS && lengths && fit && strips <= (d == 32 ? 5120 : d == 64 ? 2048 : 768)) {
        p.keys = Keys::STRIPS;
    } else if (p.keys != Keys::STRIPS && T >= 1000 && (d == 32 ? blocks > 560 : d == 64 || lengths || blocks <= 320)) {
        p.parts = most(blocks, d == 128 ? 1024 : 2300, 13);
        p.beyond = 16;
        if (p.parts > 1) p.keys = d == 128 ? Keys::KEYS_128 : Keys::ONE_GROUP;
    }
    if (p.parts == 1 && d == 128 && !lengths && fit && T > 400 && strips <= 768) p.keys = Keys::STRIPS;
    if (p.keys == Keys::STRIPS && T > 400 && strips <= 144) {
        p.parts = most(strips, d == 128 ? 512 : 320, d == 128 ? 5 : 7);
        p.beyond = 8;
    }
    return p;
}

// log2 of the run, -1: turn with every block.  A run pays where the launch is several rounds deep and
// there are enough runs to even the XCDs out: 32 of them, or 16 where 64 heads and more can be turned
// among each other as well, by o(o+1)/2 inside each octet o of heads (over octets 8x to 8x + 7 these are all 8
// turns, so that heads which are costly in every batch entry do not meet on one XCD).  Query heads that
// share a kv head, where runs win 10 to 30 % or lose as much by which heads are far, and packed batches, where a run is cut short by the
// sequences' ends, turn with every block.
// Every block / runs, us, all heads far, then a third, then none: forward B8 H16 T4096 d128 698 / 669,
// 331 / 329, 160 / 150; B1 H32 T16384 d128 2422 / 2266, 883 / 880, 165 / 154; B1 H24 T16384 d64 1078 / 1032,
// 460 / 422, 65 / 56; query-stationary backward of the same three 1049 / 1032, 524 / 530, 309 / 304;
// 3849 / 3762, 1410 / 1433, 319 / 312; 1828 / 1780, 774 / 725, 139 / 134.  Runs twice as long are
// another 1 % faster where all heads reach far and up to 20 % slower where a third does (B8 H16 T4096: 393 us).
// Smaller launches and odd head counts lose up to 20 % (B1 H27 T8192 d128: 224 / 284 with a third far).
inline int share_run(long heads, int nblk)
{
    if (heads % 8 != 0 || heads * nblk < 1536 || nblk < (heads < 64 ? 64 : 32)) return -1;
    int run = 1;
    while (nblk >> (run + 1) >= 32) ++run;
    return run;
}
// The forward and the query-stationary pass take runs in shorter launches too: blocks that sweep the same tiles one tile apart meet in
// an L2, and a far head's blocks no longer come at the same CUs in every round of the launch.
// Every block / runs of 2 (below 64 heads from 24 blocks on of 4), us, forward with m, then this pass, every third head far, a third drawn at random, all far:
//   from 64 heads    B8 H16 T2048 d64 84 / 81, 87 / 81, 102 / 99 and 95 / 93, 103 / 95, 169 / 166 (of the whole step, one third far, 2 of 314);  B4 H24 T1024 d128 43 / 40,
//                    43 / 40, 44 / 42 and 51 / 49, 51 / 49, 64 / 62;  B5 H16 T1500 d128 61 / 57, 63 / 57, 70 / 67 and 71 / 67, 73 / 69, 106 / 102;  the worst: B10 H16
//                    T3000 d64 206 / 207, 206 / 205, 268 / 264 and 224 / 230, 233 / 234, 457 / 450
//   fewer            B2 H24 T4096 d64 114 / 105, 114 / 108, 144 / 137 and 164 / 129, 163 / 149, 240 / 236;  B4 H8 T4096 d32 75 / 59, 74 / 60, 77 / 76 and
//                    122 / 90, 123 / 91, 130 / 129;  B3 H8 T6000 d64 122 / 118, 112 / 104, 154 / 147 and 179 / 174, 155 / 154, 257 / 250;  B2 H20 T2500 d64
//                    (of 2) 50 / 47, 51 / 47, 55 / 55 and 74 / 70, 77 / 70, 89 / 88;  B1 H32 T4096 d128 (of 2) 129 / 119, 127 / 126, 168 / 162 and 164 / 146,
//                    164 / 160, 266 / 260, of 4 121, 129, 157 and 145, 181, 251;  B1 H24 T12000 d32 (of 2 / of 4) 313 / 305, 318 / 303, 408 / 401 and
//                    417 / 354, 488 / 397, 742 / 730, but B1 H24 T8192 d128 319 / 317, 327 / 314, 450 / 443 and 361 / 359, 352 / 360, 720 / 712
// Whose heads are far counts for as much: over 76 shapes with a third of them drawn at random the forward is 4 % faster in the mean, the whole backward 1 %, single
// ones from 9 % slower (B1 H40 T6000 d32) to 15 % faster.  This pass not at d = 64 with 64 to 127 heads, backward, every third far, at random, all, none: B6 H12 T2307
// 164 / 179, 189 / 188, 291 / 289, 94 / 95; B10 H8 T2307 180 / 190, 189 / 199, 319 / 316, 99.5 / 98; B8 H11 T1500 110 / 114, 123 / 120, 165 / 161, 74 / 73; B9 H8 T1800
// 121 / 134, 137 / 139, 194 / 190, 74 / 74 (the forward there 45.2 / 45.2, 45.2 / 45.9, 52 / 51, 41 / 36).
// Not at d = 32 from 64 heads on, where tiles are small (B8 H16 T2048 59 / 59, 61 / 59, 71 / 72 and 69 / 73, 78 / 77, 127 / 124), with fewer than 8 blocks (B8 H24
// T700 d64, this pass, at random, 37 / 39), nor for the key-stationary pass, whose blocks outnumber their places less (B4 H8 T4096 d32, runs of 4, 84 / 90).
inline int query_run(long heads, int nblk, int d, bool backward)
{
    if (heads % 8 != 0 || heads * nblk < 768 || nblk < 8) return -1;
    if (nblk >= 64) return std::max(share_run(heads, nblk), heads < 64 && d < 128 ? 2 : 1);
    if (heads >= 64) return d == 32 || (d == 64 && backward && heads < 128) ? share_run(heads, nblk) : 1;
    return nblk >= (d == 128 ? 40 : 24) ? 2 : 1;
}

// (unsigned: a division is half as long)
__host__ __device__ __forceinline__ Share share_in_pairs(unsigned wg, int nblk)     // bh >= heads: nothing to do
{
    const unsigned npair = (unsigned)(nblk + 1) >> 1;
    const unsigned slot = wg >> 3, s = slot / npair;
    return {(int)(8 * s + ((wg + ((s * (s + 1)) >> 1)) & 7)), (int)(slot - s * npair)};
}

__host__ __device__ __forceinline__ Share share_of(unsigned wg, unsigned heads, int run)
{
    const unsigned i = wg / heads, w = wg - i * heads;
    if (run < 0) {
        // (two or four heads that turn by one with every block meet four of the XCDs each: one far head of four, d = 64, T 8192, in strips, forward
        // 94 -> 59 us, backward 235 -> 150)
        const unsigned t = heads <= 4 ? i + (i >> 2) : i;
        return {(int)((heads & 1) ? w : w + t < heads ? w + t : (w + t) % heads), (int)i};
    }
    const unsigned turn = i >> run;                           // heads a multiple of 8 from here on
    if (heads < 64) return {(int)(w + turn < heads ? w + turn : (w + turn) % heads), (int)i};
    const unsigned o = w >> 3;
    return {(int)(8 * o + ((w + turn + ((o * (o + 1)) >> 1)) & 7)), (int)i};
}

// Orders of the fp32 forward, 16 rows a block.  The longest rows of all heads come first, over all XCDs; heads in eights stay on one XCD each, whose L2 then holds their K and V.  In
// short launches, whose blocks are all on the chip at once or wait for one of the shortest, and where the L2s do not hold K and V of heads that go round the XCDs, each XCD takes
// a contiguous eighth of the (head, rows) list in place, and with it one or two heads.  In eighths / longest first, us, inputs in turn from six sets:
//   short          d = 128 H28 T117 (224 blocks) 7.2 / 8.0;  H18 T183 (216) 10.1 / 11.2;  H12 T350 (264) 14.4 / 15.4;  H7 T471 (210) 16.9 / 17.5;  d = 64 H15 T213 (210) 6.9 / 7.3;  d = 32 H15 T250 (240) 5.6 / 5.9
//     not          d = 128 H10 T419 (270) 18.5 / 16.1 (inputs in L2);  d = 64 H5 T870 (275) 18.7 / 15.8;  H10 T401 (260) 13.6 / 10.2;  d = 32 H9 T471 (270) 11.3 / 7.9;  B1 H3 T1984 37 / 27
//   K and V        d = 128 H18 T1206 (22 MB) 114 / 120;  H14 T1911 (27 MB) 187 / 215;  H28 T1944 (56 MB) 377 / 469;  d = 64 H28 T1504 (22 MB) 124 / 128;  H28 T1737 (25 MB) 157 / 175
//     not          d = 128 H10 T1928 (19.7 MB) 167 / 149;  H14 T695 (10 MB) 41 / 37;  d = 64 H20 T1958 (20 MB) 146 / 143;  H14 T1797 (13 MB) 97 / 82;  in eights, d = 128 H16 T1668 (27 MB) 159 / 156;  d = 64 H24
//                  T1948 (24 MB) 149 / 143 (B4 H8 T2048 turning 301 us, d = 128 610)
constexpr int EIGHTHS = -2;
inline int f32_run(long heads, int nblk, int T, int d)
{
    if (heads * nblk <= 264) return EIGHTHS;
    return heads % 8 == 0 ? 31 : 8.0 * heads * T * d > 20e6 ? EIGHTHS : -1;
}
__host__ __device__ __forceinline__ Share share_in_eighths(unsigned wg, unsigned heads, unsigned nblk)     // bh >= heads: nothing to do
{
    const unsigned all = heads * nblk, at = (wg & 7) * ((all >> 3) + ((all & 7) != 0)) + (wg >> 3), bh = at / nblk;
    return {(int)(at < all ? bh : heads), (int)(at - bh * nblk)};
}

// the divisions above pass through vector registers: back into scalar ones, and with it everything
// that a kernel derives from its share
__device__ __forceinline__ Share in_scalars(Share s)
{
    return {__builtin_amdgcn_readfirstlane(s.bh), __builtin_amdgcn_readfirstlane(s.i)};
}

// A sequence of n blocks has one of every length 1 .. n (the forward's and the query-stationary pass's chains run to its first row, the
// key-stationary pass's to its last), block i from the long end one of n - i.  So sum_s max(n_s - x, 0) blocks are longer than x; a bisection
// over x finds the length of the one at `place`, its rank among those of that length the sequence.  Up to 256 sequences,
// four to a lane; with more, sequence by sequence (place_of()).
template <int ROWS>
__device__ __forceinline__ Place longest_first(int place, const int* __restrict__ cu, int nseq, int Ttot, int T_arg, int lane)
{
    constexpr int MOST = 4;
    if (nseq > 64 * MOST) return place_of<ROWS>(place, cu, nseq, Ttot, T_arg, lane);
    int c0[MOST], T[MOST], n[MOST];
#pragma unroll
    for (int b = 0; b < MOST; ++b) {
        n[b] = 0;
        if (64 * b >= nseq) continue;
        const int s = min(64 * b + lane, nseq - 1);
        c0[b] = cu[s];
        const int c1 = min(cu[s + 1], Ttot);
        T[b] = 64 * b + lane < nseq && c0[b] >= 0 && c1 > c0[b] ? min(c1 - c0[b], T_arg) : 0;
        n[b] = (T[b] + ROWS - 1) / ROWS;
    }
    auto longer = [&](int x) __attribute__((always_inline)) {
        int sum = max(n[0] - x, 0);
#pragma unroll
        for (int b = 1; b < MOST; ++b)
            if (64 * b < nseq) sum += max(n[b] - x, 0);
        return __builtin_amdgcn_readlane(sum_up_to_lane(sum), 63);
    };
    int x = 0, behind = 0;                              // more than `place` blocks are longer than x, `behind` of them longer than x + 1
    if (longer(0) <= place) return {0, 0, 0, 0};
    for (int step = 1 << (31 - __builtin_clz((T_arg + ROWS - 1) / ROWS)); step > 0; step >>= 1) {
        const int more = longer(x + step);
        if (more > place) x += step;
        else behind = more;
    }
    int rank = place - behind;
    Place at = {0, 0, 0, 0};
#pragma unroll
    for (int b = 0; b < MOST; ++b) {
        if (64 * b >= nseq) continue;
        const unsigned long long has = __builtin_amdgcn_ballot_w64(n[b] > x);
        const int before = __builtin_amdgcn_mbcnt_hi((unsigned)(has >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)has, 0));
        const unsigned long long it = __builtin_amdgcn_ballot_w64(n[b] > x && before == rank);
        if (it) {
            const int l = __builtin_ctzll(it);
            at = {64 * b + l, __builtin_amdgcn_readlane(n[b], l) - 1 - x, __builtin_amdgcn_readlane(c0[b], l), __builtin_amdgcn_readlane(T[b], l)};
        }
        rank -= __builtin_popcountll(has);              // (below 0 once it is found)
    }
    return at;
}
// Heads of a packed batch whose blocks are looked up by length, in turn with every fourth block.  Eight, sixteen or twenty-four heads that turn with every block
// meet every XCD; turning with every fourth, neighbouring blocks of a sequence, which sweep the same tiles, meet on one.  With every block / every
// fourth, a third of the heads far, backward, us: H8 d64, longest 5000 413 / 373, d128 622 / 539, longest 2048 d128 197 / 189; H16 d64, longest 5000 708 / 685; H24
// d128, longest 2048 520 / 508, others of 16 and 24 heads alike.  Not for more (H32 d64 434 / 458, 1340 / 1374, d128 651 / 674), nor for other numbers,
// which change their XCD with every block anyway (H9 d128 653 / 753, H13 963 / 1075, H11 252 / 262; H6, H10 and H14 alike or 1 to 2 % slower; H12 d32, 24 up to 1500
// 84 / 90), nor where query heads share a kv head, whose tiles they find on any (H32 Hkv4 d64 1700 / 1840).
__host__ __device__ __forceinline__ bool turn_with_every_fourth(int H, int G) { return G == 1 && H % 8 == 0 && H <= 24; }
// Workgroup wg's block: its head in `head`, its sequence and the rest in the result (T = 0: none).  H heads, G of which share keys and values
template <int ROWS, bool BY_LENGTH>
__device__ __forceinline__ Place block_of(int& head, unsigned wg, int H, int G, const int* __restrict__ cu, int nseq, int Ttot, int T_arg, int lane)
{
    if constexpr (BY_LENGTH) {
        Share sh = share_of(wg, H, -1);
        if (turn_with_every_fourth(H, G)) sh.bh = (wg + (sh.i >> 2)) % (unsigned)H;
        sh = in_scalars(sh);
        head = sh.bh;
        return longest_first<ROWS>(sh.i, cu, nseq, Ttot, T_arg, lane);
    } else {
        const Share sh = in_scalars(share_of(wg, nseq * H, -1));
        const int seq = sh.bh / H, c0 = cu[seq], T = min(min(cu[seq + 1], Ttot) - c0, T_arg);     // never past the packed rows or the stated maximum
        head = sh.bh - seq * H;
        return {seq, sh.i, c0, c0 >= 0 && sh.i * ROWS < T ? T : 0};
    }
}

}  // namespace sb
