// How a decode call's keys are split over workgroups.
#pragma once
#include <algorithm>

namespace sb {

constexpr int NEAR_NW = 8;             // waves of a workgroup, first launch
constexpr int FAR_NW = 4;              // and second: smaller, so that two or three share a CU
constexpr int KW = 32;                 // keys per wave and pass
constexpr int NEAR = KW * NEAR_NW;     // keys of a first launch that has a second one behind it
constexpr int ALONE = 6 * NEAR;        // a cache that is not spread is the first launch's alone up to here (alone_up_to())
constexpr int MAXFAR = 127;            // chunks beyond the nearest keys: with those, two per lane of a wave
constexpr int FAR_KEYS = KW * FAR_NW;  // keys of a pass of the second launch
constexpr long FAR_WGS = 4096;         // workgroups of the second launch, all heads together (2048 / 4096 / 8192, a third of the heads far: B8 H16
                                       // T16384 d128 69 / 63 / 62 us, B32 H16 T1800 d64 29.7 / 27.5 / 27.5; all far 167 / 164 / 167, 44 / 44 / 43)
constexpr long ALL_WGS = 8192;         // the same where it takes all keys (see split_of())

// Partial results there is room for in decode_workspace_bytes: one per 64 keys, or per 64 * 2^i where
// those would be more than 256.
inline int room(int T)
{
    int C = 64;
    while ((T + C - 1) / C > 256) C *= 2;
    return (T + C - 1) / C;
}

// A cache that is not spread is the first launch's alone where its passes take no longer than the two other launches, whose latencies
// near heads have for nothing.  Alone / three launches, us, no head far, then a third, then all:
//   d = 32   B24 H24 Hkv8 T2048 5.5 / 11.6, 12.0 / 13.4, 12.3 / 18.2;  B30 H10 T2048 6.0 / 12.0, 15.9 / 17.2, 16.8 / 21.8;  B32 H16 T2048 7.0 / 11.7, 17.7 / 20.7,
//            26.5 / 28.9;  not B30 H10 T2560 5.7 / 11.6, 19.0 / 16.9, 20.3 / 24.1
//   d = 64   B24 H24 Hkv8 T2048 6.3 / 11.7, 16.1 / 17.7, 21.1 / 24.9;  B13 H16 T2048 5.2 / 12.1, 15.9 / 18.7, 17.8 / 24.7;  B16 H16 T2048 7.1 / 12.1, 18.6 / 19.4,
//            25.5 / 28.6;  not beyond a round of the chip:
//            B32 H16 T2048 11.4 / 13.6, 32.7 / 29.1, 47.1 / 47.9, nor where few workgroups leave the far keys' launch room: B12 H12 T1800 5.3 / 9.6,
//            15.0 / 13.5, 16.0 / 18.4
//   d = 128  not B16 H16 T2048 11.7 / 13.7, 32.8 / 30.3, 46.9 / 48.5
inline int alone_up_to(long wgs, int d)
{
    return (d == 32 && wgs <= 512) || (d == 64 && wgs >= 192 && wgs <= 256) ? 8 * NEAR : ALONE;
}

// A small cache is spread over the chip, every key read: one workgroup a head is bound by what one CU can load (per pass
// of 256 keys 2.6 us at d = 128, 1.7 at d = 64, 1.4 at d = 32), three launches by their latencies.  Two launches take 6.2, 6.5
// and 7.4 us and 0.1 us per MB of the cache.  Where m is wanted every key is read anyway.  Without m one workgroup ends with
// the pass that uses up the stick, and where that is the first in every head it is faster; how many heads end there is not
// known here.  The limits lie where what is lost then is at most two thirds of what is gained where a third of the kv heads reach far.
// One workgroup a head (beyond 1536 keys three launches) / spread, us, no head far, then a third, then all:
//   d = 128  B1 H12 Hkv4 T520 6.7 / 7.6, 10.2 / 7.6, 10.4 / 7.5; T1500 6.7 / 7.8, 18.0 / 7.8, 18.4 / 7.7
//            B4 H8 T1000 (16 MB) 6.8 / 8.0, 12.8 / 8.0, 13.0 / 8.1; B4 H8 T1500 (25 MB) 6.7 / 9.8, 17.8 / 9.9, 18.0 / 10.0
//     not    B5 H30 Hkv10 T700 (18 MB) 7.0 / 10.0, 10.7 / 10.0; T1000 (26 MB) 7.0 / 10.2, 13.5 / 10.3; B8 H16 T1280 6.8 / 17.4, 16.7 / 17.4
//   d = 64   B2 H8 T1280 4.6 / 6.6, 10.7 / 6.5, 10.8 / 6.5; T1500 4.6 / 6.5, 12.3 / 6.5, 12.4 / 6.6
//     not    B2 H8 T1000 4.6 / 6.5, 9.1 / 6.5; B4 H8 T1280 (11 MB) 4.6 / 7.4, 10.7 / 7.6; B5 H30 Hkv10 T1000 (13 MB) 4.8 / 7.8, 9.6 / 7.8
//   d = 32   B2 H8 T1500 3.9 / 6.4, 10.7 / 6.5, 10.8 / 6.5;  not T1280 3.8 / 6.4, 9.3 / 6.4
//   beyond   B1 H4 T2000 d64 9.0 / 6.1, 12.0 / 6.4; B4 H8 T2000 d128 (33 MB) 9.3 / 10.1, 15.5 / 10.2, 16.6 / 10.2; B8 H8 T2000 d64 (33 MB) 9.2 / 10.1,
//            14.0 / 10.3; beyond alone_up_to() B6 H20 T2560 d32 (39 MB) 11.6 / 11.3, 14.6 / 11.6, 15.5 / 11.4, B4 H16 T2560 d64 (42 MB) 12.3 / 11.7, 15.9 /
//            11.9, 16.5 / 11.4;  not B8 H8 T3000 d64 (49 MB) 9.2 / 12.4, 14.3 / 12.5; B2 H16 T6000 d128 (98 MB) 9.2 / 19.3, 19.8 / 19.4
inline bool spread_small(long wgs, double cache_bytes, int T, int d, bool want_m)
{
    const int passes = (T + NEAR - 1) / NEAR;
    if (passes <= 2) return false;
    if (want_m) return cache_bytes <= std::min(34e6, 12e6 * (passes - 2));
    if (T > ALONE) return cache_bytes <= (T > alone_up_to(wgs, d) ? 45e6 : 34e6);
    if (d == 128) return cache_bytes <= 5.5e6 * (passes - 1);
    return passes >= (d == 64 ? 5 : 6) && cache_bytes <= 8e6;
}

// The nearest keys in the first launch, the rest in nfar chunks of C, whole passes of
// either kernel.  With m wanted every key is read whatever the nearest ones take: they need no launch of
// their own, and as no workgroup is let off, more and smaller chunks even the CUs out.  With m, us: three
// launches / two with the same chunks / two with these: B16 H32 Hkv8 T4096 d128 55 / 49 / 48, B32 H16 T1800 d64
// 49 / 43 / 39, B1 H32 Hkv8 T65000 d128 53 / 46 / 46, B8 H16 T16384 d128 167 / 161 / 162, B1 H8 T2000 d64
// 12.8 / 9.4 / 6.7.
struct Split {
    int near, C, nfar;
    int chunks() const { return nfar + (near > 0); }
};
inline Split split_of(long wgs, double cache_bytes, int T, int d, bool want_m)
{
    Split s = {T, NEAR, 0};
    const bool spread = spread_small(wgs, cache_bytes, T, d, want_m);
    if (T <= (want_m ? ALONE : alone_up_to(wgs, d)) && !spread) return s;
    const bool all = want_m || spread;
    s.near = all ? 0 : NEAR;
    const int far = T - s.near, unit = all ? FAR_KEYS : NEAR;
    const long want = std::min((long)std::min(MAXFAR, room(T) - 1), std::max(1L, (all ? ALL_WGS : FAR_WGS) / wgs));
    s.C = (int)((far + want - 1) / want + unit - 1) / unit * unit;
    s.nfar = (far + s.C - 1) / s.C;
    return s;
}

}  // namespace sb
