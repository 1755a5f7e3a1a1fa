// How a number of equal pieces is dealt out to workgroups.  Free of device code, so that a host program can check it.
#pragma once

#if defined(__HIPCC__)
#define DFK_SHARE_HD __host__ __device__ __forceinline__
#else
#define DFK_SHARE_HD inline
#endif

namespace dfk {

// lo = floor(n s / S), hi = floor(n (s + 1) / S) for s < S <= 65535 and any n, in 32 bits: with n = q S + r that is
// q s + floor(r s / S), and r s < 2^32.  A 64-bit division by a number only known at run time is 200 instructions, with a jump to the
// far end of the kernel and back, met out of a cold instruction cache before the first load is requested.  Without them: block of
// 2304 x 9216 at 1 token 31.3 -> 30.9 us, 1024 x 2816 at 16 13.1 -> 12.8, 2048 x 5504 at 16 22.9 -> 22.6, 896 x 4864 at 1 16.0 -> 15.9.
DFK_SHARE_HD void share_of(unsigned n, unsigned S, unsigned s, int& lo, int& hi) {
    const unsigned q = n / S, r = n - q * S, t = r * s / S, rest = r * s - t * S;
    lo = (int)(q * s + t);
    hi = (int)(q * (s + 1u) + t + (rest + r >= S ? 1u : 0u));
}

// The slice (of S <= 65535) that holds piece i of n: the inverse of share_of.  32 bits are enough for up to 65536 pieces.
DFK_SHARE_HD int share_with(int n, int S, int i) {
    if (__builtin_expect(n <= 65536, 1)) return (int)((((unsigned)i + 1u) * (unsigned)S - 1u) / (unsigned)n);
    return (int)((((long long)i + 1) * S - 1) / n);
}

}  // namespace dfk
