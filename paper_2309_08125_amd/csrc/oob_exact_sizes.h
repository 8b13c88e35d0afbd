// Index arithmetic of the exact minimum (oob_exact.hip) that the host can check over everything the entry points
// accept: plain C++, so that a CPU test compiles it too.
#pragma once

#ifdef __HIPCC__
#define OOB_HD __host__ __device__
#else
#define OOB_HD
#endif

namespace oob_exact {

// i / M for an index i = l M + d of a table with M GPU counts per layer (l <= 255, d < M <= 64) as i recip(M) >> 20.  With
// e = M recip(M) - 2^20 <= M the quotient is i / M + i e / (2^20 M): exact while i e < 2^20, and i e <= (256 M - 1) M < 2^20.
// The product stays below 256 M (2^20 / M + 1) < 2^29.
constexpr int kRecipShift = 20;
OOB_HD inline unsigned recip(int M) { return (1u << kRecipShift) / (unsigned)M + 1; }
OOB_HD inline int quot(int i, unsigned recip_M) { return (int)((unsigned)i * recip_M >> kRecipShift); }

} // namespace oob_exact
