// What a check of the Hartree CG tells the host: <r, r>, and whether no iteration
// went before it (then even a residual that is not finite is the start's own, no
// divergence).  One word, so that a host which reads while the next check writes
// sees the one or the other as a whole; the bound beside it is the same for all
// checks of a solve.  Plain C++ apart from the annotations (g++ in the host tests).
#pragma once
#include <cmath>

#if defined(__HIPCC__)
#define OFKS_REPORT_HD __host__ __device__ __forceinline__
#else
#define OFKS_REPORT_HD inline
#endif

namespace ofks {

// rr >= 0 or NaN; the sign says whether the check was the first
OFKS_REPORT_HD double cg_report_word(double rr, bool first) { return std::copysign(rr, first ? -1.0 : 1.0); }

struct CgSeen {
    double rr;
    bool stop, diverged;
};
inline CgSeen cg_report_seen(double word, double tol2) {
    const double rr = std::fabs(word);
    const bool bad = !std::isfinite(rr) && !std::signbit(word);
    return {rr, !(rr > tol2) || bad, bad};
}

}  // namespace ofks
