// Sizes and LDS geometry of the kernels, as plain C++ (no HIP): what the kernels are instantiated with and what
// the host-side planning code computes workspace layouts and launch shapes from.  constexpr functions are usable
// on both sides of a HIP compilation.
#ifndef SEMICRF_GEOMETRY_H
#define SEMICRF_GEOMETRY_H

#include <stddef.h>

namespace semicrf_impl {

constexpr int NT = 256;          // threads per workgroup in the scan kernels
constexpr int PREP_CH = 256;     // positions per prefix-sum chunk (multiple of JMAX)
constexpr int JMAX = 32;         // largest scaling block
constexpr int TAB_BLOCKS_MAX = 64;  // most workgroups the exp tables (and their maxima) are spread over
constexpr int NSLOT_MAX = 1024;  // resident tasks of the interval kernel (one wave per SIMD)
constexpr int LOWMEM_SLOTS_PER_SEQ = 8;  // row slots per sequence in the low-memory plan
constexpr int GRAD_CMAX = 64;    // most labels the gradient path holds transition accumulators for
constexpr size_t LDS_LIMIT = 160 * 1024;
constexpr size_t SEQ_HDR_BYTES = 32;  // sizeof(SeqHdr), the per-sequence header at the front of the workspace
constexpr int SINK_DOUBLES = 1536;    // target of stores that must be issued but whose value nobody wants

constexpr int MB = 4;      // positions per time block of the one-wave kernels
constexpr int MG_TG = 32;  // stored-row marginals: positions staged at a time
constexpr int MG_KS = 8;   // stored-row marginals: durations per thread of the duration kernel
constexpr int FIN_SLICES = 4;    // workgroups per sequence of the carry / mean reduction (sums behind the mean per slice)
constexpr int MG_SIMDS = 1024;  // SIMDs of the chip (256 compute units of four)

// LDS bytes of the vector form of the duration statistics for that many labels and strips of MG_KS durations at once: rows of a group,
// their factors, exponents and scaling blocks, and the absolute scales of the rows that the interval can touch.
constexpr size_t mg_dur_lds(int labels, int strips, int K, int Delta)
{
    const size_t vr = (size_t)MG_TG + (size_t)MG_KS * strips + 3;
    return ((size_t)MG_TG * labels + vr * (labels | 3) + MG_TG + 2 * vr + 2 * (size_t)Delta + (size_t)K) * 8;
}

// Tasks of the one-wave stored-row marginals a SIMD holds: two where the duration strip of a lane (NKW) and the
// transition tiles (CT) leave the kernel within half the register file, else one.
constexpr int mg_waves_per_simd(int CT, int NKW) { return (CT <= 32 && NKW <= 32) ? 2 : 1; }

constexpr size_t align_up(size_t x) { return (x + 255) & ~(size_t)255; }

// What the choice of the first warm-up reads and leaves (one array of the workspace): per sequence and label what the
// comparison of two windows takes for negligible, per sequence the warm-up lengths, per chunk the sampled contrast.
struct WarmLayout {
    size_t negl, len, contrast, total;
};
constexpr WarmLayout warm_layout(int B, int C, int NCH)
{
    WarmLayout l{};
    l.negl = 0;
    l.len = align_up((size_t)B * C * 8);
    l.contrast = l.len + align_up((size_t)B * 4 * 4);
    l.total = l.contrast + align_up((size_t)B * NCH * 4);
    return l;
}

constexpr int pow2_ge8(int x)
{
    int r = 8;
    while (r < x) r <<= 1;
    return r;
}

// LDS doubles of the workgroup-per-sequence kernels (sequential scan, generic interval kernel):
//   ring[K*C]  Wl[K*C]  El[C*(C|1)]  red[G*C]  yv, zv, av, qv [C]  sc[C] (int)  and, interval kernel only, accD[K*C]
constexpr size_t lds_doubles(int K, int C, int G, bool interval)
{
    return 2 * (size_t)K * C + (size_t)C * (size_t)(C | 1) + (size_t)G * C + 5 * (size_t)C +
           (interval ? (size_t)K * C : 0);
}

// Label tile of the one-wave kernels for C labels (C <= 64).
constexpr int spec_ct_of(int C)
{
    return C <= 8 ? 8 : (C <= 16 ? 16 : (C <= 24 ? 24 : (C <= 32 ? 32 : 64)));
}

// Window entries per lane: NKW, plus one when a half-wave holds several lane groups, so
// that the groups' rows fall into different LDS banks.
constexpr int wave_nk(int CT, int NKW)
{
    return NKW + ((64 / pow2_ge8(CT)) > 2 ? 1 : 0);
}

// Rows of slack behind the sliding window: a quarter of the window (the window is moved back once
// per that many positions), an eighth for the deepest window, where the quarter would cost the
// fourth resident task of a compute unit its LDS.
constexpr int lin_slack(int KW)
{
    return KW / 4 < 8 ? 8 : (KW >= 512 ? ((KW / 8 + 3) & ~3) : ((KW / 4 + 3) & ~3));
}

constexpr size_t wave_lds_doubles(int CT, int NKW)
{
    const int CTP = pow2_ge8(CT);
    const int KW = wave_nk(CT, NKW) * (64 / CTP);
    const int YS = CTP < 16 ? 16 : CTP;
    return (size_t)(KW + lin_slack(KW)) * CT + (size_t)(CTP - CT) + (size_t)MB * YS;
}

// The scans' window lies in runs: a lane takes 16 consecutive distances (17 when a half-wave holds several lane groups, as
// above) of each run, the lane groups one after the other, so that a run is the newest of the distances not yet
// covered and the whole wave can leave the older runs alone.
constexpr int scan_runs(int NKW) { return NKW / 16; }
constexpr int scan_run(int CT) { return 16 + ((64 / pow2_ge8(CT)) > 2 ? 1 : 0); }
constexpr int scan_kw(int CT, int NKW) { return scan_runs(NKW) * scan_run(CT) * (64 / pow2_ge8(CT)); }

// Tasks of the scan kernel a SIMD holds by registers: one where the transition column or the duration strip is long.
constexpr int spec_waves_per_simd(int CT, int NKW) { return (CT == 64 || (CT == 32 && NKW == 64)) ? 1 : 2; }

// Rows of slack of the scan kernels' windows: the window is moved back once per that many positions, which costs a
// read and a write of every window entry, so the slack takes what LDS the resident tasks of a compute unit leave
// (up to a whole window), never less than lin_slack.
// two: the tasks of two waves, which keep more than the window in LDS and are half as many.
constexpr int spec2_waves_per_simd(int CT, int NKW) { return (CT <= 32 && NKW <= 32) ? 4 : 2; }
constexpr int slack_rows(int CT, int KW, size_t extra, size_t most)
{
    const size_t least = (size_t)(KW + lin_slack(KW)) * CT + extra;
    const size_t limit = LDS_LIMIT / sizeof(double);
    size_t tasks = limit / least;
    if (tasks < 1) tasks = 1;
    if (tasks > most) tasks = most;
    const size_t rows = limit / tasks > extra ? (limit / tasks - extra) / CT : 0;
    int m = rows > (size_t)KW ? (int)(rows - KW) : 0;
    if (m > KW) m = KW;
    m &= ~3;
    return m > lin_slack(KW) ? m : lin_slack(KW);
}
constexpr int scan_slack(int CT, int NKW, bool two)
{
    const int CTP = pow2_ge8(CT);
    const size_t extra = (CTP - CT) + (two ? (size_t)2 * MB * CT + (size_t)2 * MB * CTP + 2 : 0);
    return slack_rows(CT, scan_kw(CT, NKW), extra, two ? 2 * (size_t)spec2_waves_per_simd(CT, NKW) : 4 * (size_t)spec_waves_per_simd(CT, NKW));
}

// LDS of a one-wave scan task: the window.
constexpr size_t scan_lds_doubles(int CT, int NKW)
{
    return (size_t)(scan_kw(CT, NKW) + scan_slack(CT, NKW, false)) * CT + (size_t)(pow2_ge8(CT) - CT);
}

// Single-wave tasks of one workgroup of the scan kernels: one per SIMD where their LDS fits.
constexpr int waves_of_lds(size_t doubles)
{
    const size_t lds = doubles * sizeof(double);
    return 4 * lds <= LDS_LIMIT ? 4 : (2 * lds <= LDS_LIMIT ? 2 : 1);
}
constexpr int spec_waves(int CT, int NKW) { return waves_of_lds(scan_lds_doubles(CT, NKW)); }

// Single-wave tasks of one workgroup of the interval kernel.
constexpr int interval_waves(int CT, int NKW) { return CT == 64 ? 4 : (NKW == 64 ? 3 : 1); }

constexpr size_t interval_wtab_doubles(int CT, int NKW)
{
    return NKW == 64 ? (size_t)(wave_nk(CT, NKW) * (64 / pow2_ge8(CT)) + MB) * CT + (size_t)(pow2_ge8(CT) - CT) : 0;
}

constexpr size_t interval_lds_doubles(int CT, int NKW)
{
    return (CT == 64 ? 2 * (size_t)CT * CT : 0) + interval_wtab_doubles(CT, NKW) +
           (size_t)interval_waves(CT, NKW) * wave_lds_doubles(CT, NKW);
}

}  // namespace semicrf_impl
#endif
