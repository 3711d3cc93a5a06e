// Verification of the chunk-parallel scans: comparison of the states at the interval boundaries, the verdict over a
// (sequence, direction), and what an accepted one leaves for the later kernels.
// Included by semicrf.hip inside its anonymous namespace (after common.h); not a translation unit of its own.

// Largest disagreement at a boundary that is accepted: of two windows entry by entry after a default warm-up or a retry, which
// leave 1e-15 nearly everywhere; and where it is the choice of the warm-up that decides how much is left, or only what entries can
// still contribute that agrees: a length of L positions makes logZ some 3 L, whose 64 bits end at 3e-16 L or above, so that neither
// costs a digit of it.
constexpr double SPEC_TOL = 1e-10;
__device__ __forceinline__ double spec_tol_chosen(const Params &p, const int b) { return fmax(1e-13, 1e-16 * (double)p.hdr[b].L); }
// The bound of an attempt.
__device__ __forceinline__ double spec_tol(const Params &p, const int b, const int attempt)
{
    return attempt == 0 && p.warm_model && p.wlen[b].x != sum_warmup(p.K) ? spec_tol_chosen(p, b) : SPEC_TOL;
}
constexpr int SPEC_ATTEMPTS = 3;

// One workgroup per (chunk boundary j, sequence, direction): compare the state chunk j-1
// (forward) / chunk j (backward) reached at position j*Delta with the warm-up state the
// neighbouring chunk started from.  Number 0 is no boundary: its workgroup checks that the forward scan's final
// message vector can be summed (entry nint of the mismatches).
//
// negl: directions (bit 0 forward, bit 1 backward) whose windows may be compared by what their entries can still contribute
// (p.negl, see warm_plan): the difference of two entries counts against the larger of the two, or against negl[c] times the largest
// newer entry of the label, whichever is more.  At every later position an entry's difference then adds at most the bound / K of
// what the newer entry adds there, so the states agree to twice the bound in all they do: everything a state does later is a sum of
// positive multiples of these direct contributions.  Windows that agree entry by entry are not looked at this way.
// Bound by the latency of two states' loads and of the reductions: the working launch takes 16.5 us at the genomic shape (13.0 entry by
// entry alone), 16 at 32 x 2000, K = 32, C = 64 (12.5).
template <int PER>
__global__ __launch_bounds__(NT) void k_spec_cmp(Params p, int tier, int negl, int G, int per)
{
    __shared__ double part[NT / 64], newer[NT];
    const int j = blockIdx.x, b = blockIdx.y, dir = blockIdx.z, tid = threadIdx.x;
    const int lane = tid & 63, wv = tid >> 6;
    if (tier > 0 && p.spec_ok[b * 2 + dir]) return;
    const int K = p.K, KC = p.K * p.C, C = p.C, N = p.N;
    const size_t ckstride = (size_t)KC + C;
    const size_t at = (size_t)b * (N + 1) + j;
    const double *A = (dir ? p.ckB : p.ckA) + at * ckstride;    // warm-up state
    const double *A2 = (dir ? p.ckB2 : p.ckA2) + at * ckstride;  // reached state
    // thread (range of per <= PER distances, label), G ranges: all its entries are requested before anything is waited for
    const int g = tid / C, c = tid - g * C, d0 = g * per;
    const int nu = g < G ? min(per, K - d0) : 0;  // entries of this thread (none where that is negative)
    double x[PER > 0 ? PER : 1], y[PER > 0 ? PER : 1];
    const bool contrib = PER > 0 && ((negl >> dir) & 1);
    bool shorter = false;
    if (PER > 0) {
        shorter = tier == 0 && p.wlen[b].x < sum_warmup(K);
        const int tm = j * p.Delta % K;
        int sl = dir ? tm + d0 : tm - d0;  // slot of the position at that distance
        sl += dir ? (sl >= K ? -K : 0) : (sl < 0 ? K : 0);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int o = u < nu ? sl * C + c : 0;
            x[u] = A2[o];
            y[u] = A[o];
            sl += dir ? 1 : -1;
            sl = dir ? (sl == K ? 0 : sl) : (sl < 0 ? K - 1 : sl);
        }
    }
    const double Y = (dir ? p.ckYB : p.ckYA)[at], Y2 = (dir ? p.ckYB2 : p.ckYA2)[at];
    // sums of the two message vectors (their ratio is the common scale factor); C <= 64 here: every wave forms them
    double s1 = lane < C ? A[KC + lane] : 0.0, s2 = lane < C ? A2[KC + lane] : 0.0;
    const double m1 = s1, m2 = s2, ng = contrib ? p.negl[(size_t)b * C + c] : 0.0;
    const int L = p.hdr[b].L;
    const int nint = (L + p.Delta - 1) / p.Delta;
    if (j >= nint) return;
    const size_t so = ((size_t)b * 2 + dir) * (N + 1);
    if (j == 0) {
        if (dir == 0 && wv == 0) {
            const double *e = p.ckA2 + ((size_t)b * (N + 1) + nint) * ckstride;
            double s = lane < C ? e[KC + lane] : 0.0;
#pragma unroll
            for (int off = 1; off < 64; off <<= 1) s += __shfl_xor(s, off);
            const double Yl = p.ckYA2[(size_t)b * (N + 1) + nint];
            if (lane == 0) p.spec_err[so + nint] = (s > 0.0 && s < DBL_MAX && Yl == Yl) ? 0.0 : DBL_MAX;
        }
        return;
    }
    s1 = wave_sum(s1);
    s2 = wave_sum(s2);
    const double f = s2 / s1;  // reached = f * 2^(Y2-Y) * warm-up, entry by entry, if they agree
    double err = 0.0;
    if (!(s1 > 0.0) || !(s2 > 0.0) || !(f > 0.0) || !(f < DBL_MAX)) err = DBL_MAX;
    auto differ = [&](const double x, const double y, const double least) {
        const double m = fmax(fabs(x), fabs(y));
        // (a reciprocal by the hardware's estimate and one Newton step: to the last bits; 1e307: no message is larger)
        const double w = fmax(m, least), r = __builtin_amdgcn_rcp(w);
        if (m > 1e-290) err = fmax(err, fabs(x - y) * fma(fma(-w, r, 1.0), r, r));
        if (!(m < 1e307)) err = DBL_MAX;
    };
    auto over_waves = [&]() {  // the largest over the workgroup, in every thread
        err = wave_max(err);
        if (lane == 0) part[wv] = err;
        __syncthreads();
        for (int i = 0; i < NT / 64; ++i) err = fmax(err, part[i]);
    };
    if (wv == 0 && lane < C) differ(m2, m1 * f, 0.0);
    const double err0 = err;
    if (PER == 0) {
#pragma unroll 8
        for (int i = tid; i < KC; i += NT) differ(A2[i], A[i] * f, 0.0);
        over_waves();
    } else {
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            x[u] = u < nu ? x[u] : 0.0;
            y[u] = u < nu ? y[u] * f : 0.0;
        }
        // entry by entry first, where the warm-up was long enough for that
        if (!contrib || !shorter) {
#pragma unroll
            for (int u = 0; u < PER; ++u) differ(x[u], y[u], 0.0);
            over_waves();
        }
        const double whole = shorter ? DBL_MAX : err;
        if (contrib && whole > spec_tol(p, b, tier)) {
            double big = 0.0;
#pragma unroll
            for (int u = 0; u < PER; ++u) big = fmax(big, fmin(x[u], y[u]));
            newer[tid] = big;
            __syncthreads();
            err = err0;
            big = 0.0;
            for (int g0 = 0; g0 < min(g, G); g0 += 8) {
#pragma unroll
                for (int i = 0; i < 8; ++i) big = fmax(big, newer[min(g0 + i, g - 1) * C + c]);
            }
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                differ(x[u], y[u], ng * big);
                big = fmax(big, fmin(x[u], y[u]));
            }
            over_waves();
            if (!shorter && err > spec_tol_chosen(p, b)) err = whole;
        }
    }
    if (tid == 0) {
        p.spec_err[so + j] = err;
        p.spec_lr[so + j] = (Y2 - Y) + log2(f);
    }
}

// Verdict over the boundaries of a (sequence, direction), worked out by one wave, the same in every lane: accepted if
// every boundary is within the bound (and the forward scan's final vector is sound).
struct SpecVerdict {
    bool ok;
    int nint, nbad;  // intervals; boundaries that disagreed
    double worst;
};
__device__ __forceinline__ SpecVerdict spec_verdict(const Params &p, const int b, const int dir, const int lane, const int attempt)
{
    SpecVerdict v;
    const double tol = spec_tol(p, b, attempt);
    const double *err = p.spec_err + ((size_t)b * 2 + dir) * (p.N + 1);
    v.nint = (p.hdr[b].L + p.Delta - 1) / p.Delta;
    v.worst = 0.0;
    int bad = 0;
#pragma unroll 4
    for (int i = 1 + lane; i < v.nint; i += 64) {
        const double e = err[i];
        v.worst = fmax(v.worst, e);
        bad += !(e <= tol);
    }
    v.worst = wave_max(v.worst);
    v.nbad = (int)wave_sum((double)bad);
    v.ok = v.nbad == 0 && v.worst <= tol && (dir == 1 || v.nint == 0 || err[v.nint] == 0.0);
    return v;
}

// Leaves the verdict on attempt `tier` for the later kernels and, on acceptance, chains the scale factors into the
// checkpoint scales (only then: a later attempt that rewrites some of the checkpoints must find the others as their tasks
// left them) and logZ.  One wave: lane l owns a contiguous run of boundaries in scan order, the running log2 factor is a
// fixed-order prefix sum (per lane, then across lanes).
__device__ __forceinline__ void spec_settle(const Params &p, const int b, const int dir, const int ndir, const int tier,
                                            const SpecVerdict &v, const int lane)
{
    const int N = p.N, C = p.C, KC = p.K * C, nint = v.nint;
    double *lr = p.spec_lr + ((size_t)b * 2 + dir) * (N + 1);  // entry 0 is no boundary: it carries the number that disagreed
    if (dir == 0 && ndir == 1 && lane == 0) {  // the other direction is not run in this call
        p.spec_ok[b * 2 + 1] = 0;
        p.spec_rep[b * 2 + 1] = -1.0;
    }
    if (v.ok) {
        const int nb = nint > 1 ? nint - 1 : 0;  // boundaries 1 .. nint-1
        const int per = (nb + 63) / 64;
        const int i0 = min(lane * per, nb), i1 = min(i0 + per, nb);
        // i-th boundary in scan order: ascending for the forward scan, descending for the backward one
        auto jof = [&](int i) { return dir == 0 ? 1 + i : nint - 1 - i; };
        double s = 0.0;
#pragma unroll 4
        for (int i = i0; i < i1; ++i) s += lr[jof(i)];
        double inc = s;
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) {
            const double x = __shfl_up(inc, off);
            if (lane >= off) inc += x;
        }
        const double total = __shfl(inc, 63);
        double *ckY = (dir ? p.ckYB : p.ckYA) + (size_t)b * (N + 1);
        double acc = inc - s;  // log2 of the factor between the true state and the warm-up state
        for (int i = i0; i < i1; ++i) {
            acc += lr[jof(i)];
            ckY[jof(i)] += acc;
        }
        if (dir == 0) {
            double lz;
            if (nint == 0) {
                lz = log((double)C);
            } else {
                // a_L(c) / Z: mass of the segments that end at L with label c
                const double *e = p.ckA2 + ((size_t)b * (N + 1) + nint) * ((size_t)KC + C);
                const double vL = lane < C ? e[KC + lane] : 0.0;
                double sumL = vL;
#pragma unroll
                for (int off = 1; off < 64; off <<= 1) sumL += __shfl_xor(sumL, off);
                lz = (p.ckYA2[(size_t)b * (N + 1) + nint] + total) * LN2 + log(sumL);
                if (lane < C) p.inL[(size_t)b * C + lane] = vL / sumL;
            }
            if (lane == 0) {
                p.hdr[b].logZ = lz;
                p.logz[b] = (float)lz;
            }
        }
    }
    if (lane != 0) return;
    // which attempt verified it: 1 the first, or 4 the first after a warm-up as long as labels that are steps apart need
    // (warm_plan); 2 after repairs, 3 after a longer warm-up (what the later attempts did was decided by the number of
    // boundaries that had disagreed before)
    const int code = tier == 0 ? (p.warm_model && p.wlen[b].w ? 4 : 1) : (lr[0] <= (double)max(2, nint / 16) ? 2 : 3);
    p.spec_rep[b * 2 + dir] = v.worst;
    p.spec_ok[b * 2 + dir] = v.ok ? code : 0;
    lr[0] = (double)v.nbad;
}

// What the statistics of an interval start from: the backward state at its upper boundary (`at`: offset of that checkpoint),
// in the frame of the warmed-up one.  After a warm-up shorter than the window the entries that no longer matter to the scan
// may be missing there, but the expected counts of long durations are made of them: the state the task above reached there
// has them, and the two differ by a common factor, which is returned.  Every lane of a wave calls it.
__device__ __forceinline__ double state_above(const Params &p, const int b, const size_t at, const double *&ck)
{
    ck = p.ckB + at;
    if (!(p.warm_model & WARM_SHORTER) || !p.spec_ok[b * 2 + 1]) return 1.0;  // (no mended or sequential scan leaves them out)
    const int lane = threadIdx.x & 63, KC = p.K * p.C;
    const double own = lane < p.C ? ck[KC + lane] : 0.0;
    ck = p.ckB2 + at;
    return wave_sum(own) / wave_sum(lane < p.C ? ck[KC + lane] : 0.0);
}

// Verdicts in a launch of their own, for scans whose kernels do not work them out (duration-dependent transitions).
// grid (B, directions), one wave.  The backward scans there have used the forward rows of the same attempt, so a backward
// scan is accepted only where the forward one is.
__global__ __launch_bounds__(64) void k_spec_fix(Params p, int ndir, int tier)
{
    const int b = blockIdx.x, dir = blockIdx.y, lane = threadIdx.x;
    if (tier > 0 && p.spec_ok[b * 2 + dir]) return;
    SpecVerdict v = spec_verdict(p, b, dir, lane, tier);
    if (p.warm_model && tier == 0 && lane == 0) {
        const int w0 = p.wlen[b].x;
        (&p.wlen[b].y)[dir] = v.ok ? w0 : last_warm(p, w0);
    }
    if (dir == 1) v.ok = v.ok && spec_verdict(p, b, 0, lane, tier).ok;
    spec_settle(p, b, dir, ndir, tier, v, lane);
}

// Sequential scans: true if the pair needs none.  They follow the last attempt (number `tier`), whose verdict they
// work out themselves.
__device__ __forceinline__ bool spec_settled(const Params &p, const int b, const int dir, const int ndir, const int tier)
{
    if (!p.spec) return false;
    if (p.spec_ok[b * 2 + dir]) return true;
    const int lane = threadIdx.x & 63;
    const SpecVerdict v = spec_verdict(p, b, dir, lane, tier);
    if (threadIdx.x < 64) spec_settle(p, b, dir, ndir, tier, v, lane);
    return v.ok;
}

