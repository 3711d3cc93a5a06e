// Viterbi decode (max semiring): scan, verification, trace-back.
// Included by semicrf.hip inside its anonymous namespace (after common.h); not a translation unit of its own.

// ---------------------------------------------------------------------------
// Viterbi decode (max semiring) with the window / time-block organisation of the one-wave
// kernels, in the log domain (fp64 additions and maxima only; nothing needs rescaling):
//     r_s(c) = max_c' (V_s(c') + trans[c',c]) + (start score of token s) - S[s,c]        (leaves s)
//     V_t(c) = S[t,c] + (end score of token t-1) + max_k (dur[k,c] + r_{t-k}(c))          (arrives at t)
// V_0 = 0 for every label.  The scan stores V_t by position and r_t by label for every position and label; no
// back-pointers are kept.  The trace-back (k_vit_trace) finds each segment's duration and
// predecessor label by recomputing the candidates from the stored values.  Ties go to the
// smallest duration, then the smallest label.
//
// Ties are structural (a run of one label longer than K can be cut into the same durations in any order), and equal sums
// come out different in their last bits, so candidates within rounding of the best one are ties.  A stored value is a
// sum with the prefix sum in it and off by a few units in the last place of the larger of the two, more where the scores
// of two paths were added up over many segments before they meet; 2^-42 (1024 units) of |candidate| + |prefix sum| is
// well above that and far below what single-precision scores differ by.  With an exact comparison 1 % of the
// start flags depended on the order of additions (C = 3, K = 57), and so on how the scan was cut into intervals.
// ---------------------------------------------------------------------------
constexpr double VIT_TIE = 0x1p-42;

// Candidate x ties with the best one where x + vit_slack(scale) >= vit_floor(best); scale: a value of about the size of the
// prefix sums in x (ignored if infinite).  In two parts, so that only the second has to wait for the best one.
__device__ __forceinline__ double vit_slack(const double scale)
{
    const double a = fabs(scale);
    return VIT_TIE * (1.0 + (a < DBL_MAX ? a : 0.0));
}
__device__ __forceinline__ double vit_floor(const double best)
{
    const double m = fabs(best);
    return m < DBL_MAX ? fma(-VIT_TIE, m, best) : best;
}

// Best final label (smallest on ties) and score: lane holds V_L of label c in v, in the lanes `own` (one per label).
__device__ __forceinline__ void vit_best(const Params &p, const int b, const double v, const int c, const bool own,
                                         const double unit)
{
    const double best = wave_max(own ? v : -INFINITY);
    const double sum = own ? p.EI[((size_t)b * (p.T + 1) + p.hdr[b].L) * p.C + c].x : 0.0;
    int bl = own && (v + unit) + vit_slack(sum) >= vit_floor(best + unit) ? c : 0x7fffffff;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) bl = min(bl, __shfl_xor(bl, off));
    if ((threadIdx.x & 63) == 0) {
        p.vscore[b] = p.hdr[b].L > 0 ? (float)(best + unit) : 0.f;
        p.vbest[b] = bl < 0x7fffffff ? bl : 0;
    }
}

// One scan task: the whole sequence (WHOLE: the sequential scan) or one checkpoint interval
// (lo, hi] after a warm-up over the `warm` positions before it, started as a sequence that
// begins there.  A chunk task records its window and V vector at lo (-> ckA[chunk]) and at hi
// (-> ckA2[chunk+1]) for the verification, and stores V_t and r_t for lo < t <= hi (and for
// position 0 if lo = 0) in ITS OWN additive unit: max-plus recurrences are invariant under adding
// a constant to every message, and a warmed-up chunk differs from the true values by exactly such
// a constant once all best paths through the warm-up have merged.
// Lanes, window and time blocks as in the sum scans (spec_task): a maximum of sums is two
// instructions where they have one, and the transition maximum three per entry (row broadcast, add,
// max), still less than the way through LDS.  Genomic shape, 1024 tasks of 520 positions: 395 us with the
// V vector in LDS and the window read where it is used, 252 us so (an instruction issues in 69 % of a wave's cycles).
// V goes out by position, as it is made.  The trace-back looks at r along the positions of one label, so r is stored
// by label, FT positions at a time out of the window (a row of FT * 8 bytes per label).
template <int CT, int NKW, bool WHOLE>
__device__ __forceinline__ void vit_task(const Params &p, double *lds_raw, const int b, const int chunk,
                                         const int warm)
{
    using G = WaveWin<CT, NKW, 1>;
    using R = RowMap<CT>;
    constexpr int RS = G::RS, KW = G::KW, ROWS = G::ROWS, RUN = G::RUN, RUNS = G::RUNS;
    constexpr int RTOT = G::RTOT, HC = G::HC;
    const int lane = threadIdx.x & 63;
    const int K = p.K, C = p.C, KC = K * C;
    double *ring = lds_raw;          // [ROWS][RS] (+ pad): r of the last KW positions
    const int c = R::label(lane), g = R::group(lane);
    const int hh = G::H == 2 ? (lane >> 5) : 0;
    const bool cval = c < C;
    const int cc = cval ? c : 0;
    const bool writer = cval && g == 0;
    const int L = p.hdr[b].L;
    const int lo = WHOLE ? 0 : chunk * p.Delta;
    if (!WHOLE && lo >= L && !(lo == 0 && L == 0)) return;
    const int hi = WHOLE ? L : min(lo + p.Delta, L);
    const int s0 = WHOLE ? 0 : max(lo - warm, 0);
    const size_t row0 = (size_t)b * (p.T + 1);
    const double2 *LPc = p.EI + row0 * C + cc;  // (S + end score, start score - S)
    double *VV = p.vv + row0 * C, *RT = p.vrt + row0 * C;
    const size_t ts = (size_t)p.T + 1;  // positions of a label in RT
    const double NINF = -INFINITY;

    double wd[RUNS][RUN + MB - 1];  // bias of the durations of the lane's distances in each run, and of the next three
    double wfar = NINF;             // largest bias of the durations beyond the first run
#pragma unroll
    for (int u = 0; u < RUNS; ++u) {
#pragma unroll
        for (int jj = 0; jj < RUN + MB - 1; ++jj) {
            const int k = G::run_dist(u, g) + jj + 1;
            wd[u][jj] = (cval && k <= K) ? (double)p.dur[(size_t)(k - 1) * C + c] : NINF;
            if (u > 0) wfar = fmax(wfar, wd[u][jj]);
        }
    }
    wfar = group_max<G::CTP>(wfar);
    double wn[MB - 1];
#pragma unroll
    for (int jj = 0; jj < MB - 1; ++jj) wn[jj] = (cval && jj + 1 <= K) ? (double)p.dur[(size_t)jj * C + c] : NINF;
    double Treg[HC];         // trans[o, c] for the lane's half of the source labels
#pragma unroll
    for (int i = 0; i < HC; ++i) {
        const int o = hh * HC + i;
        Treg[i] = (cval && o < C) ? (double)p.trans[(size_t)o * C + c] : NINF;
    }

    for (int i = lane; i < RTOT; i += 64) ring[i] = NINF;
    lds_wave_fence();
    int r = KW - 1;
    double ylast = cval ? 0.0 : NINF;  // V of the newest position: 0 for every label where the (sub)sequence begins
    // state for the verification: r of the K positions up to t (by distance), then V_t
    const size_t ckstride = (size_t)KC + C;
    auto record = [&](double *ck) {
        if (cval) {
#pragma unroll 4
            for (int d = g; d < K; d += G::GW) ck[(size_t)d * C + c] = ring[(r - d) * RS + c];
        }
        if (writer) ck[KC + c] = ylast;
    };
    {
        const double q = R::max_product(ylast, Treg) + LPc[(size_t)s0 * C].y;
        if (writer) {
            ring[r * RS + c] = q;
            if (s0 == lo) VV[c] = 0.0;  // position 0
        }
    }
    lds_wave_fence();
    constexpr int FT = KW >= 32 ? 16 : 8;  // the window must hold FT + MB - 1 positions
    int tf = s0 == lo ? 0 : lo + 1;        // first position whose r has not been stored
    int t = s0;
    auto flush = [&]() {
        const int tp = tf + (lane & (FT - 1));
        const double *src = ring + (r - (t - tp)) * RS;
        double *dst = RT + tp;
#pragma unroll
        for (int i = 0; i < CT * FT / 64; ++i) {
            const int cl = i * (64 / FT) + lane / FT;
            if (tp <= t && cl < C) dst[cl * ts] = src[cl];
        }
        tf += FT;
    };
    double old = NINF;  // no entry of the label beyond the first run is larger
    auto load_rows = [&](double2 (&e)[MB], const int tfrom) {
#pragma unroll
        for (int i = 0; i < MB; ++i) e[i] = LPc[(size_t)min(tfrom + 1 + i, hi) * C];
    };
    double2 e[MB];
    load_rows(e, t);
    while (t < hi) {
        int nb = min(hi - t, MB);
        if (t < lo) nb = min(nb, lo - t);  // the position where the chunk proper starts ends its block
        const bool keep = t >= lo;
        double2 en[MB];
        load_rows(en, t + nb);
        if (__builtin_expect(r + MB > ROWS - 1, 0)) r = G::template move<false>(ring, lane, r);
        double acc[MB];
#pragma unroll
        for (int i = 0; i < MB; ++i) acc[i] = NINF;
        G::template window_maxima<false, MB>(ring + r * RS + G::template run_offset<false>(0, g, c), wd[0], acc);
#pragma unroll
        for (int i = 0; i < MB; ++i) acc[i] = group_max<G::CTP>(acc[i]);
        if (RUNS > 1) {
            // Older entries are looked at where one of them may win: none does while the largest of them with the largest
            // bias stays below what the first run offers, for every label and position (a maximum over fewer candidates,
            // the same to the last bit).  Splits that pay and label changes bring that about soon.
            old = fmax(old, G::template newly_old<false>(ring, r, c, [](const double a, const double x) { return fmax(a, x); }));
            const bool beaten = !cval || old + wfar <= fmin(fmin(acc[0], acc[1]), fmin(acc[2], acc[3]));
            if (!__all(beaten)) {
                double far[MB];
#pragma unroll
                for (int i = 0; i < MB; ++i) far[i] = NINF;
#pragma unroll
                for (int u = 1; u < RUNS; ++u)
                    G::template window_maxima<false, MB>(ring + r * RS + G::template run_offset<false>(u, g, c), wd[u], far);
#pragma unroll
                for (int i = 0; i < MB; ++i) acc[i] = fmax(acc[i], group_max<G::CTP>(far[i]));
            }
        }
        auto block = [&](auto store) {  // store(i, y): V of the block's position i
            double qn[MB];
            auto position = [&](const int i) {
                double x = acc[i];
#pragma unroll
                for (int jn = 0; jn < i; ++jn) x = fmax(x, wn[i - 1 - jn] + qn[jn]);
                const double y = x + e[i].x;  // V_t(c)
                ylast = y;
                const double q = R::max_product(y, Treg) + e[i].y;
                qn[i] = q;
                ++r;
                if (writer) ring[r * RS + c] = q;
                store(i, y);
            };
            if (__builtin_expect(nb == MB, 1)) {  // a whole block: nothing is decided per position
#pragma unroll
                for (int i = 0; i < MB; ++i) position(i);
                // (either kind of block takes over the next rows itself, before stores whose number differs: see spec_task)
#pragma unroll
                for (int i = 0; i < MB; ++i) e[i] = en[i];
            } else {
#pragma unroll
                for (int i = 0; i < MB; ++i) {
                    if (i < nb) position(i);
                    else qn[i] = NINF;
                }
#pragma unroll
                for (int i = 0; i < MB; ++i) e[i] = en[i];
            }
        };
        // The rows of V go out through a buffer that holds just the block's; with 64 label lanes through one pointer per lane, to a sink where
        // there is nothing to store: the transitions alone take half of a wave's registers there, and a position moves 48 values
        // between the two halves of the register file, through the buffer 66 (K <= 32).  4 x 4000 positions, K = 20, C = 48: 403 us, through the
        // buffer 421, in one piece 434 and 454; 20 labels, K = 30, in one piece 1408 and 1287.
        if constexpr (CT == 64) {
            double *rowp = p.sink + lane;
            int rstep = 0;
            if (keep && writer) {
                rowp = VV + (size_t)(t + 1) * C + c;
                rstep = C;
            }
            block([&](const int i, const double y) { __builtin_nontemporal_store(y, rowp + i * rstep); });
        } else {
            const RowStore rows(VV + (size_t)(t + 1) * C, keep ? MB * C * 8 : 0);
            const unsigned lane_row = writer ? (unsigned)c * 8u : ROW_NOWHERE;
            block([&](const int i, const double y) { rows.one(lane_row, i * C * 8, y); });
        }
        lds_wave_fence();
        t += nb;
        if (t - tf >= FT - 1) flush();
        if (!WHOLE && __builtin_expect(t == lo, 0)) record(p.ckA + ((size_t)b * (p.N + 1) + chunk) * ckstride);
    }
    if (tf <= t) flush();
    if (!WHOLE) {
        record(p.ckA2 + ((size_t)b * (p.N + 1) + chunk + 1) * ckstride);
        return;
    }
    vit_best(p, b, ylast, c, writer, 0.0);
}

// Largest disagreement at a chunk boundary that is accepted, relative to the larger of the entry
// and the prefix sums at the boundary.
constexpr double VIT_TOL = 1e-12;

// The chunk-parallel scan: spec_waves(CT, NKW) tasks per workgroup, one per wave, as k_spec.  RETRY: only the chunks
// whose warmed-up start disagreed with what the chunk before reached (chunk 0 starts exactly; by induction over the
// boundaries a chunk whose left boundary agrees is right up to its constant, so only these can be wrong).
template <int CT, int NKW, bool RETRY>
__global__ __launch_bounds__(64 * spec_waves(CT, NKW), spec_waves_per_simd(CT, NKW)) void k_vit_spec(Params p, int warm)
{
    extern __shared__ double lds_raw[];
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int task = (int)blockIdx.x * spec_waves(CT, NKW) + wave;
    const int b = task / p.N, chunk = task % p.N;
    if (b >= p.B) return;
    if (RETRY) {
        if (chunk == 0 || chunk * p.Delta >= p.hdr[b].L) return;
        if (p.spec_err[((size_t)b * 2) * (p.N + 1) + chunk] <= VIT_TOL) return;
    }
    vit_task<CT, NKW, false>(p, lds_raw + (size_t)wave * scan_lds_doubles(CT, NKW), b, chunk, RETRY ? warm : first_warm(p, b, warm));
}

// Per chunk boundary j (position j*Delta): the state chunk j-1 reached against the warmed-up
// state chunk j started from.  They must agree entry by entry up to ONE additive constant
// (taken from the largest V entry); -inf entries must coincide.  The results of the first attempt and of the second lie
// in the two halves of spec_err and spec_lr; the second compares again what its scans have rewritten.
//
// PER > 0: entries that can never win need not agree.  What an entry at distance d offers position j + 1 .. after the boundary is
// dur[j+d] + r_d; a newer entry at d' < d offers dur[j+d'] + r_d', and is still there as long as the older one is.  With
// negl[c] the most by which the duration bias of a longer duration exceeds that of a shorter one, an entry that lies negl[c] below
// a newer one of its label (in both states) is never the best, so states that agree elsewhere do the same.
template <int PER>
__global__ __launch_bounds__(NT) void k_vit_cmp(Params p, int tier, int G, int per)
{
    __shared__ double part[NT / 64], newer[2 * NT];
    const int j = blockIdx.x, b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int L = p.hdr[b].L;
    const int nint = (L + p.Delta - 1) / p.Delta;
    if (j < 1 || j >= nint) return;
    const int K = p.K, KC = p.K * p.C, C = p.C, N = p.N;
    const size_t o = ((size_t)b * 2) * (N + 1) + j, o2 = o + (tier ? N + 1 : 0);
    if (tier) {
        const double e0 = p.spec_err[o], em = j > 1 ? p.spec_err[o - 1] : 0.0;
        if (e0 <= VIT_TOL && em <= VIT_TOL) {
            if (tid == 0) {
                p.spec_err[o2] = e0;
                p.spec_lr[o2] = p.spec_lr[o];
            }
            return;
        }
    }
    const size_t ckstride = (size_t)KC + C;
    const double *A = p.ckA + ((size_t)b * (N + 1) + j) * ckstride;    // warm-up state
    const double *A2 = p.ckA2 + ((size_t)b * (N + 1) + j) * ckstride;  // reached state
    // thread (range of per <= PER distances, label), G ranges: all its entries are requested before anything is waited for
    const int g = PER > 0 ? tid / C : 0, c = tid - g * C, d0 = g * per;
    const int nu = g < G ? min(per, K - d0) : 0;
    double x[PER > 0 ? PER : 1], y[PER > 0 ? PER : 1];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int i = u < nu ? (d0 + u) * C + c : 0;
        x[u] = A2[i];
        y[u] = A[i];
    }
    // additive constant: at the largest reached V entry (smallest label on ties); every wave finds it
    const double v = lane < C ? A2[KC + lane] : -INFINITY;
    const double va = lane < C ? A[KC + lane] : -INFINITY;
    const double vm = wave_max(v);
    const unsigned long long at = __ballot(v == vm);
    const double delta = vm - __shfl(va, at ? __ffsll(at) - 1 : 0);
    double err = (vm > -INFINITY && delta == delta && fabs(delta) < DBL_MAX) ? 0.0 : DBL_MAX;
    // Every entry is a difference of prefix sums (r carries -S, V carries +S), so its rounding
    // error scales with |S| here, not with the entry: measure relative to the larger of the two.
    double smag = 1.0;
    if (lane < C) {
        const double2 lp = p.EI[((size_t)b * (p.T + 1) + (size_t)j * p.Delta) * C + lane];
        if (fabs(lp.x) < DBL_MAX) smag = fmax(smag, fabs(lp.x));
        if (fabs(lp.y) < DBL_MAX) smag = fmax(smag, fabs(lp.y));
    }
    smag = wave_max(smag);
    auto differ = [&](const double x, const double y) {
        if (x == -INFINITY || y == -INFINITY) {
            if (x != y) err = DBL_MAX;
        } else {
            err = fmax(err, fabs(x - (y + delta)) / fmax(smag, fmax(fabs(x), fabs(y + delta))));
        }
    };
    auto over_waves = [&]() {  // the largest over the workgroup, in every thread
        err = wave_max(err);
        if (lane == 0) part[wv] = err;
        __syncthreads();
        for (int i = 0; i < NT / 64; ++i) err = fmax(err, part[i]);
    };
    if (wv == 0 && lane < C) differ(v, va);
    const double err0 = err;
    if (PER == 0) {
#pragma unroll 8
        for (int i = tid; i < KC; i += NT) differ(A2[i], A[i]);
        over_waves();
    } else {
        double bx = -INFINITY, by = -INFINITY;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (u >= nu) x[u] = y[u] = -INFINITY;
            bx = fmax(bx, x[u]);
            by = fmax(by, y[u]);
        }
        newer[tid] = bx;
        newer[NT + tid] = by;
        __syncthreads();
        const double ng = c < C ? p.negl[(size_t)b * C + c] + VIT_TOL * smag : INFINITY;
        bx = by = -INFINITY;
        for (int g0 = 0; g0 < min(g, G); g0 += 8) {
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int q = min(g0 + i, g - 1) * C + c;
                bx = fmax(bx, newer[q]);
                by = fmax(by, newer[NT + q]);
            }
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            if (!(x[u] + ng <= bx && y[u] + ng <= by)) differ(x[u], y[u]);
            bx = fmax(bx, x[u]);
            by = fmax(by, y[u]);
        }
        over_waves();
    }
    if (tid == 0) {
        p.spec_err[o2] = err;
        p.spec_lr[o2] = delta;
    }
}

// Accepts or rejects a sequence after the second attempt; chains the additive constants (ckYA[b][j] = what must be added
// to the values stored by chunk j to get the true ones); best final label and score.  One wave; true if accepted.
__device__ __forceinline__ bool vit_settle_scan(const Params &p, const int b, const int lane)
{
    const int L = p.hdr[b].L, N = p.N, C = p.C, KC = p.K * C;
    const int nint = (L + p.Delta - 1) / p.Delta;
    const size_t so = ((size_t)b * 2) * (N + 1) + N + 1;
    double *off = p.ckYA + (size_t)b * (N + 1);
    // prefix sums of the constants in a fixed order: lane l owns boundaries 1 + l*per .. l*per + per,
    // sums them in order, the lane totals are scanned across the wave, then every lane walks its own
    const int per = (max(nint - 1, 0) + 63) / 64;
    const int j0 = 1 + lane * per, j1 = min(j0 + per, nint);
    double mine = 0.0, worst = 0.0;
#pragma unroll 4
    for (int j = j0; j < j1; ++j) {
        mine += p.spec_lr[so + j];
        worst = fmax(worst, p.spec_err[so + j]);
    }
    worst = wave_max(worst);
    double incl = mine;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double up = __shfl_up(incl, o);
        if (lane >= o) incl += up;
    }
    double run = incl - mine;
    for (int j = j0; j < j1; ++j) {
        run += p.spec_lr[so + j];
        off[j] = run;
    }
    const double total = __shfl(incl, 63);
    const bool ok = worst <= VIT_TOL;
    if (ok) {
        const double *e = p.ckA2 + ((size_t)b * (N + 1) + nint) * ((size_t)KC + C);
        const double v = lane < C ? (nint > 0 ? e[KC + lane] : 0.0) : -INFINITY;
        vit_best(p, b, v, lane, lane < C, total);
    }
    if (lane == 0) {
        off[0] = 0.0;
        p.spec_ok[b * 2] = ok ? 1 : 0;
        p.spec_rep[b * 2] = worst;
        p.spec_ok[b * 2 + 1] = 0;  // there is no scan in the other direction
        p.spec_rep[b * 2 + 1] = -1.0;
    }
    return ok;
}

// The verdict on the chunk-parallel scan of a sequence, and the sequential scan where there is none or it was rejected:
// one wave per sequence.
template <int CT, int NKW>
__global__ __launch_bounds__(64) void k_viterbi(Params p)
{
    extern __shared__ double lds_raw[];
    if (p.spec && vit_settle_scan(p, blockIdx.x, threadIdx.x)) return;
    vit_task<CT, NKW, true>(p, lds_raw, blockIdx.x, 0, 0);
}

// ---------------------------------------------------------------------------
// Trace-back.  Node (t, c) = "a segment with label c ends at position t"; its duration is the smallest k that
// maximises dur[k,c] + r_{t-k}(c), the label of the node before it (at t - k) the smallest c' that maximises
// V_{t-k}(c') + trans[c',c] (both up to ties as above; V_t(c) and r_{t-k}(c') show how large the prefix sums are).  Only nodes that a path runs through are looked at.
// Paths merge going back just as the scan's states do going forward, so a path is followed in pieces that are traced side
// by side and verified against each other.  A piece of n tokens [lo, hi) follows a path from the best node a few positions
// above hi down to lo; it came in by the lowest node at a position >= hi and leaves by the lowest at a position >= lo.
// Where the piece above leaves by another node than the one by which this piece came in, it is traced again from there, until
// every boundary agrees.  What starts at the root is right, so by induction all of it is THE path.
//   k_vit_trace   one workgroup per tile of VT_PIECES pieces, with the rows of V and r that they can reach in LDS and 16
//                 lanes per piece; tiles among each other are pieces again.  RETRY: the tiles that did not agree with the
//                 tile above, from the node by which that one left.
//   k_vit_settle  one workgroup per sequence: the tiles that do not even then, from the top down.
// A tile writes its own tokens only, so a wrong path is overwritten where it was written.  The retry reads the records of
// the first pass and writes others (which the first pass has filled too, for the tiles with nothing to do): no workgroup
// reads what another of its launch writes.  Where two records name the same node, they name the same path below it: the start of its segment
// is a function of the node.
// What bounds it: the instructions of the chain of a path's nodes (from global memory instead of LDS, two loads of ~1000
// clocks per node: 208 us at the genomic shape), then the reading of V and r.  A row of 16 lanes has one path because maxima
// along a row are cheap, and 24 labels or a few dozen durations do not fill a wave.
// ---------------------------------------------------------------------------
constexpr int VT_THREADS = 512;
constexpr int VT_PIECES = VT_THREADS / 16;
constexpr int VT_WARM = 4;  // warm-up of a piece inside its tile

// Tokens per piece n (tile: VT_PIECES n tokens): the most with which a compute unit holds two tiles, so that one loads while
// the other follows its paths.  A tile's own warm-up is 4 n - 1 positions, so that it reads vit_tile_rows positions.
inline __host__ __device__ int vit_tile_rows(const int n) { return VT_PIECES * n + 4 * n; }
inline __host__ __device__ int vit_row_floats(const int n) { return ((n + 15) & ~15) + 1; }
inline __host__ __device__ int vit_r_stride(const int n, const int K) { return (vit_tile_rows(n) + K) | 1; }  // max(lo - K, 0) .. top
inline size_t vit_tile_lds(const int n, const int K, const int C)
{
    return ((size_t)C * vit_r_stride(n, K) + (size_t)(vit_tile_rows(n) + 1) * C + vit_tile_rows(n) + K + 1) * sizeof(double) +
           ((size_t)C * vit_row_floats(K) + (size_t)(C + 1) * vit_row_floats(C)) * sizeof(float);
}
constexpr int VT_TILE_MIN = 2 * VT_PIECES;  // fewest tokens of a tile
inline int vit_piece_tokens(const int K, const int C)
{
    int n = 8;
    while (n > VT_TILE_MIN / VT_PIECES && vit_tile_lds(n, K, C) > LDS_LIMIT / 2 - 1024) n >>= 1;
    return n;
}

// max and min along a row of 16 lanes, in each of its lanes
__device__ __forceinline__ double row16_max(double v)
{
    v = max_row_ror<8>(v);
    v = max_row_ror<4>(v);
    v = max_row_ror<2>(v);
    return max_row_ror<1>(v);
}
__device__ __forceinline__ int row16_min(int v)
{
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x128, 0xf, 0xf, true));
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x124, 0xf, 0xf, true));
    v = min(v, __builtin_amdgcn_update_dpp(0, v, 0x122, 0xf, 0xf, true));
    return min(v, __builtin_amdgcn_update_dpp(0, v, 0x121, 0xf, 0xf, true));
}

// A tile's share of V and r, and the tables: dur by label, then trans by the label it leads to and a row of zeros (rows
// padded with -infinity to whole turns of 16 lanes, and by one so that they start in different banks).
struct VitTile {
    double *r;     // [C][rs]: r_s(c) at [c][s - rbase]
    double *v;     // [..][C]: V_s(c) at [s - vbase][c]
    double *unit;  // [..]: additive constant of position rbase + i
    float *dur, *tr;
    int K, C, ks, cs, rs, rbase, vbase;

    __device__ __forceinline__ VitTile(const Params &p, double *lds, const int n)
    {
        K = p.K;
        C = p.C;
        ks = vit_row_floats(K);
        cs = vit_row_floats(C);
        rs = vit_r_stride(n, K);
        rbase = vbase = 0;
        r = lds;
        v = r + C * rs;
        unit = v + (vit_tile_rows(n) + 1) * C;
        dur = (float *)(unit + vit_tile_rows(n) + K + 1);
        tr = dur + C * ks;
    }
    __device__ __forceinline__ void load_tables(const Params &p) const
    {
        const int tid = threadIdx.x;
        // 16 lanes to a row, rows in turn
        for (int c = tid >> 4; c < C; c += VT_PIECES) {
#pragma unroll 4
            for (int k = tid & 15; k < ks - 1; k += 16) dur[c * ks + k] = k < K ? p.dur[(size_t)k * C + c] : -INFINITY;
        }
        for (int c = tid >> 4; c <= C; c += VT_PIECES) {
#pragma unroll 4
            for (int o = tid & 15; o < cs - 1; o += 16)
                tr[c * cs + o] = o < C ? (c < C ? p.trans[(size_t)o * C + c] : 0.f) : -INFINITY;
        }
    }
    // V of positions lo .. top and r of positions max(lo - K, 0) .. top, in the unit of the whole sequence
    __device__ __forceinline__ void load_rows(const Params &p, const int b, const int lo, const int top)
    {
        const int tid = threadIdx.x;
        const size_t ts = (size_t)p.T + 1;
        rbase = max(lo - K, 0);
        vbase = lo;
        const int nr = top - rbase + 1;
        const bool chunked = p.spec && p.spec_ok[b * 2];
        const double *u = p.ckYA + (size_t)b * (p.N + 1);
        // r: 256 threads along the positions, in two groups that take the labels in turn
        const double *R = p.vrt + (size_t)b * ts * C + rbase;
        for (int i = tid & 255; i < nr; i += 256) {
            const int s = rbase + i;
            const double x = chunked ? u[s == 0 ? 0 : (unsigned)(s - 1) / (unsigned)p.Delta] : 0.0;
            if (tid < 256) unit[i] = x;
#pragma unroll 8
            for (int c = tid >> 8; c < C; c += VT_THREADS / 256) r[c * rs + i] = R[c * ts + i] + x;
        }
        __syncthreads();
        const double *V = p.vv + ((size_t)b * ts + lo) * C;
        const double *uv = unit + (lo - rbase);
        const unsigned nv = (unsigned)(top - lo + 1) * C;
#pragma unroll 8
        for (unsigned i = tid; i < nv; i += VT_THREADS) {
            const double x = V[i];
            v[i] = x + uv[i / (unsigned)C];
        }
        __syncthreads();
    }
    // Duration of the segment that ends at (t, c); l: lane of the row.  KU: candidates per lane.  Up to 16 stay in registers
    // between the search for the best one and the search for the first that ties with it; of more, the largest of every
    // four does, and the first four with one that ties are looked at again (32 in registers leave a compute unit one tile
    // fewer: whole call at 5 x 84 374, K = 388, C = 4 1188 us, all looked at again 1056, so 1044).
    template <int KU>
    __device__ __forceinline__ int duration(const int t, const int c, const int l) const
    {
        const double *rc = r + c * rs + (t - 1 - rbase);
        const float *dc = dur + c * ks;
        const int lim = min(K, t);
        constexpr int NX = KU <= 16 ? KU : 4;
        double x[NX], best = -INFINITY;
        float d[NX];
        auto load = [&](const int i0) {  // (lanes beyond the last candidate repeat it: nothing waits in a branch)
#pragma unroll
            for (int u = 0; u < NX; ++u) {
                const int i = min(i0 + 16 * u, lim - 1);
                x[u] = rc[-i];
                d[u] = dc[i];
            }
        };
        auto add = [&](const int i0) {
#pragma unroll
            for (int u = 0; u < NX; ++u) x[u] = i0 + 16 * u < lim ? x[u] + (double)d[u] : -INFINITY;
        };
        int at = 0x7fffffff;
        if constexpr (KU <= 16) {
            load(l);
            const double slack = vit_slack(v[(t - vbase) * C + c]);
            add(l);
#pragma unroll
            for (int u = 0; u < NX; ++u) best = fmax(best, x[u]);
            best = row16_max(best);
            const double floor = vit_floor(best) - slack;
#pragma unroll
            for (int u = NX - 1; u >= 0; --u) at = x[u] >= floor ? l + 16 * u : at;
        } else {
            double top[KU / 4];
            const double slack = vit_slack(v[(t - vbase) * C + c]);
#pragma unroll
            for (int q = 0; q < KU / 4; ++q) {
                top[q] = -INFINITY;
                if (K > 64 * q) {  // uniform
                    load(l + 64 * q);
                    add(l + 64 * q);
                    top[q] = fmax(fmax(x[0], x[1]), fmax(x[2], x[3]));
                }
                best = fmax(best, top[q]);
            }
            best = row16_max(best);
            const double floor = vit_floor(best) - slack;
            int i0 = -1;
#pragma unroll
            for (int q = KU / 4 - 1; q >= 0; --q) i0 = top[q] >= floor ? l + 64 * q : i0;
            if (i0 >= 0) {
                load(i0);
                add(i0);
#pragma unroll
                for (int u = NX - 1; u >= 0; --u) at = x[u] >= floor ? i0 + 16 * u : at;
            }
        }
        at = row16_min(at);
        return (best > -INFINITY ? at : 0) + 1;
    }
    // label of the node at s before one with label c (c = C: the best label at s); CU: labels per lane
    template <int CU>
    __device__ __forceinline__ int label(const int s, const int c, const int l) const
    {
        const double *vs = v + (s - vbase) * C, *rr = r + (s - rbase);
        const float *tc = tr + c * cs;
        double x[CU], z[CU], best = -INFINITY;
        float d[CU];
#pragma unroll
        for (int u = 0; u < CU; ++u) {
            const int o = min(l + 16 * u, C - 1);
            x[u] = vs[o];
            z[u] = rr[o * rs];
            d[u] = tc[l + 16 * u];  // -infinity beyond the last label: CU is the fewest shares, so rows are padded to 16 CU
        }
#pragma unroll
        for (int u = 0; u < CU; ++u) {
            x[u] += (double)d[u];
            best = fmax(best, x[u]);
            x[u] += vit_slack(z[u]);
        }
        best = row16_max(best);
        const double floor = vit_floor(best);
        int at = 0x7fffffff;
#pragma unroll
        for (int u = CU - 1; u >= 0; --u) at = x[u] >= floor ? l + 16 * u : at;
        at = row16_min(at);
        return best > -INFINITY ? at : 0;
    }
};

// Lanes' shares of the durations and labels as compile-time sizes.  First pass at the genomic shape (KU = 4, CU = 2): 164 us so;
// one kernel with four candidates per lane for all sizes 192 us, with runtime loops instead 213 us (and 168 us without the
// second search, where rounding decided the ties).
template <int KU_, int CU_>
struct VitShape {
    static constexpr int KU = KU_, CU = CU_;  // K <= 16 KU, 16 (CU - 1) < C <= 16 CU
};

// Traces tile j of sequence b (at least one token of it lies in the sequence).  from: the node (t C + c) by which the tile
// above left, and the position where its segment starts (-1: not known); from.x < 0: start at the warm-up's best node.
// rec, also: where the tile's record goes.
template <class SH>
__device__ __forceinline__ void vit_tile(const Params &p, VitTile &tile, const int b, const int j, const int n, const int2 from,
                                         int4 *rec, int4 *also)
{
    __shared__ int in[VT_PIECES];
    __shared__ int2 out[VT_PIECES];
    __shared__ int starts;
    const int C = p.C, T = p.T, L = p.hdr[b].L, tid = threadIdx.x, i = tid >> 4, l = tid & 15;
    const int tlo = j * n * VT_PIECES, thi = min(tlo + n * VT_PIECES, L);
    const int top = from.x < 0 ? min(thi + 4 * n - 1, L) : thi;
    const int last = (thi - tlo - 1) / n;  // piece that ends at the tile's upper end
    const int lo = tlo + i * n, hi = min(lo + n, L);
    const int u = lo + l;  // the lane's token (l < n)
    if (tid == 0) starts = 0;
    tile.load_rows(p, b, tlo, top);
    int lab = -1, st = 0;
    auto trace = [&](int t, int c, int s) {  // s: start of the segment that ends at (t, c), -1: not known
        lab = -1;
        st = 0;
        int entry = t * C + c;
        bool inside = false;
        int2 leave = make_int2(0, -1);
        for (;;) {
            if (t == lo) {
                leave = make_int2(t * C + c, -1);
                break;
            }
            if (s < 0) s = t - tile.template duration<SH::KU>(t, c, l);
            if (s < hi) {
                if (!inside) entry = t * C + c;
                inside = true;
                if (u >= s && u < t) {
                    lab = c;
                    st = u == s;
                }
            }
            if (s < lo) {
                leave = make_int2(t * C + c, s);
                break;
            }
            c = tile.template label<SH::CU>(s, c, l);
            t = s;
            s = -1;
        }
        if (l == 0) {
            in[i] = entry;
            out[i] = leave;
        }
    };
    if (i <= last) {
        if (i == last && from.x >= 0) {
            trace(from.x / C, from.x % C, from.y);
        } else {
            const int t = i == last ? top : min(hi + VT_WARM, top);
            trace(t, t == L ? p.vbest[b] : tile.template label<SH::CU>(t, C, l), -1);
        }
    }
    for (int round = 0; round < VT_PIECES; ++round) {  // the last piece is right; each round makes one more right
        __syncthreads();
        const int2 above = i < last ? out[i + 1] : make_int2(0, 0);
        const bool wrong = i < last && in[i] != above.x;
        if (!__syncthreads_or(wrong)) break;
        if (wrong) trace(above.x / C, above.x % C, above.y);
    }
    if (l < n && u < min(tlo + n * VT_PIECES, T)) {
        p.vlabels[(size_t)b * T + u] = u < L ? lab : -1;
        p.vstarts[(size_t)b * T + u] = u < L ? st : 0;
    }
    const int count = __popcll(__ballot(l < n && u < thi && st));
    if ((tid & 63) == 0 && count) atomicAdd(&starts, count);
    __syncthreads();
    if (tid == 0) *rec = *also = make_int4(in[last], out[0].x, out[0].y, starts);
}

template <bool RETRY, class SH>
__global__ __launch_bounds__(VT_THREADS) void k_vit_trace(Params p, int n)
{
    extern __shared__ double lds_raw[];
    const int b = blockIdx.y, j = blockIdx.x, T = p.T, L = p.hdr[b].L, nt = n * VT_PIECES, lo = j * nt;
    if (lo >= L) {
        if (!RETRY) {  // tokens beyond the sequence
            for (int u = lo + threadIdx.x; u < min(lo + nt, T); u += VT_THREADS) {
                p.vlabels[(size_t)b * T + u] = -1;
                p.vstarts[(size_t)b * T + u] = 0;
            }
        }
        return;
    }
    const size_t o = (size_t)b * gridDim.x + j;
    int2 from = make_int2(-1, -1);
    if (RETRY) {
        if (lo + nt >= L) return;
        const int4 mine = p.vtile[0][o], above = p.vtile[0][o + 1];
        from = make_int2(above.y, above.z);
        if (mine.x == from.x) return;
    }
    VitTile tile(p, lds_raw, n);
    tile.load_tables(p);
    vit_tile<SH>(p, tile, b, j, n, from, p.vtile[1] + o, p.vtile[RETRY ? 1 : 0] + o);
}

template <class SH>
__global__ __launch_bounds__(VT_THREADS) void k_vit_settle(Params p, int n)
{
    extern __shared__ double lds_raw[];
    __shared__ int total[VT_THREADS / 64];
    const int b = blockIdx.x, tid = threadIdx.x, nt = n * VT_PIECES;
    const int npl = (p.hdr[b].L + nt - 1) / nt;
    int4 *rec = p.vtile[1] + (size_t)b * ((p.T + nt - 1) / nt);
    int again = 0;
    for (int j = tid; j < npl - 1; j += VT_THREADS) again |= rec[j].x != rec[j + 1].y;
    if (__syncthreads_or(again)) {  // rarely
        VitTile tile(p, lds_raw, n);
        tile.load_tables(p);
        for (int j = npl - 2; j >= 0; --j) {
            const int2 from = make_int2(rec[j + 1].y, rec[j + 1].z);
            if (rec[j].x != from.x) vit_tile<SH>(p, tile, b, j, n, from, rec + j, rec + j);
            __threadfence_block();
            __syncthreads();
        }
    }
    int cnt = 0;
    for (int j = tid; j < npl; j += VT_THREADS) cnt += rec[j].w;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) cnt += __shfl_xor(cnt, off);
    if ((tid & 63) == 0) total[tid >> 6] = cnt;
    __syncthreads();
    if (tid == 0) {
        for (int i = 1; i < VT_THREADS / 64; ++i) cnt += total[i];
        p.vnseg[b] = cnt;
    }
}

// ---------------------------------------------------------------------------
// The same path by pointer doubling over all nodes (SEMICRF_VITERBI_GLOBAL_TRACE): looks at every node, at a cost that
// does not depend on the data; kept as the other side of the comparison.
// 1. k_vit_bp: duration and predecessor label of every node.
//    A tile of 32 positions per workgroup with the K + 32 rows of (V, r) it can
//    reach staged in LDS.  parent(t, c) = (t - k, c'); nodes at position 0 are their own parent.
// 2. k_vit_round, ceil(log2(T+1)) times: every marked node marks the node its current
//    pointer leads to, then every pointer is replaced by the pointer's pointer.  After round i
//    the marked nodes are the root's ancestors at distances < 2^(i+1): the best path.
// 3. k_vit_emit: every marked node writes its segment's tokens.
constexpr int VBP_TILE = 32;

__global__ __launch_bounds__(NT) void k_vit_bp(Params p)
{
    extern __shared__ double lds_raw[];
    const int b = blockIdx.y, tid = threadIdx.x;
    const int K = p.K, C = p.C, T = p.T;
    const int L = p.hdr[b].L;
    const int t0 = blockIdx.x * VBP_TILE;
    const int rows = K + VBP_TILE, sbase = t0 - K;  // LDS row i holds position sbase + i
    double *vv = lds_raw;                            // [rows][C]  V
    double *rr = lds_raw + (size_t)rows * C;         // [rows][C]  r
    const size_t nn = (size_t)(T + 1) * C;
    const double *VV = p.vv + (size_t)b * nn, *RT = p.vrt + (size_t)b * nn;
    // values stored by an accepted chunk-parallel scan are in their chunk's additive unit
    const bool chunked = p.spec && p.spec_ok[b * 2];
    const double *unit = p.ckYA + (size_t)b * (p.N + 1);
    for (int i = tid; i < rows * C; i += NT) {
        const int sp = sbase + i / C;
        double2 x = make_double2(-INFINITY, -INFINITY);
        if (sp >= 0 && sp <= L) {
            x = make_double2(VV[(size_t)sp * C + i % C], RT[(size_t)(i % C) * (T + 1) + sp]);
            if (chunked) {
                const double u = unit[sp == 0 ? 0 : (sp - 1) / p.Delta];
                x.x += u;
                x.y += u;
            }
        }
        vv[i] = x.x;
        rr[i] = x.y;
    }
    if (blockIdx.x == 0 && tid == 0) p.vnseg[b] = 0;
    __syncthreads();
    int *bp = p.vbp + (size_t)b * nn, *par = p.vpar[0] + (size_t)b * nn;
    unsigned char *mark = p.vmark + (size_t)b * nn;
    for (int j = tid; j < VBP_TILE * C; j += NT) {
        const int t = t0 + j / C, c = j % C;
        if (t > T) continue;
        const size_t n = (size_t)t * C + c;
        mark[n] = 0;
        if (t < 1 || t > L) {
            bp[n] = 0;
            par[n] = (int)n;
            continue;
        }
        const int kmax = min(K, t);
        const double *rcol = rr + (size_t)(t - sbase) * C + c;  // r_{t-k}(c) at rcol[-k*C]
        auto by_duration = [&](const int k) { return (double)p.dur[(size_t)(k - 1) * C + c] + rcol[-(k * C)]; };
        double best = -INFINITY;
        for (int k = 1; k <= kmax; ++k) best = fmax(best, by_duration(k));
        const double floor = vit_floor(best) - vit_slack(vv[(size_t)(t - sbase) * C + c]);
        int kb = 1;
        if (best > -INFINITY)
            while (kb < kmax && !(by_duration(kb) >= floor)) ++kb;
        const int sp = t - kb;
        const double *vrow = vv + (size_t)(sp - sbase) * C, *rrow = rr + (size_t)(sp - sbase) * C;
        auto by_label = [&](const int o) { return vrow[o] + (double)p.trans[(size_t)o * C + c]; };
        best = -INFINITY;
        for (int o = 0; o < C; ++o) best = fmax(best, by_label(o));
        const double lfloor = vit_floor(best);
        int cb = 0;
        if (best > -INFINITY)
            while (cb < C - 1 && !(by_label(cb) + vit_slack(rrow[cb]) >= lfloor)) ++cb;
        bp[n] = (kb << 8) | cb;
        par[n] = sp * C + cb;
    }
}

__global__ __launch_bounds__(NT) void k_vit_round(Params p, int src, int first)
{
    const int b = blockIdx.y;
    const size_t nn = (size_t)(p.T + 1) * p.C;
    const size_t n = (size_t)blockIdx.x * NT + threadIdx.x;
    if (n >= nn) return;
    const int *pin = p.vpar[src] + (size_t)b * nn;
    int *pout = p.vpar[src ^ 1] + (size_t)b * nn;
    unsigned char *mark = p.vmark + (size_t)b * nn;
    const int par = pin[n];
    const bool root = first && n == (size_t)p.hdr[b].L * p.C + p.vbest[b];
    if (root) mark[n] = 1;
    if (root || mark[n]) mark[par] = 1;  // a mark set earlier in this launch only arrives sooner
    pout[n] = pin[par];
}

__global__ __launch_bounds__(NT) void k_vit_emit(Params p)
{
    const int b = blockIdx.y, C = p.C, T = p.T;
    const int L = p.hdr[b].L;
    const size_t nn = (size_t)(T + 1) * C;
    const size_t n = (size_t)blockIdx.x * NT + threadIdx.x;
    if (n >= nn) return;
    const int t = (int)(n / (unsigned)C), c = (int)(n - (size_t)t * C);
    int32_t *lab = p.vlabels + (size_t)b * T, *st = p.vstarts + (size_t)b * T;
    if (c == 0 && t >= 1 && t - 1 >= L) {  // token t-1 lies beyond the sequence
        lab[t - 1] = -1;
        st[t - 1] = 0;
    }
    if (t < 1 || t > L || !p.vmark[(size_t)b * nn + n]) return;
    const int k = p.vbp[(size_t)b * nn + n] >> 8;
    for (int u = t - k; u < t; ++u) {
        lab[u] = c;
        st[u] = u == t - k ? 1 : 0;
    }
}

// nseg[b] = number of start flags (zeroed by k_vit_bp): one integer atomic per 8192 tokens, not
// one per segment, which would serialise on one address.
constexpr int VCNT_TOK = 8192;

__global__ __launch_bounds__(NT) void k_vit_count(Params p)
{
    const int b = blockIdx.y;
    const int L = p.hdr[b].L;
    const int32_t *st = p.vstarts + (size_t)b * p.T;
    const int lo = blockIdx.x * VCNT_TOK, hi = min(L, lo + VCNT_TOK);
    int cnt = 0;
    for (int u = lo + threadIdx.x; u < hi; u += NT) cnt += st[u];
#pragma unroll
    for (int off = 32; off; off >>= 1) cnt += __shfl_xor(cnt, off);
    if ((threadIdx.x & 63) == 0 && cnt) atomicAdd(&p.vnseg[b], cnt);
}
