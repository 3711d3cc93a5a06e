// The chunk-parallel scans: one-wave scan tasks with warm-up, the repair attempt, verification of the interval boundaries.
// Included by semicrf.hip inside its anonymous namespace (after common.h); not a translation unit of its own.

// ---------------------------------------------------------------------------
// Chunk-parallel scan.  A sequential scan of one sequence occupies one compute unit
// for T dependent steps.  The recurrences are positive linear maps, and products of
// positive maps forget their starting vector (up to scale) geometrically fast, so the
// ring state at a checkpoint position can instead be obtained by a short WARM-UP: start
// W positions earlier from the state a sequence beginning there would have, and run.
// Every checkpoint interval ("chunk") is then an independent task:
//   forward task j:  warm up over (j*Delta - W, j*Delta], record the state at j*Delta
//                    (-> ckA[j]), run the chunk, record the state at its end (-> ckA2[j+1]);
//   backward task j: the mirror image from above (-> ckB[j+1], ckB2[j]).
// Nothing is taken on trust: k_spec_cmp compares, for every chunk boundary, the state
// the previous chunk actually reached with the warm-up state the next chunk started
// from, entry by entry or by what an entry can still contribute, after removing their common scale
// factor.  If all boundaries of a (sequence, direction) agree (spec_tol) the warm-up states do what the
// sequential states do, to that relative accuracy (perturbations of the start do not grow: the maps
// are non-expansive in the projective metric).  The warm-up is 1.5 K positions, or what the model asks
// for (warm_plan): genomic shape 96 -> 32 (310 -> 278 us at 40); K = 512, C = 8 768 -> 44 (684 -> 388 us at 56);
// band 2 in 19 labels, K = 37 56 -> 264, so that the first attempt is accepted (225 -> 139 us).  spec_settle then chains the scale
// factors into the checkpoint scales and logZ.  Otherwise the flag stays 0 and the
// sequential scan kernel, launched after the later attempts, which returns at once for
// accepted (sequence, direction) pairs, recomputes that pair from scratch.
// One wave per task, no barriers, same register/LDS organisation as k_interval_wave.
// ---------------------------------------------------------------------------
constexpr int SPEC_RUN_MAX = 2;  // intervals one wave mends in a row in the repair attempt

// What an attempt does for one (sequence, direction) pair.
//   tier 0: every task after `warm` positions of warm-up.
//   tier 1, 2 (pairs that are still open): where a few isolated boundaries disagreed, mending: it is sequential work,
//   one task per run of disagreeing boundaries, and pays for a stretch of uninformative input, not for a model that
//   forgets slowly everywhere.  Otherwise every task again after a longer warm-up: at tier 1 what the mismatch of the
//   attempt before asks for, at tier 2 the longest.
// Whether the attempt before was accepted is worked out here, by every wave for its own pair (spec_verdict reads a few
// hundred numbers): the first task of the pair also settles it (settles: this wave is the one of its task to do so).  A launch
// in between for the verdicts alone would cost every call as much as a comparison.
struct SpecJob {
    bool idle, mend;
    int warm, nint;
    double tol;
    const double *err;
};
__device__ __forceinline__ SpecJob spec_job(const Params &p, const int b, const int dir, const int j, const int ndir,
                                            const int deflt, const int tier, const bool settles)
{
    const int warm = tier < 2 ? first_warm(p, b, deflt) : deflt;
    SpecJob s;
    s.idle = s.mend = false;
    s.warm = warm;
    s.nint = 0;
    s.tol = SPEC_TOL;
    s.err = p.spec_err + ((size_t)b * 2 + dir) * (p.N + 1);
    if (tier == 0) return s;
    const int lane = threadIdx.x & 63;
    if (tier > 1 && p.spec_ok[b * 2 + dir]) {
        s.idle = true;
        return s;
    }
    const SpecVerdict v = spec_verdict(p, b, dir, lane, tier - 1);
    s.tol = spec_tol(p, b, tier - 1);
    if (j == 0 && settles) spec_settle(p, b, dir, ndir, tier - 1, v, lane);
    s.idle = v.ok;
    s.nint = v.nint;
    s.mend = v.nbad <= max(2, v.nint / 16);
    if (tier == 1) {
        s.warm = second_warm(p, warm, v.worst);
    }
    return s;
}
// Boundary m disagreed in the attempt before.
__device__ __forceinline__ bool spec_bad(const SpecJob &s, const int m) { return m >= 1 && m <= s.nint - 1 && !(s.err[m] <= s.tol); }

// One scan task of the chunk-parallel scan, one wave (window and time blocking as above).
// repair: the task restarts from the state its neighbour in scan order REACHED at their common boundary (no
// warm-up: exact if the neighbour's own start was).
// KEEP: a call that keeps rows, whose tasks store theirs.  The others, scores and gradients of more tasks than there are row slots, do not even
// issue the stores (which would store nothing: scores at the genomic shape 196 -> 207 us; gradients of 55 x 6836 positions, K = 8,
// C = 25, 774 -> 752).
template <int CT, int NKW, bool BWD, bool KEEP>
__device__ __forceinline__ void spec_task(const Params &p, double *lds_raw, const int b, const int j,
                                          const int warm, const bool repair)
{
    using G = WaveWin<CT, NKW, 1>;
    using R = RowMap<CT>;
    constexpr int RS = G::RS, KW = G::KW, M = G::M, ROWS = G::ROWS, RUN = G::RUN, RUNS = G::RUNS;
    constexpr int RTOT = G::RTOT, H = G::H, HC = G::HC;
    const int lane = threadIdx.x & 63;
    const int K = p.K, C = p.C, KC = K * C;
    double *ring = lds_raw;          // [ROWS][RS] (+ pad)
    const int Delta = p.Delta, N = p.N;
    const size_t ckstride = (size_t)KC + C;
    const int c = R::label(lane), g = R::group(lane);
    const int hh = H == 2 ? (lane >> 5) : 0;
    const bool cval = c < C;
    const int cc = cval ? c : 0;
    const SeqHdr h = p.hdr[b];
    const int L = h.L, J = h.J, Jm = J - 1;
    const int lo = j * Delta;
    if (lo >= L) return;
    const int hi = min(lo + Delta, L);
    const size_t row0 = (size_t)b * (p.T + 1);
    const double2 *EIc = p.EI + row0 * C + cc;
    const int *nbc = p.nbase + row0 * C + cc;

    double wx[RUNS][RUN + MB - 1];  // weights of the durations of the lane's distances in each run, and of the next three
    const double wfar = G::load_weights(p, g, c, 1, wx);
    double wn[MB - 1];       // W[1..MB-1, c]: durations inside a block
#pragma unroll
    for (int jj = 0; jj < MB - 1; ++jj) wn[jj] = (cval && jj + 1 <= K) ? p.W[(size_t)jj * C + c] : 0.0;
    double Ereg[HC];
#pragma unroll
    for (int i = 0; i < HC; ++i) {
        const int o = hh * HC + i;
        const bool ok = cval && o < C;
        Ereg[i] = ok ? (BWD ? p.Etr[(size_t)c * C + o] : p.Etr[(size_t)o * C + c]) : 0.0;
    }
    // ---- start: the state of a sequence that begins (forward) / ends (backward) at s0
    const int s0 = repair ? (BWD ? hi : lo) : (BWD ? min(hi + warm, L) : max(lo - warm, 0));
    for (int i = lane; i < RTOT; i += 64) ring[i] = 0.0;
    lds_wave_fence();
    int r = BWD ? M : KW - 1;  // row of the newest message
    double ylast = 0.0;        // newest message vector, entry c (the same in every group; 0 beyond C)
    double Y = 0.0;
    double old = 0.0;          // sum of the entries of the label that went beyond the first run
    if (repair) {
        // the reached state at the boundary: K-deep window in slot order, message vector, scale
        const int bs = BWD ? j + 1 : j;
        const double *src = (BWD ? p.ckB2 : p.ckA2) + ((size_t)b * (N + 1) + bs) * ((size_t)KC + C);
        const int tm = s0 % K;
        for (int i = lane; i < KC; i += 64) {
            const int sl = i / C, col = i % C;
            const int d = G::template slot_dist<BWD>(sl, tm, K);
            ring[(BWD ? r + d : r - d) * RS + col] = src[i];
        }
        if (cval) ylast = src[KC + c];
        Y = ((BWD ? p.ckYB2 : p.ckYA2) + (size_t)b * (N + 1))[bs];
        lds_wave_fence();
        old = G::template all_old<BWD>(ring, r, g, c);
    } else {
        double q;
        if (!BWD) {
            double z = 0.0;
#pragma unroll
            for (int i = 0; i < HC; ++i) z += Ereg[i];
            if (H == 2) z = add_across_32(z);
            q = z * EIc[(size_t)s0 * C].y;
            ylast = cval ? 1.0 : 0.0;
        } else {
            q = EIc[(size_t)s0 * C].x;
            ylast = c == 0 ? 1.0 : 0.0;
        }
        if (cval && g == 0) ring[r * RS + c] = q;
    }
    lds_wave_fence();
    // checkpoint layout: message of position t' at slot t' mod K
    auto record = [&](const int t, double *ck, double *ckY) {
        const int tm = t % K;
        if (cval) {  // lane (g, c): the window rows at distances g, g + GW, ... of its label (no index divisions)
#pragma unroll 4
            for (int d = g; d < K; d += G::GW) {
                int sl = BWD ? tm + d : tm - d;  // slot of the position at that distance
                sl += BWD ? (sl >= K ? -K : 0) : (sl < 0 ? K : 0);
                ck[(size_t)sl * C + c] = ring[(BWD ? r + d : r - d) * RS + c];
            }
        }
        if (cval && g == 0) ck[KC + c] = ylast;
        if (lane == 0) *ckY = Y;
    };
    double *ck1 = (BWD ? p.ckB : p.ckA) + ((size_t)b * (N + 1)) * ckstride;
    double *ck2 = (BWD ? p.ckB2 : p.ckA2) + ((size_t)b * (N + 1)) * ckstride;
    double *ckY1 = (BWD ? p.ckYB : p.ckYA) + (size_t)b * (N + 1);
    double *ckY2 = (BWD ? p.ckYB2 : p.ckYA2) + (size_t)b * (N + 1);
    const int tstart = BWD ? hi : lo;   // where the chunk proper begins (state -> ck1)
    const int tend = BWD ? lo : hi;
    const int istart = BWD ? j + 1 : j, iend = BWD ? j : j + 1;
    // Forward tasks also leave the rows the interval stage needs, (a_t, q_t) and the scale relative
    // to the chunk's first position, for t = lo .. hi-1, in the task's own slot (the interval
    // stage then skips its forward recompute for accepted sequences).
    // Backward tasks do the same with (p_t, v_t) and the scale relative to the chunk's upper end,
    // for t = hi-1 .. lo, when the marginals are formed from the stored rows of both scans.
    const bool keep = KEEP && (BWD ? p.marg != 0 : p.fuse != 0);
    const bool writer = cval && g == 0;
    double2 *aloc = (double2 *)(BWD ? p.bloc : p.aloc) + ((size_t)b * N + j) * Delta * C;
    double *alocY = (BWD ? p.blocY : p.alocY) + ((size_t)b * N + j) * Delta;
    const unsigned lane_row = writer ? (unsigned)c * 16u : ROW_NOWHERE;
    double Yrec = 0.0;  // scale at the chunk's first position (forward) / upper end (backward)
    auto start_rows = [&]() {
        Yrec = Y;
        if (BWD) return;
        if (keep && writer) aloc[c] = make_double2(ylast, ring[r * RS + c]);
        if (keep && lane == 0) alocY[0] = 0.0;
    };
    if (s0 == tstart && !(BWD && tstart == L)) {
        record(s0, ck1 + (size_t)istart * ckstride, ckY1 + istart);
        start_rows();
    }

    int t = s0;
    auto load_rows = [&](double2 (&e)[MB], const int tfrom) {  // rows of the MB positions after tfrom
#pragma unroll
        for (int i = 0; i < MB; ++i) {
            const int tt = BWD ? max(tfrom - 1 - i, tend) : min(tfrom + 1 + i, tend);
            e[i] = EIc[(size_t)tt * C];
        }
    };
    auto block_len = [&](const int tcur) {  // positions the block starting after tcur may take
        int nb = BWD ? tcur - tend : tend - tcur;
        nb = min(nb, MB);
        // only the first position of a block may cross a scaling-block boundary
        nb = min(nb, BWD ? ((tcur - 1) & Jm) + 1 : J - ((tcur + 1) & Jm));
        // the position where the chunk proper starts ends its block (its state is recorded)
        if (BWD ? tcur > tstart : tcur < tstart) nb = min(nb, BWD ? tcur - tstart : tstart - tcur);
        return nb;
    };
    double2 e[MB];
    load_rows(e, t);
    // exponent step n_j(c) - n_{j-1}(c) of the lane's label at the scaling-block boundary j*J; the
    // one of the next boundary in the scan's direction is loaded one block of J early
    auto nbdelta = [&](const int jb) {
        return (jb >= 1 && (long)jb * J <= (long)L) ? nbc[(size_t)jb * C] - nbc[(size_t)(jb - 1) * C] : 0;
    };
    int jnx = BWD ? s0 / J : s0 / J + 1;
    int dnx = nbdelta(jnx);
    while (t != tend) {
        const int nb = block_len(t);
        const int tn = BWD ? t - nb : t + nb;
        // the next block's rows, requested before this block's stores: loads and stores retire in
        // order, so a load issued after a store could not be waited for without the store
        double2 en[MB];
        load_rows(en, tn);
        const int t1 = BWD ? t - 1 : t + 1;
        const bool inchunk = keep && (BWD ? t <= tstart : t >= tstart);  // blocks end at tstart: holds for the whole block
        const bool boundary = BWD ? (t & Jm) == 0 : (t1 & Jm) == 0;
        if (__builtin_expect(boundary, 0)) {
            // sum of the newest message vector; only its exponent is used, and any power of two would do: scaling
            // is exact
            const double prevsum = R::total(ylast);
            const int ex = safe_exponent(prevsum);
            Y += (double)ex;
            G::template rescale_live<BWD>(ring, g, c, cval, r, dnx - ex);
            old = fmin(ldexp(old, dnx - ex), DBL_MAX);
            jnx += BWD ? -1 : 1;
            dnx = nbdelta(jnx);
        }
        if (__builtin_expect(BWD ? r < MB : r + MB > ROWS - 1, 0)) r = G::template move<BWD>(ring, lane, r);
        // ---- what the window contributes to the MB positions of the block
        double acc[MB];
        G::template whole_window<BWD>(ring, r, g, c, cval, wx, wfar, old, acc);
        // ---- the positions one after the other
        double qn[MB];
        // A whole block (nearly all are): nothing is decided per position.  The rows of a block that lies in the
        // chunk go out through a buffer (the lanes that own no label store nothing), its scale once
        // for the MB positions; a block that has none issues the same stores, of nothing, and either kind of block takes over the next
        // block's rows itself: the compiler then knows how many stores lie behind those loads.  (Where it does not it waits for
        // all stores of the block before the next one begins: genomic training 522 -> 506 us, 456 with no rows stored at all.)
        // A forward block that reaches the chunk's end takes the general path (the end
        // position itself has no row).
        if (__builtin_expect(nb == MB && (BWD || !inchunk || t + MB < hi), 1)) {
            const int p0 = BWD ? t - 1 - lo : t + 1 - lo;  // slot row of the block's first position
            const RowStore rows(aloc + (ptrdiff_t)(inchunk ? (BWD ? p0 - (MB - 1) : p0) : 0) * C, inchunk ? MB * C * 16 : 0);
            const RowStore scales(alocY + (inchunk ? (BWD ? p0 - (MB - 1) : p0) : 0), inchunk ? MB * 8 : 0);
            if (KEEP) scales.one((unsigned)(lane & (MB - 1)) * 8u, 0, Y - Yrec);
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                double x = acc[i];
#pragma unroll
                for (int jn = 0; jn < i; ++jn) x = fma(wn[i - 1 - jn], qn[jn], x);
                const double y = x * (BWD ? e[i].y : e[i].x);
                ylast = y;
                const double z = R::product(y, Ereg);
                const double q = z * (BWD ? e[i].x : e[i].y);
                qn[i] = q;
                r += BWD ? -1 : 1;
                if (writer) ring[r * RS + c] = q;
                if (KEEP) rows.pair(lane_row, (BWD ? MB - 1 - i : i) * C * 16, y, q);
            }
#pragma unroll
            for (int i = 0; i < MB; ++i) e[i] = en[i];
        } else {
    #pragma unroll
            for (int i = 0; i < MB; ++i) {
                if (i < nb) {
                    double x = acc[i];
    #pragma unroll
                    for (int jn = 0; jn < i; ++jn) x = fma(wn[i - 1 - jn], qn[jn], x);
                    const double y = x * (BWD ? e[i].y : e[i].x);
                    ylast = y;
                    const double z = R::product(y, Ereg);
                    const double q = z * (BWD ? e[i].x : e[i].y);
                    qn[i] = q;
                    r += BWD ? -1 : 1;
                    if (writer) ring[r * RS + c] = q;
                    if (!BWD && inchunk && t + 1 + i < hi) {
                        if (writer) aloc[(size_t)(t + 1 + i - lo) * C + c] = make_double2(y, q);
                        if (lane == 0) alocY[t + 1 + i - lo] = Y - Yrec;
                    }
                    if (BWD && inchunk) {  // position t - 1 - i of [lo, hi)
                        if (writer) aloc[(size_t)(t - 1 - i - lo) * C + c] = make_double2(y, q);
                        if (lane == 0) alocY[t - 1 - i - lo] = Y - Yrec;
                    }
                } else {
                    qn[i] = 0.0;
                }
            }
#pragma unroll
            for (int i = 0; i < MB; ++i) e[i] = en[i];
        }
        lds_wave_fence();  // the block's new rows are read by other lanes from here on
        t = tn;
        if (__builtin_expect(t == tstart, 0)) {
            record(t, ck1 + (size_t)istart * ckstride, ckY1 + istart);
            start_rows();
        }
    }
    record(tend, ck2 + (size_t)iend * ckstride, ckY2 + iend);
}

// spec_waves(CT, NKW) independent tasks per workgroup, one per wave, no barrier between them.  A workgroup of four
// waves puts one on each SIMD; single-wave workgroups are placed as the launches before left the dispatcher, and two
// tasks on one SIMD with another SIMD idle decide how long the launch takes (forward-only genomic scan, 1024 tasks:
// 227 or 264 us depending on the shape of the kernel before).  The directions fill one half of the grid each, so that
// a SIMD with two tasks has one of each.
// rest: only the sequences the lock-step kernel (k_mscan, launched before) leaves out
// ROWS: KEEP of its tasks; kernels of their own for the same reason (all four kinds of tasks in one: speech 263 -> 268 us).
// RETRY: the later attempts; a kernel of its own, so that the first attempt is not compiled around their cases
// (one kernel for both: 304 -> 338 us at the genomic shape).
template <int CT, int NKW, bool RETRY, bool ROWS>
__global__ __launch_bounds__(64 * spec_waves(CT, NKW), spec_waves_per_simd(CT, NKW)) void k_spec(Params p, int both, int warm, int tier, int rest)
{
    constexpr int SW = spec_waves(CT, NKW);
    extern __shared__ double lds_raw[];
    const int per = both ? gridDim.x / 2 : gridDim.x;
    const int dir = (int)blockIdx.x >= per ? 1 : 0;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);  // the same in every lane: scalar registers
    const int task = ((int)blockIdx.x - dir * per) * SW + wave;
    const int b = task / p.N, j = task % p.N;
    if (b >= p.B) return;
    double *lds = lds_raw + (size_t)wave * scan_lds_doubles(CT, NKW);
    SpecJob job = {};
    if (RETRY) {
        job = spec_job(p, b, dir, j, both ? 2 : 1, warm, tier, true);
        if (job.idle) return;  // accepted by an earlier attempt
    } else if (rest && p.hdr[b].J >= MS_JMIN) {
        return;
    }
    if (!RETRY || !job.mend) {
        const int w = RETRY ? job.warm : first_warm(p, b, warm);
        if (dir == 0) spec_task<CT, NKW, false, ROWS>(p, lds, b, j, w, false);
        else spec_task<CT, NKW, true, ROWS>(p, lds, b, j, w, false);
        return;
    }
    // A run of adjacent boundaries that disagreed is taken by ONE wave, the task that starts at the first of them
    // in scan order (its neighbour started from a verified or exact state, so what that neighbour reached is
    // right): it restarts from the reached state and goes on through the run's intervals one after the other,
    // at most SPEC_RUN_MAX of them; a longer run stays open for the next attempt.  Every other task returns at
    // once and keeps what it has.  Nothing in this kernel writes spec_err.
    if (!spec_bad(job, dir ? j + 1 : j) || spec_bad(job, dir ? j + 2 : j - 1)) return;
    int jj = j;
    for (int n = 0; n < SPEC_RUN_MAX; ++n) {
        if (dir == 0) spec_task<CT, NKW, false, ROWS>(p, lds, b, jj, 0, true);
        else spec_task<CT, NKW, true, ROWS>(p, lds, b, jj, 0, true);
        const int nx = dir ? jj - 1 : jj + 1;              // the next task in scan order ...
        if (nx < 0 || nx >= job.nint || !spec_bad(job, dir ? nx + 1 : nx)) break;  // ... starts where this one ended
        __threadfence();  // the reached state this wave has just written is what it restarts from
        jj = nx;
    }
}

// The chunk-parallel scan was not attempted: say so in the report fields.
__global__ void k_spec_clear(Params p)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 2 * p.B) return;
    p.spec_ok[i] = 0;
    p.spec_rep[i] = -1.0;
}

__global__ void k_spec_report(Params p, int32_t *accepted, double *mismatch)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= 2 * p.B) return;
    if (accepted) accepted[i] = p.spec_ok[i];
    if (mismatch) mismatch[i] = p.spec_rep[i];
}

__global__ void k_seq_report(Params p, int32_t *range_exceeded, double *logz64)
{
    const int b = blockIdx.x * blockDim.x + threadIdx.x;
    if (b >= p.B) return;
    const SeqHdr h = p.hdr[b];
    if (range_exceeded) range_exceeded[b] = h.flags & 1;
    if (logz64) logz64[b] = h.logZ;
}

// The report fields sit in front of everything that differs between the gradient plans: the smallest plan of the
// caller's kind (forward only or gradients, default or low memory) locates them.
inline int report_plan_kind(int want_grad)
{
    if (want_grad < 0) return -1;
    return (want_grad & PLAN_LOW_MEMORY) | ((want_grad & 7) ? 2 : 0);
}

