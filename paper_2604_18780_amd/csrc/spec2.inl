// The chunk-parallel scan tasks with TWO waves per task.
// Included by semicrf.hip inside its anonymous namespace (after spec.inl); not a translation unit of its own.

// ---------------------------------------------------------------------------
// A one-wave scan task (spec.inl) issues about 135 instructions per position, and how fast a
// compute unit's SIMDs issue the instructions of the few waves they hold is what bounds it.
// Here a task is a workgroup of two waves that share the task's LDS window:
//   * the TIP runs the positions' dependent chains (product with ES, transition product, division)
//     and adds what the newest MB window entries and the block's own positions contribute
//     (durations 1 .. 2MB-1, from registers);
//   * the HELPER adds up, one block AHEAD, what all older window entries contribute to the MB
//     positions of the next block (durations > MB: every entry it needs is known before the tip
//     starts the current block), and hands the MB sums per label over through LDS.
// Each wave's stream is about half as long, four waves instead of two share a SIMD, and the
// helper's work is off the tip's chain.  One LDS-only workgroup barrier per block of MB positions.
// At a scaling-block boundary the tip publishes the exponent it found and scales its own registers;
// the helper rescales the window rows (the tip only writes rows the helper does not touch).  The
// helper also moves the window back when the linear buffer's end is reached.  Both waves walk the
// same sequence of blocks, so they execute the same barriers; checkpoints, stored rows and
// verification are those of the one-wave task.
// ---------------------------------------------------------------------------
template <int CT, int NKW>
__host__ __device__ constexpr size_t spec2_lds_doubles()
{
    const int CTP = pow2_ge8(CT);
    // window rows + MB spare rows at both ends (the helper's window starts MB rows behind the newest row),
    // two sets of MB far sums per label, the published exponent
    return (size_t)(scan_kw(CT, NKW) + scan_slack(CT, NKW, true) + 2 * MB) * CT + (size_t)(CTP - CT) + (size_t)2 * MB * CTP + 2;
}

template <int CT, int NKW, bool BWD, bool KEEP>
__device__ __forceinline__ void spec2_task(const Params &p, double *lds_raw, const int b, const int j,
                                           const int warm, const bool repair)
{
    using G = WaveWin<CT, NKW, 2>;
    using R = RowMap<CT>;
    constexpr int CTP = G::CTP, RS = G::RS, KW = G::KW, M = G::M, ROWS = G::ROWS, GW = G::GW, RUN = G::RUN, RUNS = G::RUNS;
    constexpr int H = G::H, HC = G::HC;
    constexpr int RTOT2 = (ROWS + 2 * MB) * RS + (CTP - CT);
    const int lane = threadIdx.x & 63;
    const bool tip = threadIdx.x < 64;
    const int K = p.K, C = p.C, KC = K * C;
    double *ring = lds_raw + MB * RS;   // logical row 0 (MB spare rows below, MB above)
    double *farb = lds_raw + RTOT2;     // [2][MB][CTP] what the older window entries add to the next block
    int *exv = (int *)(farb + 2 * MB * CTP);
    const int Delta = p.Delta, N = p.N;
    const size_t ckstride = (size_t)KC + C;
    const int c = R::label(lane), g = R::group(lane);
    const int hh = H == 2 ? (lane >> 5) : 0;
    const bool cval = c < C;
    const int cc = cval ? c : 0;
    const SeqHdr h = p.hdr[b];
    const int L = h.L, J = h.J, Jm = J - 1;
    const int lo = j * Delta;
    if (lo >= L) return;   // both waves
    const int hi = min(lo + Delta, L);
    const size_t row0 = (size_t)b * (p.T + 1);
    const int *nbc = p.nbase + row0 * C + cc;
    const int s0 = repair ? (BWD ? hi : lo) : (BWD ? min(hi + warm, L) : max(lo - warm, 0));
    const int tstart = BWD ? hi : lo;   // where the chunk proper begins (state -> ck1)
    const int tend = BWD ? lo : hi;

    // ---- what both waves compute alike: the sequence of blocks and the window's row
    auto block_len = [&](const int tcur) {  // positions the block starting after tcur may take
        int nb = BWD ? tcur - tend : tend - tcur;
        nb = min(nb, MB);
        // only the first position of a block may cross a scaling-block boundary
        nb = min(nb, BWD ? ((tcur - 1) & Jm) + 1 : J - ((tcur + 1) & Jm));
        // the position where the chunk proper starts ends its block (its state is recorded)
        if (BWD ? tcur > tstart : tcur < tstart) nb = min(nb, BWD ? tcur - tstart : tstart - tcur);
        return nb;
    };
    auto at_boundary = [&](const int tcur) { return BWD ? (tcur & Jm) == 0 : ((tcur + 1) & Jm) == 0; };
    auto must_move = [&](const int rcur) { return BWD ? rcur < MB : rcur + MB > ROWS - 1; };
    // exponent step n_j(c) - n_{j-1}(c) of the lane's label at the scaling-block boundary j*J; the
    // one of the next boundary in the scan's direction is loaded one block of J early
    auto nbdelta = [&](const int jb) {
        return (jb >= 1 && (long)jb * J <= (long)L) ? nbc[(size_t)jb * C] - nbc[(size_t)(jb - 1) * C] : 0;
    };

    // ---- start: the state of a sequence that begins (forward) / ends (backward) at s0
    for (int i = threadIdx.x; i < RTOT2; i += 128) lds_raw[i] = 0.0;
    for (int i = threadIdx.x; i < 2 * MB * CTP; i += 128) farb[i] = 0.0;
    lds_barrier();
    int r = BWD ? M : KW - 1;  // row of the newest message
    const int bs = BWD ? j + 1 : j;  // repair: the reached state at this boundary is the start (window by both waves)
    const double *reached = (BWD ? p.ckB2 : p.ckA2) + ((size_t)b * (N + 1) + bs) * ((size_t)KC + C);
    if (repair) {
        const int tm = s0 % K;
        for (int i = threadIdx.x; i < KC; i += 128) {
            const int sl = i / C, d = G::template slot_dist<BWD>(sl, tm, K);
            ring[(BWD ? r + d : r - d) * RS + (i - sl * C)] = reached[i];
        }
    }
    int t = s0;
    int jnx = BWD ? s0 / J : s0 / J + 1;
    int dnx = nbdelta(jnx);
    int nblk = 0;

    if (tip) {
        // ================================ the tip ================================
        const double2 *EIc = p.EI + row0 * C + cc;
        double wn[2 * MB - 1];   // W[1 .. 2MB-1, c]: durations inside a block and back to the MB newest entries
#pragma unroll
        for (int jj = 0; jj < 2 * MB - 1; ++jj) wn[jj] = (cval && jj + 1 <= K) ? p.W[(size_t)jj * C + c] : 0.0;
        double Ereg[HC];
#pragma unroll
        for (int i = 0; i < HC; ++i) {
            const int o = hh * HC + i;
            const bool ok = cval && o < C;
            Ereg[i] = ok ? (BWD ? p.Etr[(size_t)c * C + o] : p.Etr[(size_t)o * C + c]) : 0.0;
        }
        double ylast = 0.0;      // newest message vector, entry c (the same in every group; 0 beyond C)
        double Y = 0.0;
        if (repair) {
            if (cval) ylast = reached[KC + c];
            Y = ((BWD ? p.ckYB2 : p.ckYA2) + (size_t)b * (N + 1))[bs];
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
        auto record = [&](const int tt, double *ck, double *ckY) {
            const int tm = tt % K;
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
        const int istart = BWD ? j + 1 : j, iend = BWD ? j : j + 1;
        // rows for the interval stage / the stored-row marginals, as in the one-wave task
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
        auto load_rows = [&](double2 (&e)[MB], const int tfrom) {  // rows of the MB positions after tfrom
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                const int tt = BWD ? max(tfrom - 1 - i, tend) : min(tfrom + 1 + i, tend);
                e[i] = EIc[(size_t)tt * C];
            }
        };
        double2 e[MB];
        load_rows(e, t);
        lds_barrier();  // start: the helper may read the window
        if (repair) lds_barrier();  // ... and has added up what its older entries add to the first block
        while (t != tend) {
            const int nb = block_len(t);
            const int tn = BWD ? t - nb : t + nb;
            double2 en[MB];
            load_rows(en, tn);
            if (__builtin_expect(must_move(r), 0)) {
                lds_barrier();   // the helper moves the window back
                lds_barrier();
                r = BWD ? M : KW - 1;
            }
            const bool inchunk = keep && (BWD ? t <= tstart : t >= tstart);  // blocks end at tstart: holds for the whole block
            // what the window adds to this block: the helper's sums over the older entries, and the MB newest entries
            double far[MB], qp[MB];
            const double *fb = farb + (nblk & 1) * MB * CTP + c;
#pragma unroll
            for (int i = 0; i < MB; ++i) {
                far[i] = fb[i * CTP];
                qp[i] = ring[(BWD ? r + i : r - i) * RS + c];   // message of the position i before this block
            }
            if (__builtin_expect(at_boundary(t), 0)) {
                // sum of the newest message vector (the same value in every lane; only its exponent is used, and any
                // power of two would do: scaling is exact)
                const double prevsum = R::total(ylast);
                const int ex = safe_exponent(prevsum);
                Y += (double)ex;
                if (lane == 0) exv[0] = ex;
                const int sft = dnx - ex;
#pragma unroll
                for (int i = 0; i < MB; ++i) {
                    far[i] = fmin(ldexp(far[i], sft), DBL_MAX);
                    qp[i] = fmin(ldexp(qp[i], sft), DBL_MAX);
                }
                jnx += BWD ? -1 : 1;
                dnx = nbdelta(jnx);
                lds_barrier();   // the exponent is published (and the window entries above were read before it is rescaled)
            }
            double qn[MB];
            auto position = [&](const int i) {
                double x = far[i];
#pragma unroll
                for (int m = 0; m < MB; ++m) x = fma(wn[i + m], qp[m], x);        // duration i + 1 + m
#pragma unroll
                for (int jn = 0; jn < i; ++jn) x = fma(wn[i - 1 - jn], qn[jn], x);  // inside the block
                const double y = x * (BWD ? e[i].y : e[i].x);
                ylast = y;
                const double z = R::product(y, Ereg);
                qn[i] = z * (BWD ? e[i].x : e[i].y);
                if (writer) ring[(BWD ? r - 1 - i : r + 1 + i) * RS + c] = qn[i];
            };
            const int p0 = BWD ? t - 1 - lo : t + 1 - lo;  // slot row of the block's first position
            // (Not with 64 labels, whose positions are long next to their stores: a second copy of four positions takes the kernel from 54 to
            // 67 KB, past the 64 KB of instructions that two compute units hold, that of repeated scans from 107 to 130.  8 x 3000
            // positions, K = 20, C = 60, band 2, scans repeated 1370 -> 1386 us.)
            if (CT < 64 && __builtin_expect(nb == MB && (BWD || !inchunk || t + MB < hi), 1)) {
                // a whole block: nothing is decided per position, and it always issues the same stores (as in the one-wave task)
                const RowStore rows(aloc + (ptrdiff_t)(inchunk ? (BWD ? p0 - (MB - 1) : p0) : 0) * C, inchunk ? MB * C * 16 : 0);
                const RowStore scales(alocY + (inchunk ? (BWD ? p0 - (MB - 1) : p0) : 0), inchunk ? MB * 8 : 0);
                if (KEEP) scales.one((unsigned)(lane & (MB - 1)) * 8u, 0, Y - Yrec);
#pragma unroll
                for (int i = 0; i < MB; ++i) {
                    position(i);
                    if (KEEP) rows.pair(lane_row, (BWD ? MB - 1 - i : i) * C * 16, ylast, qn[i]);
                }
#pragma unroll
                for (int i = 0; i < MB; ++i) e[i] = en[i];
            } else {
#pragma unroll
                for (int i = 0; i < MB; ++i) {
                    if (i < nb) {
                        position(i);
                        if (inchunk && (BWD || t + 1 + i < hi)) {
                            const int at = BWD ? p0 - i : p0 + i;
                            if (writer) store_row(aloc + (size_t)at * C + c, ylast, qn[i]);
                            if (lane == 0) alocY[at] = Y - Yrec;
                        }
                    } else {
                        qn[i] = 0.0;
                    }
                }
#pragma unroll
                for (int i = 0; i < MB; ++i) e[i] = en[i];
            }
            lds_barrier();   // end of the block: the new window rows and the helper's sums for the next block are there
            r += BWD ? -nb : nb;
            t = tn;
            ++nblk;
            if (__builtin_expect(t == tstart, 0)) {
                record(t, ck1 + (size_t)istart * ckstride, ckY1 + istart);
                start_rows();
            }
        }
        record(tend, ck2 + (size_t)iend * ckstride, ckY2 + iend);
    } else {
        // ================================ the helper ================================
        double wx[RUNS][RUN + MB - 1];  // as in the one-wave task, for a window that begins MB positions behind a block's base
        const double wfar = G::load_weights(p, g, c, MB + 1, wx);
        double old = 0.0;
        // what the entries from row rb on (MB positions behind a block's base, and older) add to its MB positions
        auto far_sums = [&](const int rb, const int buf) {
            double acc[MB];
            G::template whole_window<BWD>(ring, rb, g, c, cval, wx, wfar, old, acc);
            double *fb = farb + buf * MB * CTP + c;
            if (g == 0) {
#pragma unroll
                for (int i = 0; i < MB; ++i) fb[i * CTP] = acc[i];
            }
        };
        lds_barrier();  // start
        if (repair) {
            // a mended task starts with a whole window: the first block has older entries, too (after a warm-up's start
            // there is only the newest one)
            old = G::template all_old<BWD>(ring, BWD ? r + MB : r - MB, g, c);
            far_sums(BWD ? r + MB : r - MB, 0);
            lds_barrier();
        }
        while (t != tend) {
            const int nb = block_len(t);
            const int tn = BWD ? t - nb : t + nb;
            if (__builtin_expect(must_move(r), 0)) {
                lds_barrier();
                r = G::template move<BWD>(ring, lane, r);
                lds_barrier();
            }
            if (__builtin_expect(at_boundary(t), 0)) {
                lds_barrier();   // the tip has published the exponent and read the newest entries
                const int sft = dnx - exv[0];
                jnx += BWD ? -1 : 1;
                dnx = nbdelta(jnx);
                // the KW rows that can still contribute, each lane its own label's column; the rows the tip
                // writes in this block lie beyond r and are already in the new frame
                if (cval) {
#pragma unroll 8
                    for (int d = g; d < KW; d += GW) {
                        double *q = ring + (BWD ? r + d : r - d) * RS + c;
                        *q = fmin(ldexp(*q, sft), DBL_MAX);
                    }
                }
                lds_wave_fence();
                old = fmin(ldexp(old, sft), DBL_MAX);
            }
            // what the entries at least MB positions before the NEXT block's base add to its MB positions
            // (the base is the last position of this block; its newest MB predecessors are the tip's)
            far_sums(BWD ? r - nb + MB : r + nb - MB, (nblk + 1) & 1);
            lds_barrier();   // end of the block
            r += BWD ? -nb : nb;
            t = tn;
            ++nblk;
        }
    }
}

template <int CT, int NKW, bool RETRY, bool ROWS>
__global__ __launch_bounds__(128, spec2_waves_per_simd(CT, NKW)) void k_spec2(Params p, int both, int warm, int tier, int rest)
{
    extern __shared__ double lds_raw[];
    const int ndir = both ? 2 : 1;
    const int dir = blockIdx.x % ndir;
    const int task = blockIdx.x / ndir;
    const int b = task / p.N, j = task % p.N;
    SpecJob job = {};
    if (RETRY) {
        job = spec_job(p, b, dir, j, ndir, warm, tier, threadIdx.x < 64);
        if (job.idle) return;  // accepted by an earlier attempt
    } else if (rest && p.hdr[b].J >= MS_JMIN) {
        return;
    }
    if (!RETRY || !job.mend) {
        const int w = RETRY ? job.warm : first_warm(p, b, warm);
        if (dir == 0) spec2_task<CT, NKW, false, ROWS>(p, lds_raw, b, j, w, false);
        else spec2_task<CT, NKW, true, ROWS>(p, lds_raw, b, j, w, false);
        return;
    }
    if (!spec_bad(job, dir ? j + 1 : j) || spec_bad(job, dir ? j + 2 : j - 1)) return;
    int jj = j;
    for (int n = 0; n < SPEC_RUN_MAX; ++n) {  // a run of boundaries is mended as in k_spec
        if (dir == 0) spec2_task<CT, NKW, false, ROWS>(p, lds_raw, b, jj, 0, true);
        else spec2_task<CT, NKW, true, ROWS>(p, lds_raw, b, jj, 0, true);
        const int nx = dir ? jj - 1 : jj + 1;
        if (nx < 0 || nx >= job.nint || !spec_bad(job, dir ? nx + 1 : nx)) break;
        __threadfence();
        __syncthreads();
        jj = nx;
    }
}
