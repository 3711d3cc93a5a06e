// ---------------------------------------------------------------------------
// Marginals from the stored rows of both scans (included by semicrf.hip inside its namespace).
//
// When the chunk-parallel forward AND backward scans of a sequence are accepted, both have left
// their per-position rows behind -- forward (a_t, q_t), backward (p_t, v_t), each with its
// power-of-two scale relative to its interval -- and every expected statistic of the "Gradient
// Formulas" section is a position-local product of the two:
//   duration     sum_t q_t(c) W[k,c] v_{t+k}(c) 2^(n_blk(t+k)(c) - n_blk(t)(c)) kappa(t, t+k)
//   transition   Etr[c',c] sum_t a_t(c') p_t(c) kappa(t, t)
//   emission     out_t(c) - in_t(c) = (q_t ES_t p_t - a_t v_t IE_t)(c) kappa(t, t)
//   kappa(t, s) = exp((Y_alpha(t) + Y_beta(s)) ln2 - logZ)
// (the power of two is what the backward recurrence applies to its window when it crosses the
// scaling blocks between t+k and t).  No recurrence is run again: Algorithm 3's per-interval
// backward pass has already happened inside the backward scan.  Two kernels, one workgroup per
// (sequence, interval) each; they write the same partials as the interval kernels (partD,
// partTr, the running emission sums, tot, sumR), which skip the sequences handled here.
// ---------------------------------------------------------------------------

// absolute log2 scale of the forward / backward row i of interval j
__device__ __forceinline__ double mg_ya(const Params &p, const int b, const int j, const int i)
{
    return p.ckYA[(size_t)b * (p.N + 1) + j] + p.alocY[((size_t)b * p.N + j) * p.Delta + i];
}

__device__ __forceinline__ double mg_yb(const Params &p, const int b, const int j, const int i, const int L)
{
    const int hi = min((j + 1) * p.Delta, L);
    const double top = hi == L ? 0.0 : p.ckYB[(size_t)b * (p.N + 1) + j + 1];
    return top + p.blocY[((size_t)b * p.N + j) * p.Delta + i];
}

// Duration-bias statistics by vector multiply-adds: short intervals next to the durations, and scaling blocks shorter than a
// tile of the matrix-core form below (J < 16, confident scores).  Thread (ks, c): label c, durations ks*MG_KS + 1 ..
// ks*MG_KS + MG_KS, one accumulator each: labels c0 .. c0 + CL - 1, strips s0 .. s1 - 1.  Positions are taken in groups inside one
// scaling block: the group's q rows and the v rows it can reach are staged in LDS, the latter converted to the group's frame with
// all exponents combined before anything is formed; four positions share every LDS read.  The
// absolute scales of all rows the interval can touch are fetched into LDS once, at the start.
__device__ __forceinline__ void mg_dur_vector(const Params &p, double *lds_raw, const int b, const int iv,
                                              const int c0, const int CL, const int s0, const int s1)
{
    const int tid = threadIdx.x, nth = blockDim.x;
    const int K = p.K, C = p.C, N = p.N, Delta = p.Delta;
    const SeqHdr h = p.hdr[b];
    const int L = h.L, J = h.J;
    const int lo = iv * Delta;
    const int hi = min(lo + Delta, L);
    const bool active = tid < CL * (s1 - s0);
    const int c = tid % CL, kA = (tid / CL) * MG_KS, kS = s0 * MG_KS;
    const int VR = MG_TG + MG_KS * (s1 - s0) + 3;
    double *Qrow = lds_raw;            // [MG_TG][CL]
    // rows of CP = CL|3 doubles: the threads of a wave read rows MG_KS apart (one per duration strip),
    // and MG_KS*CL is a multiple of the 32 banks (of 8 bytes) for every CL that is a multiple of 4;
    // with CP = 3 mod 4 the strips of a half-wave fall 24 banks apart instead of on top of each other
    const int CP = CL | 3;
    double *Vp = Qrow + MG_TG * CL;    // [VR][CP]
    double *qf = Vp + VR * CP;         // [MG_TG] per-row factors of the group
    double *vf = qf + MG_TG;           // [VR]
    int *ve = (int *)(vf + VR);        // [VR]
    int *vj = ve + VR;                 // [VR]
    double *yAs = vf + 2 * VR;         // [Delta]      absolute scale of the forward row lo + i
    double *yBs = yAs + Delta;         // [Delta + K]  absolute scale of the backward row lo + 1 + i
    const size_t row0 = (size_t)b * (p.T + 1);
    const double2 *EI = p.EI + row0 * C + c0;
    const int *nb = p.nbase + row0 * C + c0;
    const double2 *frow = (const double2 *)p.aloc + ((size_t)b * N) * Delta * C + c0;  // row of position t at t*C
    const double2 *brow = (const double2 *)p.bloc + ((size_t)b * N) * Delta * C + c0;  // (slots are consecutive)
    const double logZ = h.logZ;
    double acc[MG_KS];
#pragma unroll
    for (int kk = 0; kk < MG_KS; ++kk) acc[kk] = 0.0;
    for (int i = tid; i < hi - lo; i += nth) yAs[i] = mg_ya(p, b, iv, i);
    for (int i = kS + tid; i < min(hi - lo + K, hi - lo + kS + VR); i += nth) {
        const int s = lo + 1 + i;
        yBs[i] = s < L ? mg_yb(p, b, s / Delta, s % Delta, L) : 0.0;  // b_L = 1: scale 0
    }

    for (int tg0 = lo; tg0 < hi;) {
        const int tg1 = min(min(hi, (tg0 / J + 1) * J), tg0 + MG_TG);
        const int ng = tg1 - tg0, jt = tg0 / J;
        __syncthreads();  // the previous group is done with the staged rows (first: the scales are there)
        const double yA0 = yAs[tg0 - lo];
        // per row first (uniform over the labels): the scale factor of a q row; for a v row the
        // fractional factor, the integer exponent and the scaling block it was stored in
        for (int r = tid; r < MG_TG + VR; r += nth) {
            if (r < MG_TG) {
                qf[r] = r < ng ? exp2(yAs[tg0 + r - lo] - yA0) : 0.0;
            } else {
                const int rr = r - MG_TG, s = tg0 + 1 + kS + rr;
                double f = 0.0;
                int e = 0, js = jt;
                if (s <= L && kS + rr < ng + K) {
                    const double lf = (yA0 + yBs[s - lo - 1]) - logZ * LOG2E;
                    const double fl = floor(lf);
                    f = exp2(lf - fl);
                    e = whole_exponent(fl);
                    js = s / J;
                }
                vf[rr] = f;
                ve[rr] = e;
                vj[rr] = js;
            }
        }
        __syncthreads();
        // v_L = ES_L; all exponents are combined before anything is formed, so that an empty row stays
        // zero and nothing passes through infinity.  Thread (row offset, label): no index divisions in
        // the loops; the loads of several rows per thread are issued together (rows beyond the
        // sequence are clamped, their factor is zero).
        {
            const int rstep = nth / CL;              // rows per sweep of the workgroup
            const int o = tid % CL, r0 = tid / CL;     // threads with r0 >= rstep idle here
            if (r0 < rstep) {
                {
                    constexpr int UQ = 4;  // the q rows of a thread are fetched together
                    for (int rb = r0; rb < MG_TG; rb += UQ * rstep) {
                        double qv[UQ];
#pragma unroll
                        for (int u = 0; u < UQ; ++u)
                            qv[u] = frow[(size_t)(tg0 + min(rb + u * rstep, ng - 1)) * C + o].y;
#pragma unroll
                        for (int u = 0; u < UQ; ++u) {
                            const int r = rb + u * rstep;
                            if (r < MG_TG) Qrow[r * CL + o] = qv[u] * qf[r];  // qf is zero beyond the group
                        }
                    }
                }
                const int nbt = nb[(size_t)jt * C + o];
                constexpr int UV = 4;
                for (int rb = r0; rb < VR; rb += UV * rstep) {
                    double vs[UV];
                    int n1[UV];
#pragma unroll
                    for (int u = 0; u < UV; ++u) {
                        const int r = min(rb + u * rstep, VR - 1);
                        const int s = min(tg0 + 1 + kS + r, L);
                        vs[u] = s == L ? EI[(size_t)L * C + o].x : brow[(size_t)s * C + o].y;
                        n1[u] = nb[(size_t)vj[r] * C + o];
                    }
#pragma unroll
                    for (int u = 0; u < UV; ++u) {
                        const int r = rb + u * rstep;
                        if (r < VR) {
                            const double f = vf[r];
                            Vp[r * CP + o] = f != 0.0 ? fmin(ldexp(vs[u] * f, n1[u] - nbt + ve[r]), DBL_MAX) : 0.0;
                        }
                    }
                }
            }
        }
        __syncthreads();
        if (active) {
            for (int i0 = 0; i0 < ng; i0 += 4) {
                double ca[4];
#pragma unroll
                for (int i = 0; i < 4; ++i) ca[i] = i0 + i < ng ? Qrow[(i0 + i) * CL + c] : 0.0;
                double w[MG_KS + 3];
#pragma unroll
                for (int q = 0; q < MG_KS + 3; ++q) w[q] = Vp[(i0 + kA + q) * CP + c];
#pragma unroll
                for (int kk = 0; kk < MG_KS; ++kk) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) acc[kk] = fma(ca[i], w[kk + i], acc[kk]);
                }
            }
        }
        tg0 = tg1;
    }
    if (active) {
        double *pD = p.partD + ((size_t)b * p.NP + iv) * K * C;
#pragma unroll
        for (int kk = 0; kk < MG_KS; ++kk) {
            const int k = kS + kA + kk + 1;
            if (k <= K) pD[(size_t)(k - 1) * C + c0 + c] = acc[kk] * p.W[(size_t)(k - 1) * C + c0 + c];
        }
    }
}

// One workgroup per (sequence, interval).
__global__ __launch_bounds__(1024) void k_mg_dur(Params p)
{
    extern __shared__ double lds_raw[];
    const int b = blockIdx.x / p.N, iv = blockIdx.x % p.N;
    if (iv * p.Delta >= p.hdr[b].L) return;
    if (!(p.spec_ok[b * 2] && p.spec_ok[b * 2 + 1])) return;  // the interval kernel takes this sequence
    mg_dur_vector(p, lds_raw, b, iv, 0, p.C, 0, (p.K + MG_KS - 1) / MG_KS);
}

// Duration-bias statistics on the matrix cores.  For one label,
//   D[k] = sum_t q_t v_{t+k}      (each v brought into the frame of its t)
// is a correlation.  With positions in groups of sixteen, t = 16 g + s, let
//   P[s][x] = sum_g q_{16g+s} v_{16g+1+x},   so that   D[k' + 1] = sum_s P[s][s + k'].
// P is a product with the groups as the inner dimension: v_mfma_f64_16x16x4 takes four groups (64 positions) of the
// sixteen s against sixteen x, and K + 16 columns x replace K durations.  What is a frame's business happens on the way into
// the instruction: a row v lies in LDS once, in a frame of its group w of sixteen rows (16 w + 1 .. 16 w + 16), and is brought
// into the frame of group g by one power of two, 2^(E[w] - F[g]), per label and pair of groups, with all exponents
// combined in whole numbers before anything is formed.  (A group lies in one scaling block, J >= 16; its row v may be the first of
// the next block, brought down by the step the scan itself makes there.)
// Wave (label of LW, range of kb * 16 durations, kb <= KB = 8): kb + 1 tiles of P in its accumulators for the whole interval, one
// workgroup of eight waves per (interval, group of labels, part of the durations), two of them on a compute unit.  Rows go
// through LDS in a ring of RG groups, fetched a step of 64 positions ahead.  A product and the conversion of its operand element
// take 84 clocks of a SIMD (64 the product alone; a power of two by integer adds or by a multiplication is no cheaper), which
// makes 65 us of the 139 at K = 512, C = 8, T = 400 000 (vector form: 220); the rest is a workgroup's tables and first
// rows, the steps' barriers, and the sums over s at the end.  KB = 16, one workgroup per compute unit: 151.
// Sequences with J < 16 take the vector form: a share is a group of labels with all durations, or with one of vparts ranges of them
// where a workgroup's LDS or threads do not hold that, and a sequence's first workgroups take its shares one after the other, all
// sequences side by side: every parts-th workgroup alone would meet in a quarter of the compute units.  Calls with scores N(0, 20^2), in
// shares of the parts' own durations, which each fetch scales and positions again / by every parts-th workgroup / so: K = 512, C = 8,
// 50 000 positions 1900 / 2430 / 1790 us, eight such sequences 8440 / 7000 / 4715; K = 256, C = 16, two 1566 / 1890 / 1285.
constexpr int MGD_NT = 512;
constexpr int MGD_J = 16;  // shortest scaling block of this form: a tile's positions
constexpr int MGD_KB = 8;
constexpr int mgd_fill(int LW) { return ((8 / LW) * MGD_KB + 4 + 3) / 4 * 4; }  // groups of rows a step of 64 positions reads, whole steps
constexpr int mgd_ring(int LW) { return mgd_fill(LW) + 4 <= 16 ? 16 : 32; }
static_assert(mgd_fill(8) + 4 <= mgd_ring(8) && mgd_fill(4) + 4 <= mgd_ring(4), "a step's rows next to those of the one before");
constexpr int MGD_QS = 72;                                                            // doubles of a label's positions of a step
constexpr int mgd_steps(int Delta) { return (Delta + 15 + 15) / 64 + 1; }             // most steps of an interval
constexpr size_t mgd_lds(int LW, int K, int Delta)
{
    return ((size_t)LW * mgd_ring(LW) * 16 + 2 * LW * MGD_QS + Delta + K + 2 * ((size_t)K / Delta + 4)) * sizeof(double) +
           ((size_t)LW * (4 * mgd_steps(Delta) + mgd_fill(LW)) + (size_t)LW * 4 * mgd_steps(Delta) + Delta + K +
            (size_t)LW * ((Delta + K) / MGD_J + 2)) * sizeof(int);
}

template <int LW>
__global__ __launch_bounds__(MGD_NT, 4) void k_mg_dur_mx(Params p, int nlg, int parts, int kb, int vparts)
{
    typedef double double4_t __attribute__((ext_vector_type(4)));
    constexpr int KB = MGD_KB, RANGES = 8 / LW, RG = mgd_ring(LW), FILL = mgd_fill(LW), NST = FILL / 4, ROWS = 64;
    extern __shared__ double lds_raw[];
    const int tid = threadIdx.x;
    const int K = p.K, C = p.C, N = p.N, Delta = p.Delta;
    const int b = blockIdx.x, x = blockIdx.y;
    const SeqHdr h = p.hdr[b];
    const int L = h.L, J = h.J;
    if (!(p.spec_ok[b * 2] && p.spec_ok[b * 2 + 1])) return;  // the interval kernel takes this sequence
    if (J < MGD_J) {
        const int vpart = x % vparts, l0 = x / vparts % nlg * LW, viv = x / (vparts * nlg), strips = (K + MG_KS - 1) / MG_KS;
        if (viv < N && viv * Delta < L)
            mg_dur_vector(p, lds_raw, b, viv, l0, min(LW, C - l0), strips * vpart / vparts, strips * (vpart + 1) / vparts);
        return;
    }
    const int part = x % parts, lg = x / parts % nlg, iv = x / (parts * nlg);
    const int lo = iv * Delta;
    if (lo >= L) return;
    const int hi = min(lo + Delta, L), smax = min(hi - 1 + K, L);  // rows v_s, lo < s <= smax
    const int ljb = __builtin_ctz(J), blk0 = lo >> ljb, nblk = (smax >> ljb) - blk0 + 1;
    const int g0 = lo >> 4, w0 = g0 + part * RANGES * kb;  // first group of positions, of rows
    const int steps = (((hi + 15) >> 4) - g0 + 3) / 4, NG = 4 * (steps - 1) + FILL;
    double *const V = lds_raw;                     // [LW][RG * 16]  rows, by group modulo RG
    double *const Q = V + LW * RG * 16;            // [2][LW][MGD_QS] q of the step's positions
    double *const rowF = Q + 2 * LW * MGD_QS;      // [Delta + K]    per row lo + 1 + i: factor in [1, 2) ...
    double *const tabF = rowF + Delta + K;         // per interval the rows reach into, and one for row L: the same at its upper end
    int *const tabE = (int *)(tabF + K / Delta + 4);
    int *const rowE = (int *)(tabF + 2 * (K / Delta + 4));  // [Delta + K] ... and exponent of its scale
    int *const Es = rowE + Delta + K;              // [NG][LW]       exponent of a group of rows w0 + i
    int *const Fs = Es + LW * NG;                  // [4 steps][LW]  exponent of a group of positions g0 + i
    int *const nbl = Fs + LW * 4 * steps;          // [nblk][LW]     block exponents
    const size_t row0 = (size_t)b * (p.T + 1);
    const int *nb = p.nbase + row0 * C;
    const char *const frow = (const char *)((const double2 *)p.aloc + ((size_t)b * N + iv) * Delta * C);  // row of position lo + i at i*C
    const char *const brow = (const char *)((const double2 *)p.bloc + ((size_t)b * N + iv) * Delta * C);  // (slots are consecutive)
    const double *frowY = p.alocY + ((size_t)b * N + iv) * Delta, *browY = p.blocY + ((size_t)b * N + iv) * Delta;

    // ---- staging: thread (row of 64, label of LW)
    const int sl = tid % LW, sr = tid / LW;
    const int sc = min(lg * LW + sl, C - 1);
    const double vL = p.EI[(row0 + L) * C + sc].x;  // v_L = ES_L, scale 0
    const int slast = min(smax, L - 1) - lo;         // last stored row (relative to the interval, as all that follow)
    auto row_of = [&](const int q) { return 16 * (w0 + 4 * q) + 1 + sr - lo; };
    // (every thread, whatever it does with them: loads under a condition are waited for where the condition ends)
    auto fetch = [&](const int q) {  // four groups of rows
        const unsigned s = (unsigned)max(min(row_of(q), slast), 0);
        return *(const double *)(brow + (s * (unsigned)C + (unsigned)sc) * 16u + 8u);
    };
    auto place = [&](const int q, const double v) {
        if (sr >= ROWS) return;
        const int s = row_of(q), i = max(min(s, smax - lo), 1), g = 4 * q + (sr >> 4);
        const int e = rowE[i - 1] + nbl[(((i + lo) >> ljb) - blk0) * LW + sl] - Es[g * LW + sl];
        const double x = fmin(ldexp((i + lo == L ? vL : v) * rowF[i - 1], e), DBL_MAX);
        V[(sl * RG + (g & (RG - 1))) * 16 + (sr & 15)] = s == i ? x : 0.0;  // (rows before lo + 1 and after smax: none)
    };
    auto fetch_q = [&](const int k) {
        const unsigned t = (unsigned)max(min(16 * (g0 + 4 * k) + sr, hi - 1) - lo, 0);
        return *(const double *)(frow + (t * (unsigned)C + (unsigned)sc) * 16u + 8u);
    };
    auto place_q = [&](const int k, const double q) {
        const int t = 16 * (g0 + 4 * k) + sr;
        if (sr < ROWS) Q[((k & 1) * LW + sl) * MGD_QS + sr] = t >= lo && t < hi ? q : 0.0;
    };
    double first[NST];
#pragma unroll
    for (int q = 0; q < NST; ++q) first[q] = fetch(q);
    const double fq = fetch_q(0);

    // What 2^(Y_alpha(lo) + Y_beta(s)) / Z takes apart into: stored scales are whole numbers relative to their interval's upper
    // end.  All that the tables are made of is requested before the first of it is waited for.
    constexpr int RB = 3;  // rows per thread and sweep
    double rowY[RB];
    auto fetch_scales = [&](const int i0) {
#pragma unroll
        for (int u = 0; u < RB; ++u) rowY[u] = browY[min(i0 + u * MGD_NT + tid + 1, slast)];
    };
    fetch_scales(0);
    auto block_exponent = [&](const int i) { return nb[(size_t)(blk0 + min(i / LW, nblk - 1)) * C + min(lg * LW + i % LW, C - 1)]; };
    const int nb_first = block_exponent(tid);
    auto first_position = [&](const int i) { return max(16 * (g0 + i / LW), lo); };  // of a group of positions
    const double fy_first = frowY[min(first_position(tid), hi - 1) - lo];
    const int nj = slast / Delta + 1;
    for (int i = tid; i <= nj; i += MGD_NT) {
        const double top = i == nj || iv + i == (L - 1) / Delta ? 0.0 : p.ckYB[(size_t)b * (N + 1) + iv + i + 1];
        const double lf = (p.ckYA[(size_t)b * (N + 1) + iv] + top) - h.logZ * LOG2E, fl = floor(lf);
        tabF[i] = exp2(lf - fl);
        tabE[i] = whole_exponent(fl);
    }
    for (int i = tid; i < nblk * LW; i += MGD_NT) nbl[i] = i == tid ? nb_first : block_exponent(i);
    __syncthreads();
    for (int i0 = 0; i0 < smax - lo; i0 += RB * MGD_NT) {
        if (i0 > 0) fetch_scales(i0);
#pragma unroll
        for (int u = 0; u < RB; ++u) {
            const int i = i0 + u * MGD_NT + tid, s = i + 1;  // row lo + s
            if (i < smax - lo) {
                const bool last = lo + s == L;
                const int jj = last ? nj : (int)((unsigned)s / (unsigned)Delta);
                rowF[i] = tabF[jj];
                rowE[i] = tabE[jj] + (last ? 0 : (int)rowY[u]);
            }
        }
    }
    for (int i = tid; i < LW * 4 * steps; i += MGD_NT) {
        const int t = first_position(i);
        if (t < hi) Fs[i] = nbl[((t >> ljb) - blk0) * LW + i % LW] - (int)(i == tid ? fy_first : frowY[t - lo]);
        else Fs[i] = 0;
    }
    __syncthreads();
    for (int i = tid; i < LW * NG; i += MGD_NT) {  // the frame of a group of rows: that of its first
        const int f = max(16 * (w0 + i / LW) + 1, lo + 1);
        Es[i] = f <= smax ? rowE[f - lo - 1] + nbl[((f >> ljb) - blk0) * LW + i % LW] : 0;
    }
    __syncthreads();
#pragma unroll
    for (int q = 0; q < NST; ++q) place(q, first[q]);
    place_q(0, fq);
    __syncthreads();

    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, m = lane >> 4, n = lane & 15;
    const int wl = wave % LW, wr = wave / LW, c = lg * LW + wl, kb0 = (part * RANGES + wr) * kb;
    const bool mine = c < C && kb0 * 16 < K;
    double4_t P[KB + 1];
#pragma unroll
    for (int j = 0; j <= KB; ++j) P[j] = double4_t{0.0, 0.0, 0.0, 0.0};
    const char *const vbase = (const char *)(V + wl * RG * 16 + n);
    const int *const ebase = Es + (m + wr * kb) * LW + wl, *const fbase = Fs + m * LW + wl;
    for (int k = 0; k < steps; ++k) {
        const double nv = fetch(k + NST), nq = fetch_q(k + 1);
        const bool more = k + 1 < steps;
        if (mine) {
            const double a = Q[((k & 1) * LW + wl) * MGD_QS + lane];
            const int F = fbase[4 * k * LW], rel = 4 * k + m + wr * kb;
            // all operand elements are requested first; each is converted while the product before it runs
            double raw[KB + 1];
            int e[KB + 1];
#pragma unroll
            for (int j = 0; j <= KB; ++j) {
                raw[j] = *(const double *)(vbase + ((rel * 128 + j * 128) & (RG * 128 - 1)));
                e[j] = ebase[(4 * k + j) * LW];
            }
            __builtin_amdgcn_sched_barrier(0);
            double x = fmin(ldexp(raw[0], e[0] - F), DBL_MAX);
#pragma unroll
            for (int j = 0; j <= KB; ++j) {
                const double xn = j < KB ? fmin(ldexp(raw[j + 1], e[j + 1] - F), DBL_MAX) : 0.0;
                __builtin_amdgcn_sched_barrier(0);
                if (j <= kb) P[j] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, x, P[j], 0, 0, 0);
                x = xn;
            }
        }
        if (more) {
            place(k + NST, nv);
            place_q(k + 1, nq);
            __syncthreads();
        }
    }
    if (!mine) return;
    // ---- D[k' + 1] = sum_s P[s][s + k']: tile element (s = 4 v + m, n) belongs to k' = 16 j + n - s
    double *pD = p.partD + ((size_t)b * p.NP + iv) * K * C;
    double w[KB];
#pragma unroll
    for (int j = 0; j < KB; ++j) w[j] = p.W[(size_t)min((kb0 + j) * 16 + n, K - 1) * C + c];
#pragma unroll
    for (int j = 0; j < KB; ++j) {
        double sum = 0.0;
#pragma unroll
        for (int v = 0; v < 4; ++v) {
            const int s = 4 * v + m;
            sum += __shfl(n >= s ? P[j][v] : P[j + 1][v], (lane & 48) | ((n + s) & 15));
        }
        sum = add_across_32(add_across_16(sum));
        const int kk = (kb0 + j) * 16 + n;
        if (m == 0 && j < kb && kk < K) pD[(size_t)kk * C + c] = sum * w[j];
    }
}

// Transition statistics and the running emission sums (K >= 128, so C <= 32).  A workgroup of W waves (eight; four with more than 16
// labels, whose rows take more registers) takes an interval from its upper end downwards (the emission sums are suffix sums), W * S
// positions at a time, S of them to a wave.  A wave takes
// 64 / LB positions by LB labels at once (LB = 8 up to eight labels, else 16, twice with more than 16), the rows of the next ones
// requested a step ahead; every lane forms a_t kappa, p_t and (out - in) kappa of its position and label, which are
// the operands of the transition product as they stand (v_mfma_f64_16x16x4, inner index the position; with eight
// labels the instruction's lower and upper eight rows and columns are two sets of positions, of whose products only
// the two blocks on the diagonal are wanted), and the running sums within the wave by three or two steps between lanes.
// They go through LDS, where the waves above add theirs, and out in rows.  Bound by memory: 48 bytes read and 4 written per
// position and label.  K = 512, C = 8, T = 400 000:
// 33 us (4.9 TB/s), against 69 with the rows staged in LDS for a thread per pair of labels and one per label for the sums.
constexpr int mgt_seg(int C) { return C <= 8 ? 64 : (C <= 16 ? 32 : 16); }  // S
constexpr size_t mgt_lds(int W, int C) { return ((size_t)W * mgt_seg(C) * C + (2 * W + 2) * (size_t)C + (size_t)C * C) * sizeof(double); }
static_assert(mgt_lds(8, 8) <= 65536 && mgt_lds(8, 16) <= 65536 && mgt_lds(4, 32) <= 65536, "what a kernel may have without asking");

template <int LB, int TL, int W>
__global__ __launch_bounds__(64 * W, TL == 2 ? 3 : 4) void k_mg_te(Params p)
{
    typedef double double4_t __attribute__((ext_vector_type(4)));
    constexpr int PP = 64 / LB;  // positions of a step
    extern __shared__ double lds_raw[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int C = p.C, CC = C * C, N = p.N, Delta = p.Delta;
    const int b = blockIdx.x / N, iv = blockIdx.x % N;
    const SeqHdr h = p.hdr[b];
    const int L = h.L;
    const int lo = iv * Delta;
    if (lo >= L) return;
    if (!(p.spec_ok[b * 2] && p.spec_ok[b * 2 + 1])) return;
    const int hi = min(lo + Delta, L);
    const int S = mgt_seg(C), CH = W * S;
    double *const Rl = lds_raw;              // [CH][C]  running sums of a chunk, each wave's from its own upper end
    double *const seg = Rl + (size_t)CH * C;  // [W][C]   what a wave's positions add up to
    double *const ssum = seg + W * C;    // [W][C]   sum of its running sums
    double *const top = ssum + W * C;    // [C]      what the chunks above add up to
    double *const tsum = top + C;            // [C]      sum of the running sums so far
    double *const trs = tsum + C;            // [C][C]
    const size_t row0 = (size_t)b * (p.T + 1), slot = (size_t)b * N + iv;
    const double2 *EI = p.EI + (row0 + lo) * C;
    const double2 *frow = (const double2 *)p.aloc + slot * Delta * C, *brow = (const double2 *)p.bloc + slot * Delta * C;
    const double *frowY = p.alocY + slot * Delta, *browY = p.blocY + slot * Delta;
    // kappa(t,t) = exp((Y_alpha + Y_beta) ln2 - logZ): the stored scales are whole numbers relative to the interval's ends
    const double kx = (p.ckYA[(size_t)b * (N + 1) + iv] + (hi == L ? 0.0 : p.ckYB[(size_t)b * (N + 1) + iv + 1])) - h.logZ * LOG2E;
    const double kxi = floor(kx), kfrac = exp2(kx - kxi);
    const int kint = whole_exponent(kxi);
    const int pi = lane / LB, pl = lane % LB;  // position (from the upper end) and label of the lane
    int cc[TL];
#pragma unroll
    for (int u = 0; u < TL; ++u) cc[u] = min(u * LB + pl, C - 1);
    double4_t acc[TL][TL];
#pragma unroll
    for (int u = 0; u < TL; ++u)
#pragma unroll
        for (int x = 0; x < TL; ++x) acc[u][x] = double4_t{0.0, 0.0, 0.0, 0.0};
    if (tid < 2 * C) top[tid] = 0.0;  // and tsum
    struct Rows {
        double2 a[TL], v[TL], e[TL];
        double ya, yb;
    };
    auto fetch = [&](const int t) {  // relative to lo; every lane, whatever is asked for
        Rows r;
        const int i = max(t, 0);
#pragma unroll
        for (int u = 0; u < TL; ++u) {
            const unsigned o = (unsigned)i * (unsigned)C + (unsigned)cc[u];
            r.a[u] = frow[o];
            r.v[u] = brow[o];
            r.e[u] = EI[o];
        }
        r.ya = frowY[i];
        r.yb = browY[i];
        return r;
    };
    Rows r = fetch(hi - lo - wave * S - 1 - pi);
    for (int tg1 = hi - lo; tg1 > 0; tg1 -= CH) {
        const int s1 = tg1 - wave * S, n = min(s1, S);  // the wave's positions: s1 - 1 downwards, n of them (none if not positive)
        double R[TL], sR[TL];
#pragma unroll
        for (int u = 0; u < TL; ++u) R[u] = sR[u] = 0.0;
        for (int i0 = 0; i0 < n; i0 += PP) {
            const Rows rn = fetch((i0 + PP < n ? s1 - (i0 + PP) : s1 - CH) - 1 - pi);  // (after the last step: the next chunk's first)
            const int i = i0 + pi, t = s1 - 1 - i;
            const bool on = i < n;
            const double kap = on ? ldexp(kfrac, kint + (int)(r.ya + r.yb)) : 0.0;
            double ak[TL];
#pragma unroll
            for (int u = 0; u < TL; ++u) {
                ak[u] = r.a[u].x * kap;
                // a segment of the label starts at t (z_t p_t, z = q ES) / ends at t (a_t b_t, b = v IE; none ends at 0)
                const double d = r.a[u].y * kap * r.e[u].x * r.v[u].x - (t + lo >= 1 ? ak[u] * r.v[u].y * r.e[u].y : 0.0);
                double inc = on ? d : 0.0;
#pragma unroll
                for (int off = LB; off < 64; off <<= 1) {
                    const double x = __shfl_up(inc, off);
                    inc += lane >= off ? x : 0.0;
                }
                const double run = R[u] + (inc - (on ? d : 0.0));
                if (on && u * LB + pl < C) Rl[(size_t)(wave * S + i) * C + u * LB + pl] = run;
                sR[u] += on ? run : 0.0;
                R[u] += __shfl(inc, 64 - LB + pl);
            }
#pragma unroll
            for (int u = 0; u < TL; ++u)
#pragma unroll
                for (int x = 0; x < TL; ++x)
                    acc[u][x] = __builtin_amdgcn_mfma_f64_16x16x4f64(ak[u], r.v[x].x, acc[u][x], 0, 0, 0);
            r = rn;
        }
#pragma unroll
        for (int u = 0; u < TL; ++u) {
#pragma unroll
            for (int off = LB; off < 64; off <<= 1) sR[u] += __shfl_xor(sR[u], off);
            if (lane < LB && u * LB + pl < C) {
                seg[wave * C + u * LB + pl] = R[u];
                ssum[wave * C + u * LB + pl] = sR[u];
            }
        }
        __syncthreads();
        const int m = min(tg1, CH);  // positions of the chunk
        if (tid < C) {
            double above = top[tid], sum = tsum[tid];
            for (int w = 0; w < W; ++w) {
                const double own = seg[w * C + tid];
                sum += ssum[w * C + tid] + above * (double)max(min(m - w * S, S), 0);
                seg[w * C + tid] = above;
                above += own;
            }
            top[tid] = above;
            tsum[tid] = sum;
        }
        __syncthreads();
        // rows in ascending order of addresses: row x of the chunk is position tg1 - 1 - x
        float *const out = p.grad_emis + ((size_t)b * p.T + lo + tg1 - m) * C;
        for (int i = tid; i < m * C; i += 64 * W) {
            const int x = m - 1 - i / C, c = i % C;
            out[i] = (float)(Rl[(size_t)x * C + c] + seg[x / S * C + c]);
        }
        __syncthreads();
    }
    for (int i = tid; i < CC; i += 64 * W) trs[i] = 0.0;
    for (int w = 0; w < W; ++w) {  // the waves' products, one after the other
        __syncthreads();
        if (wave == w) {
#pragma unroll
            for (int hf = 0; hf < (LB == 8 ? 2 : 1); ++hf) {
#pragma unroll
                for (int u = 0; u < TL; ++u)
#pragma unroll
                    for (int x = 0; x < TL; ++x)
#pragma unroll
                        for (int v = 0; v < 4; ++v) {  // tile element (4 v + lane / 16, lane % 16)
                            const int src = u * 16 + 4 * v + (lane >> 4) - 8 * hf, dst = x * 16 + (lane & 15) - 8 * hf;
                            const bool in = LB == 16 || (src >= 0 && dst >= 0 && src < 8 && dst < 8);
                            if (in && src < C && dst < C) trs[src * C + dst] += acc[u][x][v];
                        }
                lds_wave_fence();
            }
        }
    }
    __syncthreads();
    double *pT = p.partTr + slot * CC;
    for (int i = tid; i < CC; i += 64 * W) pT[i] = trs[i];
    if (tid < C) {
        p.tot[slot * C + tid] = top[tid];
        p.sumR[slot * C + tid] = tsum[tid];
    }
}

// ---------------------------------------------------------------------------
// The same statistics for short maximal durations (K < 128), where the work of an interval fits single waves.
// One wave per (sequence, interval, part): an interval is cut into p.msplit parts of equal length, each its own
// task, so that the chip holds two tasks per SIMD where there are few intervals; nothing in these statistics
// depends on the position before, only the running emission sums do, and those restart with every part (the
// partial sums tot, sumR, partD, partTr are per part: index interval*msplit + part).  Lane organisation of the
// interval kernel (lane (g, c): label c, durations g*NK + 1 ..): the wave walks its part from the upper end
// downwards, as the backward scan did, but takes p_t and v_t from that scan's stored rows instead of running the
// recurrence.  The K-deep window of v rows slides through LDS in the frame of the current scaling block (rescaled
// by the same powers of two at the same positions as in the scan, read off the stored scales), so the duration
// statistics are NK multiply-adds per position and lane with every window entry read once per block of MB
// positions; the transition statistics run on the matrix cores, four positions per v_mfma_f64_16x16x4; the
// emission sums are running sums.  The rows of the next block are requested as soon as the current block's have
// been turned into the few values the multiply-adds need.
// BT: calls with boundary terms.  The pair of a position is then no longer (E, 1/E), so the masses of the segments that
// start and end there are formed with the reciprocals of its two factors, and go out as the gradients of the boundary
// projections and, summed over the labels, as the boundary posterior.  (Genomic shape with all of them: 196 us, 665 us
// for the call; with the interval kernel's own recurrence the call takes 1025 us.)
template <int CT, int NKW, bool BT>
__global__ __launch_bounds__(64, mg_waves_per_simd(CT, NKW)) void k_mg_wave(Params p)
{
    using G = WaveWin<CT, NKW>;
    constexpr int CTP = G::CTP, RS = G::RS, NK = G::NK, KW = G::KW, M = G::M, RTOT = G::RTOT, TRN = G::TRN;
    typedef double double4_t __attribute__((ext_vector_type(4)));
    extern __shared__ double lds_raw[];
    double *ring = lds_raw;  // [ROWS][RS] (+ pad), then 64 doubles nobody reads
    const int lane = threadIdx.x;
    const int K = p.K, C = p.C, KC = K * C, CC = C * C, N = p.N, Delta = p.Delta;
    const int S = p.msplit, Dm = Delta / S;
    const int sub = blockIdx.x % S, b = (blockIdx.x / S) / N, iv = (blockIdx.x / S) % N;
    const SeqHdr h = p.hdr[b];
    const int L = h.L, J = h.J, Jm = J - 1;
    const int t0 = iv * Delta;      // the interval: its rows are stored relative to t0
    const int ta = t0 + sub * Dm;   // this task's positions: ta <= t < tb
    if (ta >= L) return;
    if (!(p.spec_ok[b * 2] && p.spec_ok[b * 2 + 1])) return;  // the interval kernel takes this sequence
    const int t1 = min(t0 + Delta, L);
    const int tb = min(ta + Dm, L);
    const int c = lane % CTP, g = lane / CTP;
    const bool cval = c < C;
    const int cc = cval ? c : 0;
    const bool writer = cval && g == 0;  // one lane per label
    const int pj = lane >> 4, pl = lane & 15;  // matrix-core operands: position pj of the block, label pl of the tile
    const size_t row0 = (size_t)b * (p.T + 1);
    const double2 *EIc = p.EI + row0 * C + cc;
    const int *nbc = p.nbase + row0 * C + cc;
    const size_t slot = (size_t)b * N + iv;
    const size_t part = (size_t)b * p.NP + (size_t)iv * S + sub;
    const double2 *arow = (const double2 *)p.aloc + slot * Delta * C;  // (a_t, q_t) of position t0 + i at i*C
    const double2 *brow = (const double2 *)p.bloc + slot * Delta * C;  // (p_t, v_t)
    const double *arowY = p.alocY + slot * Delta;
    const double *browY = p.blocY + slot * Delta;
    const double logZ = h.logZ;
    const double Y0 = p.ckYA[(size_t)b * (N + 1) + iv];
    const double Ytop = t1 == L ? 0.0 : p.ckYB[(size_t)b * (N + 1) + iv + 1];

    // ---- the window above the part
    for (int i = lane; i < RTOT; i += 64) ring[i] = 0.0;
    lds_wave_fence();
    int r = M;  // row of the newest (lowest) position
    double ybPrev = 0.0;  // stored scale (relative to the interval's upper end) of the frame the window is in
    if (tb == L) {  // v_L = E_L
        if (writer) ring[r * RS + c] = EIc[(size_t)L * C].x;
    } else if (tb == t1) {  // the state the backward task started from
        const double *ck;
        const double fi = state_above(p, b, ((size_t)b * (N + 1) + iv + 1) * ((size_t)KC + C), ck);
        const int tm = t1 % K;
        if (cval) {  // lane (g, c): the window rows at distances g, g + GW, ... of its label (no index divisions)
#pragma unroll 8
            for (int d = g; d < K; d += G::GW) {
                int sl = tm + d;  // checkpoint slot of the position at that distance
                sl -= sl >= K ? K : 0;
                ring[(r + d) * RS + c] = fi * ck[(size_t)sl * C + c];
            }
        }
    } else {
        // inside the interval: the rows v_tb .. v_{tb+K-1} as the backward task stored them (a part is at least
        // K positions long, so they all belong to this interval, or are v_L), each brought from the frame of its own
        // scaling block into that of position tb: the powers of two the scan applied on its way down from there
        // and the difference of the stored scales (whole numbers).  Lane (g, c) fills its own strip, rows g*NK ..
        // of label c; everything is loaded first, so that the loads of all rows are in flight together.
        const int nbt = nbc[(size_t)(tb / J) * C];
        const double ybt = browY[tb - t0];
        const int top = min(t1 - 1, L - 1) - t0;  // last stored row of the interval
        double vr[NK], ys[NK];
        int ns[NK];
#pragma unroll
        for (int u = 0; u < NK; ++u) {
            const int i = min(tb - t0 + g * NK + u, top);  // v_L and what lies beyond are dealt with below
            vr[u] = brow[(size_t)i * C + cc].y;
            ys[u] = browY[i];
            ns[u] = nbc[(size_t)((t0 + i) / J) * C];
        }
        const double vL = EIc[(size_t)L * C].x;  // scale 0 relative to the upper end
        const int nsL = nbc[(size_t)(L / J) * C];
#pragma unroll
        for (int u = 0; u < NK; ++u) {
            const int d = g * NK + u, sp = tb + d;
            const int e = whole_exponent((sp == L ? 0.0 : ys[u]) - ybt) + (sp == L ? nsL : ns[u]) - nbt;
            const double val = fmin(ldexp(sp == L ? vL : vr[u], e), DBL_MAX);
            if (cval && d < K && sp <= L) ring[(r + d) * RS + c] = val;
        }
        ybPrev = browY[tb - t0];
    }
    lds_wave_fence();

    double dx[NK + MB - 1];  // sum_t q_t(c) kappa_t v_{t+k}(c), k = g*NK + jj + 1 (times W[k,c] at the end)
    double dn[MB - 1];       // the same for k = 1..MB-1 from inside the blocks (lanes g == 0)
    double4_t accT[TRN][TRN];
#pragma unroll
    for (int jj = 0; jj < NK + MB - 1; ++jj) dx[jj] = 0.0;
#pragma unroll
    for (int jj = 0; jj < MB - 1; ++jj) dn[jj] = 0.0;
#pragma unroll
    for (int i = 0; i < TRN; ++i)
#pragma unroll
        for (int o = 0; o < TRN; ++o) accT[i][o] = double4_t{0.0, 0.0, 0.0, 0.0};
    double R = 0.0, sR = 0.0;
    float *const sink = (float *)p.sink + lane;
    float *const gout = p.grad_emis + ((size_t)b * p.T) * C + cc;

    // The rows of one block of positions, as they come from memory.  Where a label's lanes come in pairs 32 apart
    // (CTP <= 32) the lower half of the wave fetches the block's first two positions and the upper half the
    // other two: half the row loads, which is what this kernel waits for most (the few values the other half
    // needs travel by v_permlane32_swap).  With 64 labels per lane group every lane fetches all four.
    static_assert(MB == 4, "the split of a block between the halves of the wave is written for four positions");
    constexpr bool SPLIT = CTP <= 32;
    constexpr int NPL = SPLIT ? MB / 2 : MB;  // positions of a block this lane fetches
    const int pofs = SPLIT ? (lane >> 5) * NPL : 0;  // the first of them
    double2 aq[NPL], pv[NPL], e[NPL];  // this lane's label, positions pofs .. pofs+NPL-1 below tfrom
    double aA[TRN], bB[TRN];        // operand elements: position pj of the block, label pl of tile tr
    double ya, yb;                  // stored scales of the position just below tfrom (forward, backward)
    int nhi, nlo;                   // exponents of this lane's label on both sides of the scaling-block boundary tfrom
    // Byte offsets from the (wave-uniform) starts of the interval's rows fit 32 bits: a slot has Delta*C < 2^27
    // pairs (the plan's limits), a sequence fewer than 2^31 position-label pairs (checked by the caller).
    const char *const arb = (const char *)arow, *const brb = (const char *)brow;
    const char *const eib = (const char *)(p.EI + (row0 + t0) * C);
    const unsigned C16 = (unsigned)C * 16u, cc16 = (unsigned)cc * 16u;
    unsigned cpo16[TRN];  // label pl of tile tr (clamped: what lies beyond C lands in tile rows nobody stores), less pj rows
#pragma unroll
    for (int tr = 0; tr < TRN; ++tr) cpo16[tr] = (unsigned)min(tr * 16 + pl, C - 1) * 16u;
    auto ld2 = [](const char *base, const unsigned off) { return *(const double2 *)(base + off); };
    auto ld1 = [](const char *base, const unsigned off) { return *(const double *)(base + off); };
    // the block below tfrom; rows below the part's first are replaced by that one (nobody uses them)
    auto request = [&](const int tfrom) {
#pragma unroll
        for (int l = 0; l < NPL; ++l) {
            const unsigned o = (unsigned)(max(tfrom - 1 - l - pofs, ta) - t0) * C16 + cc16;
            aq[l] = ld2(arb, o);
            pv[l] = ld2(brb, o);
            e[l] = ld2(eib, o);
        }
        const unsigned om = (unsigned)(max(tfrom - 1 - pj, ta) - t0) * C16;
#pragma unroll
        for (int tr = 0; tr < TRN; ++tr) {
            aA[tr] = ld1(arb, om + cpo16[tr]);
            bB[tr] = ld1(brb, om + cpo16[tr]);
        }
        // what a scaling-block boundary at tfrom needs, fetched with every block: a load inside the (rare)
        // boundary branch would make the wave wait there for everything in flight
        const int i0 = max(tfrom - 1 - t0, 0);
        ya = arowY[i0];
        yb = browY[i0];
        const int jb = max(tfrom / J, 1);
        // (taken apart where it is used: a choice here puts the loads under a condition, and the wave waits for everything
        // it has just requested, block after block; genomic shape: call 506 -> 484 us with the
        // product above the stores)
        nhi = nbc[(size_t)min(jb, L / J) * C];
        nlo = nbc[(size_t)(jb - 1) * C];
    };
    // kappa(t,t) = exp((Y_alpha + Y_beta) ln2 - logZ) of the positions of a scaling block (they share both scales):
    // the stored scales are whole numbers, so it is one fixed factor in [1, 2) times a power of two
    const double kx = (Y0 + Ytop) - logZ * LOG2E, kxi = floor(kx);
    const double kfrac = exp2(kx - kxi);
    const int kint = whole_exponent(kxi);
    auto kappa_of = [&]() { return ldexp(kfrac, kint + (int)(ya + yb)); };

    int t = tb;
    const int rdoff = g * NK * RS + c;
    request(t);
    double kappa = kappa_of();
    // mass of the segments of a label that start / end at a position: z p kappa with z = q ES, and a b kappa with b = v IE
    // (no factor in these orders exceeds what BLOCK_NATS allows)
    // (a forbidden start or end has mass 0; so has one whose factor is below 1e-300, which is a score of -690)
    auto recip0 = [](const double x) { return x > 1e-300 ? recip(x) : 0.0; };
    auto start_mass = [&](const double2 &a, const double2 &ev, const double2 &v) {
        return BT ? a.y * recip0(ev.y) * v.x * kappa : a.y * kappa * ev.x * v.x;
    };
    auto end_mass = [&](const double2 &a, const double2 &ev, const double2 &v) {
        return BT ? a.x * recip0(ev.x) * v.y * kappa : a.x * kappa * v.y * ev.y;
    };
    const double wb = BT && p.grad_logz ? (double)p.grad_logz[b] : 1.0;
    // what a position gives the boundary outputs; on: it belongs to the block and the lane to a label
    auto boundary = [&](const int tt, const double out, const double in, const bool on) {
        if (!BT) return;
        if (p.g_proj_start && on) p.g_proj_start[((size_t)b * p.T + tt) * C + c] = (float)(wb * out);
        if (p.g_proj_end && on && tt >= 1) p.g_proj_end[((size_t)b * p.T + tt - 1) * C + c] = (float)(wb * in);
        if (p.bdy_post) {  // posterior of a boundary: total mass of the segments that end there
            double s = on && (SPLIT ? (lane & 31) : lane) < CTP ? in : 0.0;
            s = add_row_ror<1>(add_row_ror<2>(add_row_ror<4>(add_row_ror<8>(s))));
            s = add_across_16(s);
            if (!SPLIT) s = add_across_32(s);
            if (on && tt >= 1 && (SPLIT ? (lane & 31) : lane) == 0) p.bdy_post[(size_t)b * (p.T + 1) + tt] = (float)s;
        }
        if (tt == 0 && on) p.out0[(size_t)b * C + c] = out;
    };
    float *const gseq = p.grad_emis + ((size_t)b * p.T) * C;
    while (t > ta) {
        const int nb = min(min(t - ta, MB), ((t - 1) & Jm) + 1);
        if (__builtin_expect((t & Jm) == 0, 0)) {
            // the scan stepped into a new scaling block here: same shift of the live window, read off its scales
            const int nd = t >= J ? nhi - nlo : 0;  // (t <= L: the block of position t is there)
            G::template rescale_live<true>(ring, g, c, cval, r, nd - (int)(yb - ybPrev));
            ybPrev = yb;
            kappa = kappa_of();
        }
        if (__builtin_expect(r < MB, 0)) r = G::template move<true>(ring, lane, r);
        // ---- everything the block needs from its rows; v_t(c) enters the window at once (the rows below the
        // newest are not among those the block reads)
        double coef[MB];
        const bool whole = nb == MB && t - MB >= 1;
        {
            // transition statistics on the matrix cores (before the block's stores, whose number differs: a wait for these
            // operands behind them would be one for the stores); label rows beyond C are never stored, positions beyond a
            // short block's end must count nothing
            const bool on = whole || pj < nb;
#pragma unroll
            for (int tr = 0; tr < TRN; ++tr) {
                const double a = on ? aA[tr] * kappa : 0.0;
#pragma unroll
                for (int tc = 0; tc < TRN; ++tc)
                    accT[tr][tc] = __builtin_amdgcn_mfma_f64_16x16x4f64(a, bB[tc], accT[tr][tc], 0, 0, 0);
            }
        }
        if (SPLIT && whole) {
            // This lane's positions of the block: pofs + l, rows t-1-pofs-l.  A whole block (nearly all are) decides
            // nothing per position: every lane works on its label cc (the lanes of one label and half hold the same
            // rows and store the same values to the same places; what lanes beyond C add up is never stored).
            double dl[NPL];
#pragma unroll
            for (int l = 0; l < NPL; ++l) {
                both_halves(aq[l].y * kappa, coef[l], coef[NPL + l]);  // q_t(c) kappa of positions l and NPL + l
                // a segment of this label starts at the position (z p, z = q ES) / ends at it (a b, b = v IE)
                if (BT) {
                    const double out = start_mass(aq[l], e[l], pv[l]), in = end_mass(aq[l], e[l], pv[l]);
                    boundary(t - 1 - pofs - l, out, in, cval);
                    dl[l] = out - in;
                } else {
                    dl[l] = start_mass(aq[l], e[l], pv[l]) - end_mass(aq[l], e[l], pv[l]);
                }
            }
            // durations 1..3 inside the block: this lane's v rows with the coefficients of the later positions
            // (lower half: positions 0, 1; upper half: 2, 3; the two halves are added up at the end)
            const bool lowh = pofs == 0;
            const double k13 = lowh ? coef[1] : coef[3], k2 = lowh ? coef[2] : 0.0, k3 = lowh ? coef[3] : 0.0;
            dn[0] = fma(k13, pv[0].y, dn[0]);
            dn[1] = fma(k2, pv[0].y, dn[1]);
            dn[2] = fma(k3, pv[0].y, dn[2]);
            dn[0] = fma(k2, pv[1].y, dn[0]);
            dn[1] = fma(k3, pv[1].y, dn[1]);
            // running emission sums: R before the block, plus what the positions before this lane's add
            double s01, s23;
            both_halves(dl[0] + dl[1], s01, s23);
            const double r0 = lowh ? R : R + s01, r1 = r0 + dl[0];
            sR += r0 + r1;
            R = (R + s01) + s23;
            float *gp = gseq + ((unsigned)(t - 1 - pofs) * (unsigned)C + (unsigned)cc);
            double *rw = ring + (r - 1 - pofs) * RS + cc;
            rw[0] = pv[0].y;
            rw[-RS] = pv[1].y;
            gp[0] = (float)r0;
            gp[-C] = (float)r1;
        } else if (SPLIT) {
            // A short block (at most two at the part's upper end, the last one, the one with position 0): the
            // positions beyond its end count nothing and their stores go to the pad and to the sink.  The lanes
            // beyond C keep label cc's running sums here too: in whole blocks they store them.
            double dl[NPL];
            bool act[NPL];
#pragma unroll
            for (int l = 0; l < NPL; ++l) {
                const int tt = t - 1 - pofs - l;
                act[l] = pofs + l < nb;
                both_halves((act[l] && cval) ? aq[l].y * kappa : 0.0, coef[l], coef[NPL + l]);
                // none ends at position 0
                const double out = act[l] ? start_mass(aq[l], e[l], pv[l]) : 0.0;
                const double in = act[l] && tt >= 1 ? end_mass(aq[l], e[l], pv[l]) : 0.0;
                boundary(tt, out, in, act[l] && cval);
                dl[l] = out - in;
            }
            const bool lowh = pofs == 0;
            const double k13 = lowh ? coef[1] : coef[3], k2 = lowh ? coef[2] : 0.0, k3 = lowh ? coef[3] : 0.0;
            dn[0] = fma(k13, pv[0].y, dn[0]);
            dn[1] = fma(k2, pv[0].y, dn[1]);
            dn[2] = fma(k3, pv[0].y, dn[2]);
            dn[0] = fma(k2, pv[1].y, dn[0]);
            dn[1] = fma(k3, pv[1].y, dn[1]);
            double s01, s23;
            both_halves(dl[0] + dl[1], s01, s23);
            const double r0 = lowh ? R : R + s01, r1 = r0 + dl[0];
            sR += (act[0] ? r0 : 0.0) + (act[1] ? r1 : 0.0);
            R = (R + s01) + s23;
#pragma unroll
            for (int l = 0; l < NPL; ++l) {
                const int i = pofs + l;
                const bool on = act[l] && cval;
                double *rdst = on ? ring + (r - 1 - i) * RS + c : ring + RTOT + lane;
                *rdst = pv[l].y;
                float *dst = on ? gout + (unsigned)(t - 1 - i) * (unsigned)C : sink;
                *dst = (float)(l == 0 ? r0 : r1);
            }
        } else if (whole) {
            // 64 labels per lane group: every lane holds all four positions of its label
            float *gp = gseq + ((unsigned)(t - 1) * (unsigned)C + (unsigned)cc);
            double *rw = ring + (r - 1) * RS + cc;
#pragma unroll
            for (int i = 0; i < NPL; ++i) {
                coef[i] = aq[i].y * kappa;
#pragma unroll
                for (int jn = 0; jn < i; ++jn) dn[i - 1 - jn] = fma(coef[i], pv[jn].y, dn[i - 1 - jn]);
                rw[-i * RS] = pv[i].y;
                const double out = start_mass(aq[i], e[i], pv[i]), in = end_mass(aq[i], e[i], pv[i]);
                boundary(t - 1 - i, out, in, cval);
                const double d = out - in;
                gp[-i * C] = (float)R;
                sR += R;
                R += d;
            }
        } else {
#pragma unroll
            for (int i = 0; i < NPL; ++i) {
                const bool on = i < nb;
                const int tt = t - 1 - i;
                coef[i] = (cval && on) ? aq[i].y * kappa : 0.0;
                const double cg = g == 0 ? coef[i] : 0.0;
#pragma unroll
                for (int jn = 0; jn < i; ++jn) dn[i - 1 - jn] = fma(cg, pv[jn].y, dn[i - 1 - jn]);
                double *rdst = (on && writer) ? ring + (r - 1 - i) * RS + c : ring + RTOT + lane;
                *rdst = pv[i].y;
                const double out = on ? start_mass(aq[i], e[i], pv[i]) : 0.0;
                const double in = on && tt >= 1 ? end_mass(aq[i], e[i], pv[i]) : 0.0;
                boundary(tt, out, in, on && cval);
                const double d = out - in;
                float *dst = (on && writer) ? gout + (unsigned)tt * (unsigned)C : sink;
                *dst = (float)R;
                sR += on ? R : 0.0;
                R += d;
            }
        }
        // ---- the next block's rows
        request(t - nb);
        // window reads in groups of four, each group requested before the multiply-adds of the one before it
        // (all NK at once would cost their registers, one group at a time would wait for every one)
        const double *base = ring + r * RS + rdoff;
        double vc[4], vn[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) vc[q] = base[q * RS];
#pragma unroll
        for (int jg = 0; jg < NK; jg += 4) {
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (jg + 4 + q < NK) vn[q] = base[(jg + 4 + q) * RS];
#pragma unroll
            for (int q = 0; q < 4; ++q) {  // distance g*NK + jg + q from the newest (NK need not be a multiple of 4)
                if (jg + q < NK) {
#pragma unroll
                    for (int i = 0; i < MB; ++i) dx[jg + q + i] = fma(coef[i], vc[q], dx[jg + q + i]);
                }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < 4; ++q) vc[q] = vn[q];
        }
        r -= nb;
        lds_wave_fence();
        t -= nb;
    }
    // ---- partials of this task.  Duration sums: the strips of neighbouring lane groups overlap by MB-1
    // durations; they are combined through LDS in a fixed order (own strip, then the neighbour's overlap, then
    // the in-block terms) and scaled by W[k,c].
    lds_wave_fence();
    if (SPLIT) {  // what the two halves of the wave gathered separately
#pragma unroll
        for (int jj = 0; jj < MB - 1; ++jj) dn[jj] = add_across_32(dn[jj]);
        sR = add_across_32(sR);
    }
    double *tmp = ring;  // [KW + MB - 1][CT], row m = duration m + 1
    {
        double *tl = tmp + g * NK * CT + c;
        if (cval) {
#pragma unroll
            for (int jj = 0; jj < NK; ++jj) tl[jj * CT] = dx[jj];
        }
        if (cval && g == G::GW - 1) {
#pragma unroll
            for (int jj = NK; jj < NK + MB - 1; ++jj) tl[jj * CT] = 0.0;
        }
        lds_wave_fence();
        if (cval) {
#pragma unroll
            for (int jj = NK; jj < NK + MB - 1; ++jj) tl[jj * CT] += dx[jj];
        }
        lds_wave_fence();
        if (writer) {
#pragma unroll
            for (int jj = 0; jj < MB - 1; ++jj) tl[jj * CT] += dn[jj];
        }
        lds_wave_fence();
    }
    double *pD = p.partD + part * KC;
    if (cval) {
#pragma unroll 8
        for (int k = g; k < K; k += G::GW) pD[(size_t)k * C + c] = p.W[(size_t)k * C + c] * tmp[k * CT + c];
    }
    double *pT = p.partTr + part * CC;
#pragma unroll
    for (int tr = 0; tr < TRN; ++tr)
#pragma unroll
        for (int tc = 0; tc < TRN; ++tc)
#pragma unroll
            for (int v = 0; v < 4; ++v) {  // tile element (4v + lane/16, lane%16)
                const int src = tr * 16 + 4 * v + pj, dst = tc * 16 + pl;
                if (src < C && dst < C) pT[(size_t)src * C + dst] = accT[tr][tc][v];
            }
    if (lane < C) {
        p.tot[part * C + lane] = R;
        p.sumR[part * C + lane] = sR;
    }
}
