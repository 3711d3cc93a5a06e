// ---------------------------------------------------------------------------
// Duration-dependent transitions on the matrix cores (included by semicrf.hip after durtrans.inl).
//
// The recurrences of durtrans.inl, four interval tasks per workgroup in lock step, four positions of each at a time:
// sixteen (task, position) pairs are the rows (forward) or columns (backward) of v_mfma_f64_16x16x4 products with the
// table G[k][c'][c], so a table entry fetched from L2 once serves sixteen positions instead of four, and one
// instruction does 1024 multiply-adds.  (With vector multiply-adds, four positions per table entry and one task per
// workgroup, the scans of the genomic shape ran at 8 % of the fp64 rate: 4.65 and 5.3 ms; DESIGN has the figures.)
// fp64 matrix and vector instructions have the same peak here; what is won is table traffic, LDS operand traffic and
// instruction count.  Everything that is not the product with the table (scaling, the durations inside a block of four
// positions, checkpoints, stored rows) follows durtrans.inl, whose kernels still rescan what the verification rejects.
//
// Tasks of a workgroup are consecutive (sequence, interval) pairs; each has its own position, block length and scale, and
// the workgroup runs until all four are done (a finished task's rows are zeros).
//
// v_mfma_f64_16x16x4: A row = lane % 16, inner index = lane / 16; B inner index = lane / 16, column = lane % 16;
// D register v: row = 4 v + lane / 16, column = lane % 16.
// ---------------------------------------------------------------------------
constexpr int DX_TASKS = 4;   // tasks per workgroup
constexpr int DX_MB = 4;      // positions per block
constexpr int DX_NT = 512;    // threads: eight waves, two per SIMD
typedef double dx_d4 __attribute__((ext_vector_type(4)));

struct DxGeom {
    int khp;          // half of the durations, rounded up to a multiple of four (forward tiles hold two halves)
    int ncg;          // label groups of eight (forward tiles)
    int sf2;          // pairs of inner steps of the forward product (source labels, eight per pair)
    int mt;           // tiles of sixteen source labels (backward, marginals)
    int ks;           // inner steps of the backward product (four durations each), even
    int kr;           // ring slots: K + 4, so that all targets of a block are different slots, and at least 8, so that
                      // the next block's four slots are not those of this one
    int xs, ts;       // doubles per task of the forward / backward ring
    int cp, cpb;      // row length of the small per-position arrays
    size_t gf, gb;    // doubles of the two tables in operand order
    size_t lds_f, lds_b;
    bool ok;
};

__host__ __device__ inline DxGeom dx_geometry(const int K, const int C)
{
    DxGeom g;
    g.khp = ((K + 1) / 2 + 3) & ~3;
    g.ncg = (C + 7) / 8;
    g.sf2 = (C + 7) / 8;
    g.mt = (C + 15) / 16;
    g.ks = ((K + 3) / 4 + 1) & ~1;
    g.kr = K + DX_MB < 2 * DX_MB ? 2 * DX_MB : K + DX_MB;
    // tasks 8 doubles (16 LDS banks) apart modulo the banks: the four tasks of an access do not collide
    g.xs = ((g.kr * C + 31) & ~31) + 8;
    g.ts = ((g.kr * C + 31) & ~31) + 8;
    g.cp = 8 * g.sf2;
    g.cpb = 16 * g.mt;
    g.gf = (size_t)g.ncg * g.khp * g.sf2 * 128;
    g.gb = (size_t)C * g.ks * g.mt * 64;
    g.lds_f = ((size_t)DX_TASKS * g.xs + 2 * (size_t)16 * g.cp) * sizeof(double) + 64;
    g.lds_b = ((size_t)DX_TASKS * g.ts + 5 * (size_t)16 * g.cpb + (size_t)8 * C * 16 + (size_t)(DX_MB - 1) * C * C) * sizeof(double) + 64;
    g.ok = C <= 32 && g.lds_f <= LDS_LIMIT && g.lds_b <= LDS_LIMIT;
    return g;
}

// The table in the operand order of the two products (zero beyond K and C):
//   forward   [label group][kk][step pair][lane][2]: column j = lane % 16 is duration kk + 1 + (j / 8) khp, label
//             8 group + j % 8; inner index: source label 8 pair + 4 (0, 1) + lane / 16
//   backward  [label][step][lane][mt] (two label tiles) or [label][step pair][lane][2] (one): row: source label
//             16 mt + lane % 16, inner index: duration 4 step + lane / 16 + 1
__global__ __launch_bounds__(NT) void k_dx_tables(Params p)
{
    const int K = p.K, C = p.C, CC = C * C;
    const DxGeom g = dx_geometry(K, C);
    const size_t n0 = (size_t)K * CC, n1 = n0 + g.gf, n2 = n1 + g.gb;
    const size_t i = (size_t)blockIdx.x * NT + threadIdx.x;
    if (i >= n2) return;
    int k, o, c;  // duration (from 1), source label, label
    double *dst;
    if (i < n0) {
        k = (int)(i / CC) + 1;
        o = (int)(i % CC) / C;
        c = (int)(i % C);
        dst = p.G3 + i;
    } else if (i < n1) {
        const size_t q = i - n0;
        const int u = (int)(q & 1), lane = (int)(q >> 1) & 63, j = lane & 15;
        const size_t tile = (q >> 7) / g.sf2;
        const int s = (int)((q >> 7) % g.sf2);
        k = (int)(tile % g.khp) + 1 + (j >> 3) * g.khp;
        c = (int)(tile / g.khp) * 8 + (j & 7);
        o = 8 * s + 4 * u + (lane >> 4);
        dst = p.GF + q;
    } else {
        const size_t q = i - n1;
        const int u = (int)(q & 1), lane = (int)(q >> 1) & 63;
        const size_t r = q >> 7;  // label * steps + step (two tiles), label * step pairs + pair (one)
        const int per = g.mt == 2 ? g.ks : g.ks / 2;
        c = (int)(r / per);
        const int s = g.mt == 2 ? (int)(r % per) : 2 * (int)(r % per) + u;
        o = (g.mt == 2 ? 16 * u : 0) + (lane & 15);
        k = 4 * s + (lane >> 4) + 1;
        dst = p.GB + q;
    }
    *dst = (k <= K && o < C && c < C)
               ? exp((double)p.dur[(size_t)(k - 1) * C + c] + (double)p.trans3[((size_t)(k - 1) * C + o) * C + c])
               : 0.0;
}

// One task of a lock-step workgroup: the same values in all 128 threads that own it.
struct DxTask {
    int b, chunk, L, J, lo, hi;
    bool active;
};
__device__ __forceinline__ DxTask dx_task(const Params &p, const int id, const int dir, const int tier)
{
    DxTask t;
    t.active = id < p.B * p.N;
    t.b = t.active ? id / p.N : 0;
    t.chunk = t.active ? id % p.N : 0;
    if (tier > 0 && t.active && p.spec_ok[t.b * 2 + dir]) t.active = false;
    const SeqHdr h = p.hdr[t.b];
    t.L = h.L;
    t.J = h.J;
    t.lo = t.chunk * p.Delta;
    if (t.lo >= t.L) t.active = false;
    t.hi = min(t.lo + p.Delta, t.L);
    return t;
}

__device__ __forceinline__ int dx_wrap(int i, const int kr) { return i >= kr ? i - kr : (i < 0 ? i + kr : i); }

// ---------------------------------------------------------------------------
// Forward ("push"): the product of a block's sixteen message rows with the whole table; column (k, c) of row (task, t)
// goes, times IE_t(c), into the ring entry of position t + k.  A lane holds the four positions of one task for its
// column and walks consecutive durations of one label, so the four positions' terms for one target are added up in
// registers and the ring is touched once per duration.  Waves own whole runs of durations (multiples of four); the last three
// targets of a run belong to the next run too and are added after a barrier: every entry has one writer at a time and
// the order of additions is fixed.
// ---------------------------------------------------------------------------
template <int SF2>
__global__ __launch_bounds__(DX_NT, 2) void k_dx_fwd(Params p, int warm, int tier)
{
    extern __shared__ double lds_raw[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g4 = lane >> 4, j = lane & 15;
    const int K = p.K, C = p.C, CC = C * C, KC = K * C, N = p.N;
    const DxGeom g = dx_geometry(K, C);
    const int KR = g.kr, KHP = g.khp, XS = g.xs;
    constexpr int CP = 8 * SF2;
    double *X = lds_raw;                       // [task][slot][C] partial sums of the positions to come
    double *av = X + DX_TASKS * XS;            // [task][pos][CP] message vectors of the block (zero beyond it)
    double *ieL = av + 16 * CP;                // [task][pos][CP] 1/ES
    int *ctl = (int *)(ieL + 16 * CP);         // [task] block length, [task] slot of its first position, [task] rebase
    const int q = wave >> 1;                   // the thread's own task, its position in a block and label
    const int pos = (tid >> 5) & 3, c = tid & 31;
    const bool cv = c < C;
    const DxTask tk = dx_task(p, blockIdx.x * DX_TASKS + q, 0, tier);
    const int L = tk.L, J = tk.J, lo = tk.lo, hi = tk.hi;
    const int s0 = max(lo - warm, 0);
    const size_t row0 = (size_t)tk.b * (p.T + 1);
    const double2 *EI = p.EI + row0 * C + (cv ? c : 0);
    const int *nb = p.nbase + row0 * C + (cv ? c : 0);
    double *rowA = p.dtA + row0 * C, *rowY = p.dtY + row0;
    const size_t ckstride = (size_t)KC + C;
    double *Xq = X + q * XS, *avq = av + q * 4 * CP, *ieq = ieL + q * 4 * CP;

    // column c of the tables of the durations inside a block (thread's duration pos + 1)
    double gcol[CP];
#pragma unroll
    for (int o = 0; o < CP; ++o)
        gcol[o] = (pos < DX_MB - 1 && pos < K && cv && o < C) ? p.G3[(size_t)pos * CC + (size_t)o * C + c] : 0.0;

    for (int i = tid; i < DX_TASKS * XS + 2 * 16 * CP; i += DX_NT) lds_raw[i] = 0.0;
    double Y = 0.0, Ybase = 0.0;
    int t0 = s0, rb = 0, last = 0;  // rb: ring slot of t0; last: position of the newest message vector in av
    bool done = !tk.active;
    auto load_ei = [&](const int tb) {
        double2 e = make_double2(0.0, 0.0);
        if (!done && cv && tb + pos <= hi) e = EI[(size_t)(tb + pos) * C];
        return e;
    };
    double2 e = load_ei(t0);
    lds_barrier();

    // runs of durations: units of four tiles, a contiguous share per wave
    const int units = g.ncg * (KHP / 4), per = (units + 7) / 8;
    const int u0 = wave * per, u1 = min(u0 + per, units);

    for (;;) {
        int nbk = 0;
        bool bd = false;
        if (!done) {
            nbk = min(DX_MB, hi - t0 + 1);
            if (t0 <= lo) nbk = min(nbk, lo - t0 + 1);  // the interval's first position ends its block
            nbk = min(nbk, J - (t0 & (J - 1)));         // no scaling-block boundary inside a block
            bd = t0 > s0 && (t0 & (J - 1)) == 0;
        }
        if ((tid & 127) == 0) {
            ctl[q] = nbk;
            ctl[4 + q] = rb;
            ctl[8 + q] = bd;
        }
        lds_barrier();
        if ((ctl[0] | ctl[1] | ctl[2] | ctl[3]) == 0) break;
        if (ctl[8] | ctl[9] | ctl[10] | ctl[11]) {
            if (bd) {
                double pm = 0.0;
                for (int i = 0; i < C; ++i) pm += avq[last * CP + i];
                const int ex = safe_exponent(pm);
                Y += (double)ex;
                if (cv) {
                    const int sft = nb[(size_t)(t0 / J) * C] - nb[(size_t)(t0 / J - 1) * C] - ex;
                    for (int r = pos; r < KR; r += 4) Xq[r * C + c] = fmin(ldexp(Xq[r * C + c], sft), DBL_MAX);
                }
            }
            lds_barrier();
        }
        // ---- the block's positions, one after the other
        if (cv) ieq[pos * CP + c] = pos < nbk ? e.y : 0.0;
#pragma unroll
        for (int i = 0; i < DX_MB; ++i) {
            if (pos == i && cv) {
                double a = 0.0;
                const int tt = t0 + i;
                if (i < nbk) {
                    a = tt == s0 ? 1.0 : e.x * Xq[dx_wrap(rb + i, KR) * C + c];
                    if (tt > lo || tt == 0) rowA[(size_t)tt * C + c] = a;
                    if (c == 0 && (tt > lo || tt == 0)) rowY[tt] = Y - Ybase;
                }
                avq[i * CP + c] = a;
            }
            lds_barrier();
            if (i < DX_MB - 1) {
                // durations that stay inside the block: duration pos + 1
                if (pos < DX_MB - 1 && pos < K && cv && i + pos + 1 < nbk) {
                    double m0 = 0.0, m1 = 0.0;
                    const double2 *a2 = (const double2 *)(avq + i * CP);
#pragma unroll
                    for (int o = 0; o < CP / 2; ++o) {
                        const double2 v = a2[o];
                        m0 = fma(v.x, gcol[2 * o], m0);
                        m1 = fma(v.y, gcol[2 * o + 1], m1);
                    }
                    double *x = Xq + dx_wrap(rb + i + pos + 1, KR) * C + c;
                    *x = fma(ieq[i * CP + c], m0 + m1, *x);
                }
                lds_barrier();
            }
        }
        if (nbk) last = nbk - 1;
        const double2 en = load_ei(t0 + nbk);  // the next block's factors, requested before the long part
        // ---- durations that leave the block
        {
            double A[2 * SF2];
#pragma unroll
            for (int s = 0; s < 2 * SF2; ++s) A[s] = av[((j & 3) * 4 + (j >> 2)) * CP + 4 * s + g4];
            const int nbD = ctl[g4], rbD = ctl[4 + g4];
            double *XD = X + g4 * XS;
            const double2 *GF = (const double2 *)p.GF + lane;
            double2 Bn[SF2];
            auto fetch = [&](const int tile, double2 (&B)[SF2]) {
#pragma unroll
                for (int s = 0; s < SF2; ++s) B[s] = GF[((size_t)tile * SF2 + s) * 64];
            };
            // sums whose targets the next run writes too, per run (a wave's share meets at most two label groups)
            double pend[2][3];
            int pslot[2] = {0, 0}, pk[2] = {0, 0};
            bool first = true;
            double w1 = 0.0, w2 = 0.0, w3 = 0.0, ier[DX_MB];
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int i = 0; i < 3; ++i) pend[a][i] = 0.0;
#pragma unroll
            for (int i = 0; i < DX_MB; ++i) ier[i] = 0.0;
            if (u0 < u1) fetch(u0 * 4, Bn);
            int cg = -1, cl = 0;
            for (int tile = u0 * 4; tile < u1 * 4; ++tile) {
                double2 B[SF2];
#pragma unroll
                for (int s = 0; s < SF2; ++s) B[s] = Bn[s];
                if (tile + 1 < u1 * 4) fetch(tile + 1, Bn);
                const int ncg = tile / KHP, kk = tile - ncg * KHP;
                if (ncg != cg) {  // uniform: a new label group (the first one included)
                    cg = ncg;
                    cl = cg * 8 + (j & 7);
#pragma unroll
                    for (int i = 0; i < DX_MB; ++i) ier[i] = ieL[(g4 * 4 + i) * CP + cl];
                    w1 = w2 = w3 = 0.0;
                }
                dx_d4 D = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 0; s < SF2; ++s) {
                    D = __builtin_amdgcn_mfma_f64_16x16x4f64(A[2 * s], B[s].x, D, 0, 0, 0);
                    D = __builtin_amdgcn_mfma_f64_16x16x4f64(A[2 * s + 1], B[s].y, D, 0, 0, 0);
                }
                const int k1 = kk + 1 + (j >> 3) * KHP;  // the lane's duration
                double d0 = ier[0] * D[0], d1 = ier[1] * D[1], d2 = ier[2] * D[2], d3 = ier[3] * D[3];
                if (kk < DX_MB - 1 && k1 < DX_MB) {  // targets inside the block were served above
                    d0 = k1 >= nbD ? d0 : 0.0;
                    d1 = k1 + 1 >= nbD ? d1 : 0.0;
                    d2 = k1 + 2 >= nbD ? d2 : 0.0;
                    d3 = k1 + 3 >= nbD ? d3 : 0.0;
                }
                const double w0 = w1 + d0;
                w1 = w2 + d1;
                w2 = w3 + d2;
                w3 = d3;
                if (cl < C && k1 <= K + DX_MB - 1) {
                    double *x = XD + dx_wrap(rbD + k1, KR) * C + cl;
                    *x += w0;
                }
                if (tile + 1 == u1 * 4 || kk + 1 == KHP) {  // uniform: the run ends
                    if (first) {
                        pend[0][0] = w1; pend[0][1] = w2; pend[0][2] = w3;
                        pk[0] = k1;
                        pslot[0] = cl;
                    } else {
                        pend[1][0] = w1; pend[1][1] = w2; pend[1][2] = w3;
                        pk[1] = k1;
                        pslot[1] = cl;
                    }
                    first = false;
                }
            }
            lds_barrier();
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const int k1 = pk[a] + 1 + i;
                    if (pk[a] > 0 && pslot[a] < C && k1 <= K + DX_MB - 1) XD[dx_wrap(rbD + k1, KR) * C + pslot[a]] += pend[a][i];
                }
            if (cv && pos < nbk) Xq[dx_wrap(rb + pos, KR) * C + c] = 0.0;  // consumed: free for a later target
        }
        lds_barrier();
        // ---- checkpoints
        const int tlast = t0 + nbk - 1;
        t0 += nbk;
        rb = dx_wrap(rb + nbk, KR);
        e = en;
        if (!done) {
            auto record = [&](double *ck, double *ckY) {
                if (cv) {
                    for (int d = pos; d < K; d += 4) {  // position t0 + d
                        ck[(size_t)((t0 + d) % K) * C + c] = Xq[dx_wrap(rb + d, KR) * C + c];
                    }
                    if (pos == 0) ck[KC + c] = avq[last * CP + c];
                }
                if ((tid & 127) == 0) *ckY = Y;
            };
            const size_t at = (size_t)tk.b * (N + 1) + tk.chunk;
            if (tlast == lo) {
                record(p.ckA + at * ckstride, p.ckYA + at);
                Ybase = Y;
            }
            if (t0 > hi) {
                record(p.ckA2 + (at + 1) * ckstride, p.ckYA2 + at + 1);
                done = true;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Backward ("pull"): for every label c a product [source labels] x [durations] . [durations] x [sixteen (task,
// position) columns] of the table with the ring of v; IE_t(c) is applied to its result, which is then added up over
// the labels (b_t) and, weighted with a_t, over the source labels (mass of the segments that start at t).  A wave takes the
// labels wave, wave + 8, ...; the waves' sums for b meet in LDS.
// ---------------------------------------------------------------------------
template <int MT>
__global__ __launch_bounds__(DX_NT, 2) void k_dx_bwd(Params p, int warm, int tier)
{
    extern __shared__ double lds_raw[];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g4 = lane >> 4, j = lane & 15;
    const int K = p.K, C = p.C, CC = C * C, KC = K * C, N = p.N;
    const DxGeom g = dx_geometry(K, C);
    const int KR = g.kr, TS = g.ts, KS = g.ks;
    constexpr int CPB = 16 * MT;
    double *V = lds_raw;                       // [task][C][slot] v of the positions above
    double *avL = V + DX_TASKS * TS;           // [task][pos][CPB] a_t
    double *ieL = avL + 16 * CPB;              // [task][pos][CPB] 1/ES
    double *esL = ieL + 16 * CPB;              // [task][pos][CPB] ES
    double *bL = esL + 16 * CPB;               // [task][pos][CPB] b_t
    double *oL = bL + 16 * CPB;                // [task][pos][CPB] segments that start at t and leave the block
    double *bp = oL + 16 * CPB;                // [wave][C][16] the waves' shares of b
    double *Gs = bp + 8 * C * 16;              // [DX_MB-1][C][C] the durations inside a block
    int *ctl = (int *)(Gs + (DX_MB - 1) * CC);
    const int q = wave >> 1;
    const int pos = (tid >> 5) & 3, c = tid & 31;    // own (task, position, label)
    const int cs = (tid >> 2) & 31, sl = tid & 3;    // own (source label, slice of the labels) in the serial part
    const bool cv = c < C;
    const DxTask tk = dx_task(p, blockIdx.x * DX_TASKS + q, 1, tier);
    const int L = tk.L, J = tk.J, lo = tk.lo, hi = tk.hi;
    const int s1 = min(hi + warm, L);
    const size_t row0 = (size_t)tk.b * (p.T + 1);
    const double2 *EI = p.EI + row0 * C + (cv ? c : 0);
    const int *nb = p.nbase + row0 * C + (cv ? c : 0);
    const double *rowA = p.dtA + row0 * C + (cv ? c : 0);
    double *rowV = p.dtV + row0 * C, *rowD = p.dtD + row0 * C, *rowYb = p.dtYb + row0;
    const size_t ckstride = (size_t)KC + C;
    double *Vq = V + q * TS;
    const int qo = q * 4 * CPB;

    for (int i = tid; i < DX_TASKS * TS + 5 * 16 * CPB; i += DX_NT) lds_raw[i] = 0.0;
    for (int i = tid; i < (DX_MB - 1) * CC; i += DX_NT) Gs[i] = i < K * CC ? p.G3[i] : 0.0;
    lds_barrier();
    // table entries of the serial part: durations 1 .. 3, source label cs, labels sl, sl + 4, ...
    double gr[DX_MB - 1][8];
#pragma unroll
    for (int k = 0; k < DX_MB - 1; ++k)
#pragma unroll
        for (int m = 0; m < 8; ++m) {
            const int cc = sl + 4 * m;
            gr[k][m] = (cs < C && cc < C) ? Gs[(k * C + cs) * C + cc] : 0.0;
        }
    bool done = !tk.active;
    double Yb = 0.0, Ytop = 0.0;
    int t0 = s1 - 1, rb = KR - 1;  // slot of s1 is 0, of s1 - 1 is KR - 1, ...
    // a sequence that ends at s1 (exactly so when s1 = L): b = 1, v = ES; scale reference: a single 1
    if (!done && cv && pos == 0) {
        const double v = EI[(size_t)s1 * C].x;
        Vq[c * KR] = v;
        bL[qo + c] = c == 0 ? 1.0 : 0.0;
        if (s1 == L) rowV[(size_t)L * C + c] = v;
        if (s1 == L && c == 0) rowYb[L] = 0.0;
    }
    int last = 0;  // position of the newest b in bL
    double2 e = make_double2(0.0, 0.0);
    double a = 0.0;
    auto load_rows = [&](const int tb) {
        e = make_double2(0.0, 0.0);
        a = 0.0;
        if (!done && cv && tb - pos >= lo) {
            e = EI[(size_t)(tb - pos) * C];
            a = rowA[(size_t)(tb - pos) * C];
        }
    };
    load_rows(t0);

    for (;;) {
        int nbk = 0;
        bool bd = false;
        if (!done) {
            nbk = min(DX_MB, t0 - lo + 1);
            if (t0 >= hi) nbk = min(nbk, t0 - hi + 1);     // the interval's upper end ends its block
            nbk = min(nbk, (t0 & (J - 1)) + 1);             // no scaling-block boundary inside a block
            bd = ((t0 + 1) & (J - 1)) == 0;
        }
        if ((tid & 127) == 0) {
            ctl[q] = nbk;
            ctl[4 + q] = rb;
            ctl[8 + q] = bd;
        }
        lds_barrier();
        if ((ctl[0] | ctl[1] | ctl[2] | ctl[3]) == 0) break;
        if (ctl[8] | ctl[9] | ctl[10] | ctl[11]) {
            if (bd) {
                double pm = 0.0;
                for (int i = 0; i < C; ++i) pm += bL[qo + last * CPB + i];
                const int ex = safe_exponent(pm);
                Yb += (double)ex;
                if (cv) {
                    const int sft = nb[(size_t)(t0 / J + 1) * C] - nb[(size_t)(t0 / J) * C] - ex;
                    for (int r = pos; r < KR; r += 4) Vq[c * KR + r] = fmin(ldexp(Vq[c * KR + r], sft), DBL_MAX);
                }
            }
            lds_barrier();
        }
        // rows of the block (zeros beyond it), then the next block's requested
        if (cv) {
            const bool in = pos < nbk;
            avL[qo + pos * CPB + c] = in ? a : 0.0;
            ieL[qo + pos * CPB + c] = in ? e.y : 0.0;
            esL[qo + pos * CPB + c] = in ? e.x : 0.0;
        }
        const double a_own = a, ie_own = e.y;
        load_rows(t0 - nbk);
        lds_barrier();
        // ---- durations that reach beyond the block (entries of its own positions are zeros in the ring)
        {
            const int tn = j & 3, pn = j >> 2;  // column: task, position
            double An[4 * MT], bacc[MT][4];
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    An[4 * m + v] = avL[(tn * 4 + pn) * CPB + 16 * m + 4 * v + g4];
                    bacc[m][v] = 0.0;
                }
            const int ib = dx_wrap(ctl[4 + tn] - pn, KR);
            const int i0 = dx_wrap(ib + g4 + 1, KR);
            for (int cc = wave; cc < C; cc += 8) {
                const double *Vc = V + tn * TS + cc * KR;
                const double2 *GB = (const double2 *)p.GB + (size_t)cc * KS * MT * 32 + lane;
                dx_d4 D[MT];
#pragma unroll
                for (int m = 0; m < MT; ++m) D[m] = dx_d4{0.0, 0.0, 0.0, 0.0};
                // steps in pairs; the table entries of a pair are requested two pairs ahead
                constexpr int LP = MT;  // double2 loads per pair of steps
                double2 G0[LP], G1[LP];
                const int np = KS / 2;
#pragma unroll
                for (int u = 0; u < LP; ++u) {
                    G0[u] = GB[(size_t)u * 64];
                    G1[u] = GB[(size_t)(min(1, np - 1) * LP + u) * 64];
                }
                int idx = i0;
                for (int s = 0; s < np; ++s) {
                    const int idx2 = dx_wrap(idx + 4, KR);
                    const double b0 = Vc[idx], b1 = Vc[idx2];
                    idx = dx_wrap(idx2 + 4, KR);
                    double2 Gc[LP];
#pragma unroll
                    for (int u = 0; u < LP; ++u) {
                        Gc[u] = G0[u];
                        G0[u] = G1[u];
                        G1[u] = GB[(size_t)(min(s + 2, np - 1) * LP + u) * 64];
                    }
                    if (MT == 2) {  // .x, .y: the two label tiles of one step
                        D[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(Gc[0].x, b0, D[0], 0, 0, 0);
                        D[MT - 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(Gc[0].y, b0, D[MT - 1], 0, 0, 0);
                        D[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(Gc[LP - 1].x, b1, D[0], 0, 0, 0);
                        D[MT - 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(Gc[LP - 1].y, b1, D[MT - 1], 0, 0, 0);
                    } else {        // .x, .y: the two steps
                        D[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(Gc[0].x, b0, D[0], 0, 0, 0);
                        D[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(Gc[0].y, b1, D[0], 0, 0, 0);
                    }
                }
                const double ie = ieL[(tn * 4 + pn) * CPB + cc];
                double o = 0.0;
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        bacc[m][v] = fma(ie, D[m][v], bacc[m][v]);
                        o = fma(An[4 * m + v], D[m][v], o);
                    }
                o = add_across_32(add_across_16(o));
                if (g4 == 0) oL[(tn * 4 + pn) * CPB + cc] = ie * o;
            }
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = 16 * m + 4 * v + g4;
                    if (r < C) bp[(wave * C + r) * 16 + j] = bacc[m][v];
                }
        }
        // what a segment of duration k <= pos inside the block adds to the mass that starts at the thread's position:
        // sum over the source labels of a G[k] (the factor v follows when it is known)
        double wk[DX_MB - 1];
#pragma unroll
        for (int k = 0; k < DX_MB - 1; ++k) {
            wk[k] = 0.0;
            if (cv && k < pos && pos < nbk) {
                double m = 0.0;
#pragma unroll 8
                for (int o = 0; o < C; ++o) m = fma(avL[qo + pos * CPB + o], Gs[(k * C + o) * C + c], m);
                wk[k] = m;
            }
        }
        lds_barrier();
        if (cs < C) {
            double b = 0.0;
#pragma unroll
            for (int w = 0; w < 8; ++w) b += bp[(w * C + cs) * 16 + q + 4 * sl];
            bL[qo + sl * CPB + cs] = b;
        }
        lds_barrier();
        // ---- finish the positions one after the other
#pragma unroll
        for (int i = 0; i < DX_MB; ++i) {
            if (i < nbk && cs < C) {
                double s = 0.0;
#pragma unroll
                for (int k = 1; k <= i; ++k) {
                    const int slot = dx_wrap(rb - i + k, KR);  // position t0 - i + k, finished just before
#pragma unroll
                    for (int m = 0; m < 8; ++m) {
                        const int cc = sl + 4 * m;
                        if (cc < C) s = fma(gr[k - 1][m], ieL[qo + i * CPB + cc] * Vq[cc * KR + slot], s);
                    }
                }
                if (i > 0) {  // over the four slices: lanes of a quad
                    s += __shfl_xor(s, 1);
                    s += __shfl_xor(s, 2);
                }
                if (sl == 0) {
                    const double b = bL[qo + i * CPB + cs] + s;
                    bL[qo + i * CPB + cs] = b;
                    Vq[cs * KR + dx_wrap(rb - i, KR)] = b * esL[qo + i * CPB + cs];
                }
            }
            lds_barrier();
        }
        if (nbk) last = nbk - 1;
        if (cv && pos < nbk) {
            const int tt = t0 - pos;
            if (tt < hi) {
                const double b = bL[qo + pos * CPB + c];
                double o = oL[qo + pos * CPB + c];
#pragma unroll
                for (int k = 1; k < DX_MB; ++k)
                    if (k <= pos) o = fma(wk[k - 1] * ie_own, Vq[c * KR + dx_wrap(rb - pos + k, KR)], o);
                rowV[(size_t)tt * C + c] = Vq[c * KR + dx_wrap(rb - pos, KR)];
                rowD[(size_t)tt * C + c] = o - (tt >= 1 ? a_own * b : 0.0);
                if (c == 0) rowYb[tt] = Yb - Ytop;
            }
        }
        const int tlast = t0 - nbk + 1;
        const int rlast = dx_wrap(rb - nbk + 1, KR);  // slot of tlast
        t0 -= nbk;
        rb = dx_wrap(rb - nbk, KR);
        // slots of the next block's positions: free (their old contents lie more than K above)
        if (!done && cv) Vq[c * KR + dx_wrap(rb - pos, KR)] = 0.0;
        if (!done) {
            auto record = [&](double *ck, double *ckY) {
                if (cv) {
                    for (int d = pos; d < K; d += 4) {  // position tlast + d
                        ck[(size_t)((tlast + d) % K) * C + c] = Vq[c * KR + dx_wrap(rlast + d, KR)];
                    }
                    if (pos == 0) ck[KC + c] = bL[qo + last * CPB + c];
                }
                if ((tid & 127) == 0) *ckY = Yb;
            };
            const size_t at = (size_t)tk.b * (N + 1);
            if (tlast == hi && hi < L) {
                record(p.ckB + (at + tk.chunk + 1) * ckstride, p.ckYB + at + tk.chunk + 1);
                Ytop = Yb;
            }
            if (tlast == lo) {
                if (lo > 0) record(p.ckB2 + (at + tk.chunk) * ckstride, p.ckYB2 + at + tk.chunk);
                done = true;
            }
        }
    }
}

// ---------------------------------------------------------------------------
// Running emission-gradient sums per interval (as k_dt_emis, for the same consumers): one workgroup per (sequence,
// interval), eight contiguous segments of positions side by side.  A segment is summed, the segments above it are added,
// then it is walked again.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(NT) void k_dx_emis(Params p)
{
    __shared__ double segR[8][32], segS[8][32];
    const int b = blockIdx.x / p.N, jv = blockIdx.x % p.N;
    const int sg = threadIdx.x >> 5, c = threadIdx.x & 31;
    const int C = p.C, Delta = p.Delta, N = p.N;
    const int L = p.hdr[b].L;
    const int lo = jv * Delta;
    if (lo >= L) return;
    const int hi = min(lo + Delta, L);
    const size_t row0 = (size_t)b * (p.T + 1);
    const double *rowD = p.dtD + row0 * C;
    const double *rowY = p.dtY + row0, *rowYb = p.dtYb + row0;
    const double *ckYA = p.ckYA + (size_t)b * (N + 1);
    const double logZ = p.hdr[b].logZ;
    const double ytop = dt_ytop(p, b, jv, L);
    const int per = (hi - lo + 7) / 8;
    const int th = hi - sg * per, tl = max(lo, th - per);  // positions tl .. th-1, walked downwards
    const bool act = c < C;
    double R = 0.0, sR = 0.0;
    for (int pass = 0; pass < 2; ++pass) {
        double kappa = 0.0, kY = -1.0e300;
        for (int t1 = th; t1 > tl; t1 -= 8) {
            double d[8], y[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int tt = max(t1 - 1 - i, tl);
                d[i] = act ? rowD[(size_t)tt * C + c] : 0.0;
                y[i] = ckYA[tt == 0 ? 0 : (tt - 1) / Delta] + rowY[tt] + ytop + rowYb[tt];
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int tt = t1 - 1 - i;
                if (tt < tl) break;
                if (y[i] != kY) {  // the same in the 32 lanes of a segment
                    kY = y[i];
                    kappa = exp(kY * LN2 - logZ);
                }
                if (pass && act) p.grad_emis[((size_t)b * p.T + tt) * C + c] = (float)R;
                sR += R;
                R = fma(d[i], kappa, R);
            }
        }
        if (pass) break;
        segR[sg][c] = R;
        __syncthreads();
        R = 0.0;
        sR = 0.0;
        for (int s = 0; s < sg; ++s) R += segR[s][c];
    }
    segS[sg][c] = sR;
    __syncthreads();
    // the last segment's running sum is the interval's total (empty segments carry it on)
    if (sg == 7 && act) {
        double s = 0.0;
        for (int i = 0; i < 8; ++i) s += segS[i][c];
        p.tot[((size_t)b * p.NP + jv) * C + c] = R;
        p.sumR[((size_t)b * p.NP + jv) * C + c] = s;
    }
}

// ---------------------------------------------------------------------------
// Marginals (the sums of k_dt_acc): for every label c a product [source labels] x [positions] . [positions] x
// [durations] of a_t(c') with IE_t(c) v_{t+k}(c).  A wave owns one label and 64 durations (four tiles) for a persistent
// share of the (sequence, interval) tasks: its sums stay in the accumulators; a workgroup is eight waves, which share
// the staged a rows.  grid (shares, ceil(C * ceil(K/64) / 8)).
// ---------------------------------------------------------------------------
constexpr int DXA_K = 64;
constexpr int DXA_VR = DT_TG + DXA_K + 4;   // rows of v a group of positions can reach
constexpr int DXA_W = 8;                     // waves per workgroup
__host__ __device__ constexpr size_t dxa_lds_doubles(int mt) { return (size_t)DT_TG * (16 * mt + 1) + (size_t)DXA_W * (DT_TG + DXA_VR); }
template <int MT>
__global__ __launch_bounds__(64 * DXA_W, 2) void k_dx_acc(Params p)
{
    extern __shared__ double lds_raw[];
    constexpr int AS = 16 * MT + 1;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g4 = lane >> 4, j = lane & 15;
    const int K = p.K, C = p.C, CC = C * C, N = p.N, Delta = p.Delta;
    const int kgs = (K + DXA_K - 1) / DXA_K;
    const int item = blockIdx.y * DXA_W + wave;
    const bool mine = item < C * kgs;
    const int c = mine ? item / kgs : 0, kA = mine ? (item % kgs) * DXA_K : 0;  // durations kA + 1 .. kA + 64
    double *Arow = lds_raw;                            // [DT_TG][AS]  a_t(c') w_b 2^(YA(t) - YA(group)), zero beyond C
    double *IEw = Arow + DT_TG * AS + wave * (DT_TG + DXA_VR);  // [DT_TG] 1/ES of the wave's label
    double *Vw = IEw + DT_TG;                          // [DXA_VR] v of the wave's label from position group + kA + 1 on
    dx_d4 acc[MT][4];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int k = 0; k < 4; ++k) acc[m][k] = dx_d4{0.0, 0.0, 0.0, 0.0};

    const int ntask = p.B * N;
    for (int task = blockIdx.x; task < ntask; task += gridDim.x) {
        const int b = task / N, chunk = task % N;
        const SeqHdr h = p.hdr[b];
        const int L = h.L, J = h.J;
        const int lo = chunk * Delta;
        if (lo >= L) continue;
        const int hi = min(lo + Delta, L);
        const size_t row0 = (size_t)b * (p.T + 1);
        const double2 *EI = p.EI + row0 * C;
        const int *nb = p.nbase + row0 * C;
        const double *rowA = p.dtA + row0 * C, *rowV = p.dtV + row0 * C;
        const double *rowY = p.dtY + row0, *rowYb = p.dtYb + row0;
        const double *ckYA = p.ckYA + (size_t)b * (N + 1);
        const double lz2 = h.logZ * LOG2E;
        const double wb = p.grad_logz ? (double)p.grad_logz[b] : 1.0;
        for (int tg0 = lo; tg0 < hi;) {
            const int tg1 = min(min(hi, (tg0 / J + 1) * J), tg0 + DT_TG);
            const int ng = tg1 - tg0, jt = tg0 / J;
            const double yA0 = ckYA[tg0 == 0 ? 0 : (tg0 - 1) / Delta] + rowY[tg0];
            __syncthreads();  // the previous group is done with the staged rows
            for (int i = tid; i < ((ng + 3) & ~3) * 16 * MT; i += 64 * DXA_W) {
                const int r = i / (16 * MT), o = i % (16 * MT), tt = tg0 + r;
                double a = 0.0;
                if (r < ng && o < C) {
                    const double yA = ckYA[tt == 0 ? 0 : (tt - 1) / Delta] + rowY[tt];
                    a = rowA[(size_t)tt * C + o] * wb * exp2(yA - yA0);
                }
                Arow[r * AS + o] = a;
            }
            if (lane < DT_TG) IEw[lane] = (mine && lane < ng) ? EI[(size_t)(tg0 + lane) * C + c].y : 0.0;
            const int nbt = nb[(size_t)jt * C + c];
            for (int r = lane; r < ng + DXA_K + 3; r += 64) {
                const int s = tg0 + kA + 1 + r;
                double v = 0.0;
                if (mine && s <= L && r < ng + DXA_K) {
                    const int js = s / J;
                    const double yB = s == L ? 0.0 : dt_ytop(p, b, s / Delta, L) + rowYb[s];
                    // all exponents are combined before anything is formed, so that an empty row
                    // stays zero and nothing passes through infinity
                    const double lf = (yA0 + yB) - lz2;
                    const double fl = floor(lf);
                    const int sh = nb[(size_t)js * C + c] - nbt;
                    const double ef = fmin(fmax(fl, -100000.0), 100000.0);
                    v = fmin(ldexp(rowV[(size_t)s * C + c] * exp2(lf - fl), sh + (int)ef), DBL_MAX);
                }
                Vw[r] = v;
            }
            __syncthreads();
            for (int i0 = 0; i0 < ng; i0 += 4) {  // positions i0 .. i0+3 (zero rows beyond the group)
                double A[MT];
#pragma unroll
                for (int m = 0; m < MT; ++m) A[m] = Arow[(i0 + g4) * AS + 16 * m + j];
                const double ie = IEw[i0 + g4];
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    const double bv = ie * Vw[i0 + g4 + 16 * k + j];
#pragma unroll
                    for (int m = 0; m < MT; ++m) acc[m][k] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[m], bv, acc[m][k], 0, 0, 0);
                }
            }
            tg0 = tg1;
        }
    }
    if (!mine) return;
    double *pg = p.partG + (size_t)blockIdx.x * K * CC;
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int k = 0; k < 4; ++k)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int o = 16 * m + 4 * v + g4, kd = kA + 16 * k + j;
                if (o < C && kd < K) {
                    const size_t at = (size_t)kd * CC + (size_t)o * C + c;
                    pg[at] = acc[m][k][v] * p.G3[at];
                }
            }
}
