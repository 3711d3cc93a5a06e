// ---------------------------------------------------------------------------
// Duration-dependent transitions on the matrix cores (included by semicrf.hip after durtrans.inl).
//
// The recurrences of durtrans.inl, four interval tasks per workgroup in lock step, four positions of each at a time:
// sixteen (task, position) pairs are the rows (forward) or columns (backward) of v_mfma_f64_16x16x4 products with the
// table G[k][c'][c], so a table entry fetched from L2 once serves sixteen positions instead of four, and one
// instruction does 1024 multiply-adds.  Scans of the genomic shape (K = 64, C = 24, 4 x 100 000), forward and backward: 4.9
// and 6.3 ms with vector multiply-adds, four positions per table entry and one task per workgroup (durtrans.inl), 1.00 and
// 1.21 ms so, the matrix pipes busy 43 and 48 % of the clocks.  The products wait for the table, so its entries are fetched as far
// ahead as registers allow: three tiles or groups for up to sixteen labels, else one (two, with 25 registers spilled: k_dx_fwd 1003 ->
// 1031 us at the genomic shape).  One ahead against three: 1 x 1293, K = 380, C = 10 forward 627 -> 585, backward 447 -> 435 us;
// 3 x 58043, K = 373, C = 6 forward 640 -> 603; 15 x 11034, K = 39, C = 4 392 -> 380, 341 -> 337.
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
    int ncg;          // label groups of eight (forward tiles), and pairs of inner steps of the forward product
    int mt;           // tiles of sixteen source labels (backward, marginals)
    int ks;           // inner steps of the backward product (four durations each), a multiple of four
    int kr;           // forward ring slots: K + 4, so that all targets of a block are different slots
    int w, m;         // rows of the backward window per label (positions upwards), and its slack
    int xs, ts;       // doubles per task of the forward ring / backward window
    size_t gf, gb, gs; // doubles of the tables in operand order (gs: durations 1 .. 3, forward order by label tiles)
    size_t lds_f, lds_b;
    bool ok;
};
constexpr int DX_CTL = 4 * 4 + 4 * 32;  // ints: block length, first slot / row, rescale and record flags, shifts per label

__host__ __device__ inline DxGeom dx_geometry(const int K, const int C)
{
    DxGeom g;
    g.khp = ((K + 1) / 2 + 3) & ~3;
    g.ncg = (C + 7) / 8;
    g.mt = (C + 15) / 16;
    g.ks = ((K + 3) / 4 + 3) & ~3;
    g.kr = K + DX_MB;
    g.gf = (size_t)g.ncg * g.khp * g.ncg * 128;
    g.gb = (size_t)C * g.ks * g.mt * 64;
    g.gs = (size_t)(DX_MB - 1) * g.mt * g.ncg * 128;
    // tasks 8 doubles (16 LDS banks) apart modulo the banks: the four tasks of an access do not collide
    g.xs = ((g.kr * C + 31) & ~31) + 8;
    // (the rows of the small per-position arrays are an odd number of doubles long: a wave reads them across)
    g.lds_f = ((size_t)DX_TASKS * g.xs + 2 * (size_t)16 * (8 * g.ncg + 1)) * sizeof(double) + DX_CTL * sizeof(int);
    g.m = 32;
    for (;; g.m -= 8) {
        g.w = 4 * g.ks + DX_MB + g.m;
        g.ts = ((g.w * C + 31) & ~31) + 8;
        g.lds_b = ((size_t)DX_TASKS * g.ts + (size_t)(4 + DX_MB - 1) * 16 * (16 * g.mt + 1) + 16 * (size_t)4 * (16 * g.mt + 1) + (size_t)8 * C * 16) * sizeof(double) + DX_CTL * sizeof(int);
        if (g.m == 8 || g.lds_b <= LDS_LIMIT) break;
    }
    g.ok = C <= 32 && g.lds_f <= LDS_LIMIT && g.lds_b <= LDS_LIMIT;
    return g;
}

// The table in the operand order of the two products (zero beyond K and C):
//   forward   [label group][kk][step pair][lane][2]: column j = lane % 16 is duration kk + 1 + (j / 8) khp, label
//             8 group + j % 8; inner index: source label 8 pair + 4 (0, 1) + lane / 16
//   backward  [label][step][lane][mt] (two label tiles) or [label][step pair][lane][2] (one): row: source label
//             16 mt + lane % 16, inner index: duration 4 step + lane / 16 + 1
//   short     [duration - 1][label tile][step pair][lane][2]: durations 1 .. 3, column: label 16 tile + lane % 16, inner
//             index as forward
__global__ __launch_bounds__(NT) void k_dx_tables(Params p)
{
    const int K = p.K, C = p.C, CC = C * C;
    const DxGeom g = dx_geometry(K, C);
    const size_t n0 = (size_t)K * CC, n1 = n0 + g.gf, n2 = n1 + g.gb, n3 = n2 + g.gs;
    const size_t i = (size_t)blockIdx.x * NT + threadIdx.x;
    if (i >= n3) return;
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
        const size_t tile = (q >> 7) / g.ncg;
        const int s = (int)((q >> 7) % g.ncg);
        k = (int)(tile % g.khp) + 1 + (j >> 3) * g.khp;
        c = (int)(tile / g.khp) * 8 + (j & 7);
        o = 8 * s + 4 * u + (lane >> 4);
        dst = p.GF + q;
    } else if (i >= n2) {
        const size_t q = i - n2;
        const int u = (int)(q & 1), lane = (int)(q >> 1) & 63, s = (int)((q >> 7) % g.ncg);
        const int tile = (int)((q >> 7) / g.ncg);
        k = tile / g.mt + 1;
        c = (tile % g.mt) * 16 + (lane & 15);
        o = 8 * s + 4 * u + (lane >> 4);
        dst = p.GS + q;
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
// registers and the ring is touched once per duration.  Waves own whole runs of durations (multiples of four); the last
// three targets of a run belong to the next run too and are added after a barrier: every entry has one writer at a time
// and the order of additions is fixed.
// The block's own four positions are finished by one wave per task (waves 0 .. 3), in registers: its transition
// products are row broadcasts (RowMap), and durations 1 .. 3 inside the block never touch the ring.  fp64 matrix and
// vector instructions share one pipe, so the loop over the tiles carries as few of the latter as possible: the ring entry
// is read before the product it is added to, indices run instead of being computed.
// ---------------------------------------------------------------------------
template <int SF2>
__global__ __launch_bounds__(DX_NT, 2) void k_dx_fwd(Params p, int warm, int tier)
{
    extern __shared__ double lds_raw[];
    constexpr int CT = 8 * SF2, CS = CT + 1;
    constexpr int AHEAD = SF2 <= 2 ? 3 : 1;  // tiles of 2 SF2 products whose table entries are fetched ahead
    using R = RowMap<CT>;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g4 = lane >> 4, j = lane & 15;
    const int K = p.K, C = p.C, CC = C * C, KC = K * C, N = p.N;
    const DxGeom g = dx_geometry(K, C);
    const int KR = g.kr, KHP = g.khp, XS = g.xs;
    double *X = lds_raw;                       // [task][slot][C] partial sums of the positions to come
    double *av = X + DX_TASKS * XS;            // [task][pos][CS] message vectors of the block (zero beyond it)
    double *ieL = av + 16 * CS;                // [task][pos][CS] 1/ES
    int *ctl = (int *)(ieL + 16 * CS);         // per task: block length, slot of its first position, rescale, record
    int *sftL = ctl + 16;                      // [task][32] shift per label at a scaling-block boundary
    const int q = wave & 3;                    // the wave's task; waves 0 .. 3 run the chains
    const bool chain = wave < 4;
    const int c = R::label(lane), gr = R::group(lane);
    const bool cv = c < C, owner = cv && gr == 0;
    bool any = false;  // nothing to do for any of the four tasks: the whole workgroup leaves
    for (int i = 0; i < DX_TASKS; ++i) any = any || dx_task(p, blockIdx.x * DX_TASKS + i, 0, tier).active;
    if (!any) return;
    const DxTask tk = dx_task(p, blockIdx.x * DX_TASKS + q, 0, tier);
    const int L = tk.L, J = tk.J, lo = tk.lo, hi = tk.hi;
    const int s0 = max(lo - dt_warm(p, tk.b, 0, tier, warm), 0);
    const size_t row0 = (size_t)tk.b * (p.T + 1);
    const double2 *EI = p.EI + row0 * C + (cv ? c : 0);
    const int *nb = p.nbase + row0 * C + (cv ? c : 0);
    double *rowA = p.dtA + row0 * C, *rowY = p.dtY + row0;
    const size_t ckstride = (size_t)KC + C;
    double *Xq = X + q * XS, *avq = av + q * 4 * CS, *ieq = ieL + q * 4 * CS;

    // the lane's part of the tables of durations 1 .. 3
    double Ek[DX_MB - 1][R::HC];
#pragma unroll
    for (int k = 0; k < DX_MB - 1; ++k)
#pragma unroll
        for (int i = 0; i < R::HC; ++i) {
            const int o = (lane >> 5) * R::HC + i;
            const bool ok = chain && k < K && cv && o < C;
            const double v = p.G3[ok ? (size_t)k * CC + (size_t)o * C + c : 0];
            Ek[k][i] = ok ? v : 0.0;
        }

    for (int i = tid; i < DX_TASKS * XS + 2 * 16 * CS; i += DX_NT) lds_raw[i] = 0.0;
    double Y = 0.0, Ybase = 0.0, ylast = 0.0;
    int t0 = s0, rb = 0;  // rb: ring slot of t0
    bool done = !tk.active;
    double2 e[DX_MB];
    auto load_ei = [&](const int tb) {
#pragma unroll
        for (int i = 0; i < DX_MB; ++i) {
            e[i] = make_double2(0.0, 0.0);
            if (chain && !done) e[i] = EI[(size_t)min(tb + i, hi) * C];
        }
    };
    load_ei(t0);
    auto nbdelta = [&](const int jb) {  // exponent step of the lane's label at the scaling-block boundary jb
        return (chain && !done && jb >= 1 && (long)jb * J <= (long)L) ? nb[(size_t)jb * C] - nb[(size_t)(jb - 1) * C] : 0;
    };
    int jnx = s0 / J + 1, dnx = nbdelta(jnx);
    lds_barrier();

    // runs of durations: units of four tiles, a contiguous share per wave (at most two label groups)
    const int units = g.ncg * (KHP / 4), per = (units + 7) / 8;
    const int u0 = wave * per, u1 = min(u0 + per, units);

    double2 B0[SF2];  // the first tile's entries: the same in every block
#pragma unroll
    for (int s = 0; s < SF2; ++s) B0[s] = ((const double2 *)p.GF + (size_t)(min(u0, units - 1) * 4) * (SF2 * 64) + lane)[s * 64];

    for (;;) {
        int nbk = 0;
        bool rec = false;
        if (!done) {
            nbk = min(DX_MB, hi - t0 + 1);
            if (t0 <= lo) nbk = min(nbk, lo - t0 + 1);  // the interval's first position ends its block
            nbk = min(nbk, J - (t0 & (J - 1)));         // no scaling-block boundary inside a block
            rec = t0 + nbk - 1 == lo || t0 + nbk > hi;
        }
        if (chain) {
            const bool bd = !done && t0 > s0 && (t0 & (J - 1)) == 0;
            if (bd) {
                const int ex = safe_exponent(R::total(ylast));
                Y += (double)ex;
                if (owner) sftL[q * 32 + c] = dnx - ex;
                ++jnx;
                dnx = nbdelta(jnx);
            }
            if (lane == 0) {
                ctl[q] = nbk;
                ctl[4 + q] = rb;
                ctl[8 + q] = bd;
                ctl[12 + q] = rec;
            }
        }
        lds_barrier();
        if ((ctl[0] | ctl[1] | ctl[2] | ctl[3]) == 0) break;
        const bool anyrec = (ctl[12] | ctl[13] | ctl[14] | ctl[15]) != 0;  // (read here: the next block's are written early)
        if (ctl[8] | ctl[9] | ctl[10] | ctl[11]) {
            if (ctl[8 + q] && (lane & 31) < C) {
                const int sft = sftL[q * 32 + (lane & 31)];
#pragma unroll 4
                for (int r = (wave >> 2) * 2 + (lane >> 5); r < KR; r += 4) {
                    double *x = Xq + r * C + (lane & 31);
                    *x = fmin(ldexp(*x, sft), DBL_MAX);
                }
            }
            lds_barrier();
        }
        // ---- the block's positions, one after the other
        if (chain) {
            double x[DX_MB];
#pragma unroll
            for (int i = 0; i < DX_MB; ++i) x[i] = Xq[dx_wrap(rb + i, KR) * C + (cv ? c : 0)];
#pragma unroll
            for (int i = 0; i < DX_MB; ++i) {
                double a = 0.0;
                if (i < nbk) {  // uniform
                    const int tt = t0 + i;
                    a = cv ? (tt == s0 ? 1.0 : e[i].x * x[i]) : 0.0;
                    ylast = a;
#pragma unroll
                    for (int k = 1; i + k < DX_MB; ++k)
                        if (i + k < nbk) x[i + k] = fma(e[i].y, R::product(a, Ek[k - 1]), x[i + k]);
                    if (owner) Xq[dx_wrap(rb + i, KR) * C + c] = 0.0;  // consumed: free for a later target
                }
                if (owner) {
                    avq[i * CS + c] = a;
                    ieq[i * CS + c] = e[i].y;
                }
            }
            load_ei(t0 + nbk);  // the next block's factors, requested before the long part
        }
        lds_barrier();
        // ---- durations that leave the block
        {
            double A[2 * SF2];
#pragma unroll
            for (int s = 0; s < 2 * SF2; ++s) A[s] = av[((j & 3) * 4 + (j >> 2)) * CS + 4 * s + g4];
            const int nbD = ctl[g4], rbD = ctl[4 + g4];
            double *XD = X + g4 * XS;
            double pend[2][3];  // sums whose targets the next run writes too
            int pslot[2] = {0, 0}, pk[2] = {0, 0};
#pragma unroll
            for (int a = 0; a < 2; ++a) pend[a][0] = pend[a][1] = pend[a][2] = 0.0;
            int u = u0;
#pragma unroll
            for (int sgm = 0; sgm < 2; ++sgm) {
                if (u >= u1) break;  // uniform
                const int cg = u * 4 / KHP, ka = u * 4 - cg * KHP, kb = min(KHP, ka + (u1 - u) * 4);
                const int cl = cg * 8 + (j & 7);
                const double2 *GF = (const double2 *)p.GF + (size_t)(u * 4) * (SF2 * 64) + lane;
                double ier[DX_MB];
#pragma unroll
                for (int i = 0; i < DX_MB; ++i) ier[i] = ieL[(g4 * 4 + i) * CS + cl];
                double w1 = 0.0, w2 = 0.0, w3 = 0.0;
                int k1 = ka + 1 + (j >> 3) * KHP;         // the lane's duration
                int slot = dx_wrap(rbD + k1, KR);
                if (slot >= KR) slot = 0;                  // beyond K + 3: not used
                const int kmax = cl < C ? K + DX_MB - 1 : 0;
                constexpr int NB = AHEAD + 1;  // tiles by turns (runs are multiples of four)
                double2 B[NB][SF2];
#pragma unroll
                for (int h = 0; h < AHEAD; ++h)
#pragma unroll
                    for (int s = 0; s < SF2; ++s) B[h][s] = sgm == 0 && h == 0 ? B0[s] : GF[(h * SF2 + s) * 64];
                const double2 *const GF0 = GF;
                GF += (AHEAD - 1) * (SF2 * 64);
                for (int kk = ka; kk < kb; kk += NB) {
#pragma unroll
                    for (int h = 0; h < NB; ++h) {
                        const bool use = k1 <= kmax;
                        double *xp = XD + slot * C + cl;
                        double xo = 0.0;
                        if (use) xo = *xp;
                        GF += SF2 * 64;
                        // the entries of the tile AHEAD (behind the run's last one the first again: loads under a condition make the
                        // compiler wait for them before the tiles in front; genomic call 3160 -> 3125 us, 64 x 256 positions 252 -> 245, both scans)
                        const double2 *const next = h == 0 || kk + NB < kb ? GF : GF0;
#pragma unroll
                        for (int s = 0; s < SF2; ++s) B[(h + AHEAD) % NB][s] = next[s * 64];
                        dx_d4 D = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                        for (int s = 0; s < SF2; ++s) {
                            D = __builtin_amdgcn_mfma_f64_16x16x4f64(A[2 * s], B[h][s].x, D, 0, 0, 0);
                            D = __builtin_amdgcn_mfma_f64_16x16x4f64(A[2 * s + 1], B[h][s].y, D, 0, 0, 0);
                        }
                        if (NB == 4 ? h < DX_MB - 1 && kk == 0 : kk < DX_MB - 1) {  // uniform: targets inside the block were served above
                            D[0] = k1 >= nbD ? D[0] : 0.0;
                            D[1] = k1 + 1 >= nbD ? D[1] : 0.0;
                            D[2] = k1 + 2 >= nbD ? D[2] : 0.0;
                        }
                        const double w0 = fma(ier[0], D[0], w1);
                        w1 = fma(ier[1], D[1], w2);
                        w2 = fma(ier[2], D[2], w3);
                        w3 = ier[3] * D[3];
                        if (use) *xp = xo + w0;
                        ++k1;
                        ++slot;
                        slot = slot == KR ? 0 : slot;
                    }
                }
                pend[sgm][0] = w1;
                pend[sgm][1] = w2;
                pend[sgm][2] = w3;
                pk[sgm] = k1;      // duration of the first pending target
                pslot[sgm] = cl;
                u += (kb - ka) / 4;
            }
            lds_barrier();
#pragma unroll
            for (int a = 0; a < 2; ++a)
#pragma unroll
                for (int i = 0; i < 3; ++i) {
                    const int k1 = pk[a] + i;
                    if (pk[a] > 0 && pslot[a] < C && k1 <= K + DX_MB - 1) XD[dx_wrap(rbD + k1, KR) * C + pslot[a]] += pend[a][i];
                }
        }
        // The block's rows, by the waves that have nothing to do until the next long part: in the chains they delayed these, and the
        // table entries fetched after them retired after them (launch 1005 -> 970 us at the genomic shape; C = 6, K = 373 600 -> 586).
        // In a block that has rows, a position without one goes to a sink; lanes that own no label store what the owner of theirs, or
        // of label 0, stores.  A block of the warm-up has none and stores nothing: see k_dx_bwd.
        if (nbk > 0 && (t0 + nbk - 1 > lo || t0 == 0)) {  // uniform
            if (!chain) {
#pragma unroll
                for (int i = 0; i < DX_MB; ++i) {
                    const int tt = t0 + i;
                    const bool row = i < nbk && (tt > lo || tt == 0);  // uniform
                    *(row ? rowA + (size_t)tt * C + (cv ? c : 0) : p.sink + tid) = avq[i * CS + (cv ? c : 0)];
                }
            } else {
                const int tt = t0 + lane;
                *(lane < nbk && (tt > lo || tt == 0) ? rowY + tt : p.sink + tid) = Y - Ybase;
            }
        }
        const int tlast = t0 + nbk - 1;
        t0 += nbk;
        rb = dx_wrap(rb + nbk, KR);
        // ---- checkpoints
        if (anyrec) {
            lds_barrier();
            if (rec) {
                auto record = [&](double *ck, double *ckY) {
                    if ((lane & 31) < C) {
                        for (int d = (wave >> 2) * 2 + (lane >> 5); d < K; d += 4)  // position t0 + d
                            ck[(size_t)((t0 + d) % K) * C + (lane & 31)] = Xq[dx_wrap(rb + d, KR) * C + (lane & 31)];
                    }
                    if (chain && owner) ck[KC + c] = ylast;
                    if (chain && lane == 0) *ckY = Y;
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
            lds_barrier();  // the ring is read by both waves of a task before either goes on
        }
    }
}

// ---------------------------------------------------------------------------
// Backward ("pull"): for every label c a product [source labels] x [durations] . [durations] x [sixteen (task,
// position) columns] of the table with the window of v; IE_t(c) is applied to its result, which is then added up over
// the labels (b_t) and, weighted with a_t, over the source labels (mass of the segments that start at t).  A wave takes the
// labels wave, wave + 8, ...; the waves' sums for b meet in LDS.  The window lies label by label along the positions, so
// that the product's operand comes with immediate offsets; it slides downwards and is moved back every m positions.
// Inside the block, one wave per task (0 .. 3) finishes the positions by row broadcasts, while the other (4 .. 7) forms what
// durations 1 .. 3 add to the mass that starts at a position; it then writes the block's rows.
// Bound by the products (of 26 thousand clocks per block at the genomic shape their matrix instructions alone take 13) and by what
// lies between two of them: the tables of those sums held in registers that only the chain waves need otherwise, the sums
// formed beside the chains, and rows stored unconditionally took the launch from 1278 to 1190 us (K = 39, C = 6: 672 -> 650).
// ---------------------------------------------------------------------------
template <int MT, int SF2, bool BEHIND>
__global__ __launch_bounds__(DX_NT, 2) void k_dx_bwd(Params p, int warm, int tier)
{
    extern __shared__ double lds_raw[];
    constexpr int CT = 8 * SF2;
    using R = RowMap<CT>;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g4 = lane >> 4, j = lane & 15;
    const int K = p.K, C = p.C, CC = C * C, KC = K * C, N = p.N;
    const DxGeom g = dx_geometry(K, C);
    const int W = g.w, M = g.m, TS = g.ts, KS = g.ks;
    constexpr int CPB = 16 * MT + 1;
    double *V = lds_raw;                       // [task][C][W] v of the positions from the block upwards
    double *avL = V + DX_TASKS * TS;           // [task][pos][CPB] a_t
    double *ieL = avL + 16 * CPB;              // [task][pos][CPB] 1/ES
    double *esL = ieL + 16 * CPB;              // [task][pos][CPB] ES
    double *bL = esL + 16 * CPB;               // [task][pos][CPB] b_t
    double *wL = bL + 16 * CPB;                 // [k][task][pos][CPB] sum over the source labels of a_t G[k], k = 1 .. 3
    double *oL = wL + 3 * 16 * CPB;            // [g4][task][pos][CPB] segments that start at t and leave the block, in four parts
    double *bp = oL + 4 * 16 * CPB;            // [wave][C][16] the waves' shares of b
    int *ctl = (int *)(bp + 8 * C * 16);       // per task: block length, row of its first position, rescale, record
    int *sftL = ctl + 16;                      // [task][32] shift per label at a scaling-block boundary
    const int q = wave & 3;
    const bool chain = wave < 4;
    const int c = R::label(lane), gr = R::group(lane);
    const bool cv = c < C, owner = cv && gr == 0;
    const int cc0 = cv ? c : 0;
    bool any = false;  // nothing to do for any of the four tasks: the whole workgroup leaves
    for (int i = 0; i < DX_TASKS; ++i) any = any || dx_task(p, blockIdx.x * DX_TASKS + i, 1, tier).active;
    if (!any) return;
    const DxTask tk = dx_task(p, blockIdx.x * DX_TASKS + q, 1, tier);
    const int L = tk.L, J = tk.J, lo = tk.lo, hi = tk.hi;
    const int s1 = min(hi + dt_warm(p, tk.b, 1, tier, warm), L);
    const size_t row0 = (size_t)tk.b * (p.T + 1);
    const double2 *EI = p.EI + row0 * C + cc0;
    const int *nb = p.nbase + row0 * C + cc0;
    const double *rowA = p.dtA + row0 * C + cc0;
    double *rowV = p.dtV + row0 * C, *rowD = p.dtD + row0 * C, *rowYb = p.dtYb + row0;
    const size_t ckstride = (size_t)KC + C;
    double *Vq = V + q * TS;
    const int qo = q * 4 * CPB;

    for (int i = tid; i < DX_TASKS * TS + 4 * 16 * CPB; i += DX_NT) lds_raw[i] = 0.0;
    // the lane's part of the tables of durations 1 .. 3: chain waves the contraction over the label, the others the operands of
    // their two tiles of sum_c' a_t(c') G[k][c'][c] (below)
    constexpr int NSH = (DX_MB - 1) * MT;  // tiles (duration - 1, label tile)
    double Ek[(DX_MB - 1) * R::HC];
    if (chain) {
#pragma unroll
        for (int k = 0; k < DX_MB - 1; ++k)
#pragma unroll
            for (int i = 0; i < R::HC; ++i) {
                const int o = (lane >> 5) * R::HC + i;
                const bool ok = k < K && cv && o < C;
                const double v = p.G3[ok ? (size_t)k * CC + (size_t)c * C + o : 0];
                Ek[k * R::HC + i] = ok ? v : 0.0;
            }
    } else {
        static_assert(4 * SF2 <= (DX_MB - 1) * R::HC && NSH <= 8, "two tiles per wave, in the chain waves' registers");
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int s = 0; s < SF2; ++s) {
                const double2 gs = ((const double2 *)p.GS)[((size_t)min(q + 4 * u, NSH - 1) * SF2 + s) * 64 + lane];
                Ek[(u * SF2 + s) * 2] = gs.x;
                Ek[(u * SF2 + s) * 2 + 1] = gs.y;
            }
    }
    lds_barrier();
    bool done = !tk.active;
    double Yb = 0.0, Ytop = 0.0, blast = 0.0;
    int t0 = s1 - 1, r0 = M + DX_MB - 1;  // window row of t0
    // a sequence that ends at s1 (exactly so when s1 = L): b = 1, v = ES; scale reference: a single 1
    if (!done && chain) {
        blast = c == 0 ? 1.0 : 0.0;
        const double v = EI[(size_t)s1 * C].x;
        if (owner) {
            Vq[c * W + r0 + 1] = v;
            if (s1 == L) rowV[(size_t)L * C + c] = v;
        }
        if (s1 == L && lane == 0) rowYb[L] = 0.0;
    }
    double2 e[DX_MB];
    double a[DX_MB];
    auto load_rows = [&](const int tb) {
#pragma unroll
        for (int i = 0; i < DX_MB; ++i) {
            e[i] = make_double2(0.0, 0.0);
            a[i] = 0.0;
            if (!done) {
                const size_t o = (size_t)max(tb - i, lo) * C;
                e[i] = EI[o];
                if (!chain) a[i] = rowA[o];
            }
        }
    };
    load_rows(t0);
    auto nbdelta = [&](const int jb) {
        return (chain && !done && jb >= 1 && (long)jb * J <= (long)L) ? nb[(size_t)jb * C] - nb[(size_t)(jb - 1) * C] : 0;
    };
    int jnx = s1 / J, dnx = nbdelta(jnx);

    for (;;) {
        int nbk = 0;
        bool rec = false;
        if (!done) {
            nbk = min(DX_MB, t0 - lo + 1);
            if (t0 >= hi) nbk = min(nbk, t0 - hi + 1);     // the interval's upper end ends its block
            nbk = min(nbk, (t0 & (J - 1)) + 1);             // no scaling-block boundary inside a block
            rec = t0 - nbk + 1 == hi || t0 - nbk + 1 == lo;
        }
        const bool bd = !done && ((t0 + 1) & (J - 1)) == 0;
        if (chain) {
            if (bd) {
                const int ex = safe_exponent(R::total(blast));
                Yb += (double)ex;
                if (owner) sftL[q * 32 + c] = dnx - ex;
                --jnx;
                dnx = nbdelta(jnx);
            }
            if (lane == 0) {
                ctl[q] = nbk;
                ctl[4 + q] = r0 < DX_MB - 1 ? M + DX_MB - 1 : r0;
                ctl[8 + q] = bd || r0 < DX_MB - 1;
                ctl[12 + q] = rec;
            }
        }
        lds_barrier();
        if ((ctl[0] | ctl[1] | ctl[2] | ctl[3]) == 0) break;
        // window rows: each wave of a task looks after its half of the labels
        const int lh = (C + 1) / 2, c0 = chain ? 0 : lh, c1 = chain ? lh : C;
        if (ctl[8] | ctl[9] | ctl[10] | ctl[11]) {
            if (r0 < DX_MB - 1) {
                // move the K live rows back up, four labels by sixteen rows at a time
                const int sh = M + DX_MB - 1 - r0;
                for (int d0 = (K - 1) & ~15; d0 >= 0; d0 -= 16) {
                    double v[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int cl = c0 + 4 * u + g4, d = d0 + j;
                        v[u] = (cl < c1 && d < K) ? Vq[cl * W + r0 + 1 + d] : 0.0;
                    }
                    lds_wave_fence();
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const int cl = c0 + 4 * u + g4, d = d0 + j;
                        if (cl < c1 && d < K) Vq[cl * W + r0 + 1 + d + sh] = v[u];
                    }
                    lds_wave_fence();
                }
                r0 += sh;
            }
            if (bd) {
                for (int cl = c0 + g4; cl < c1; cl += 4) {
                    const int sft = sftL[q * 32 + cl];
#pragma unroll 4
                    for (int d = j; d < K; d += 16) {
                        double *x = Vq + cl * W + r0 + 1 + d;
                        *x = fmin(ldexp(*x, sft), DBL_MAX);
                    }
                }
            }
        }
        // rows of the block (zeros beyond it) and its window rows (zeros until they are known); the next rows requested
        for (int cl = c0 + g4; cl < c1; cl += 4)
            if (j < DX_MB && !done) Vq[cl * W + r0 - j] = 0.0;
        if (owner) {
#pragma unroll
            for (int i = 0; i < DX_MB; ++i) {
                if (chain) {
                    esL[qo + i * CPB + c] = i < nbk ? e[i].x : 0.0;
                    ieL[qo + i * CPB + c] = i < nbk ? e[i].y : 0.0;
                } else {
                    avL[qo + i * CPB + c] = i < nbk ? a[i] : 0.0;
                }
            }
        }
        lds_barrier();
        // ---- durations that reach beyond the block
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
            const double *Vn = V + tn * TS + (ctl[4 + tn] - pn + g4 + 1);
            // table entries: one double2 per lane and step (two label tiles) or pair of steps (one), four steps at a
            // time, AHEAD groups ahead (across labels).  BEHIND: always fetched, behind the last group one that is there already, as a
            // fetch under a condition makes the compiler wait for it before the group in front.
            constexpr int LG = 2 * MT;
            constexpr int NBUF = MT == 1 ? 4 : 2, AHEAD = NBUF - 1;
            double2 Gg[NBUF][LG];
            double bg[NBUF][4];
            auto fetch = [&](const int cc, const int s, double2 (&G)[LG], double (&b)[4]) {
                const double2 *GB = (const double2 *)p.GB + ((size_t)min(cc, C - 1) * KS + s) * (MT * 32) + lane;
                const double *Vc = Vn + min(cc, C - 1) * W + 4 * s;
#pragma unroll
                for (int u = 0; u < LG; ++u) G[u] = GB[u * 64];
#pragma unroll
                for (int u = 0; u < 4; ++u) b[u] = Vc[4 * u];
            };
            dx_d4 D[MT];
            auto group = [&](const double2 (&G)[LG], const double (&b)[4]) {
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (MT == 2) {
                        D[0] = __builtin_amdgcn_mfma_f64_16x16x4f64(G[u % LG].x, b[u], D[0], 0, 0, 0);
                        D[MT - 1] = __builtin_amdgcn_mfma_f64_16x16x4f64(G[u % LG].y, b[u], D[MT - 1], 0, 0, 0);
                    } else {
                        D[0] = __builtin_amdgcn_mfma_f64_16x16x4f64((u & 1) ? G[u / 2].y : G[u / 2].x, b[u], D[0], 0, 0, 0);
                    }
                }
            };
            auto finish = [&](const int cc) {
                const double ie = ieL[(tn * 4 + pn) * CPB + cc];
                double o = 0.0;
#pragma unroll
                for (int m = 0; m < MT; ++m)
#pragma unroll
                    for (int v = 0; v < 4; ++v) {
                        bacc[m][v] = fma(ie, D[m][v], bacc[m][v]);
                        o = fma(An[4 * m + v], D[m][v], o);
                    }
                oL[((g4 * 4 + tn) * 4 + pn) * CPB + cc] = o;
            };
            if (wave < C) {
                // groups of all the wave's labels in one sequence, NBUF per turn
                const int ng = KS / 4, total = ((C - wave + 7) / 8) * ng;
                int cc = wave, gq = 0;        // group being multiplied
                int ccn = wave, gn = 0;       // group being fetched
                auto next = [&](int &cx, int &gx) {
                    if (++gx == ng) {
                        gx = 0;
                        cx += 8;
                    }
                };
#pragma unroll
                for (int h = 0; h < AHEAD; ++h) {
                    if (BEHIND || h == 0 || h < total) fetch(ccn, 4 * gn, Gg[h], bg[h]);
                    next(ccn, gn);
                }
                for (int i = 0; i < total; i += NBUF) {
#pragma unroll
                    for (int h = 0; h < NBUF; ++h) {
                        if (i + h < total) {  // uniform
                            if (BEHIND || i + h + AHEAD < total) fetch(ccn, 4 * gn, Gg[(h + AHEAD) % NBUF], bg[(h + AHEAD) % NBUF]);
                            next(ccn, gn);
                            if (gq == 0) {
#pragma unroll
                                for (int m = 0; m < MT; ++m) D[m] = dx_d4{0.0, 0.0, 0.0, 0.0};
                            }
                            group(Gg[h], bg[h]);
                            if (gq == ng - 1) finish(cc);
                            next(cc, gq);
                        }
                    }
                }
            }
#pragma unroll
            for (int m = 0; m < MT; ++m)
#pragma unroll
                for (int v = 0; v < 4; ++v) {
                    const int r = 16 * m + 4 * v + g4;
                    if (r < C) bp[(wave * C + r) * 16 + j] = bacc[m][v];
                }
        }
        if (chain && lane < nbk && t0 - lane < hi) rowYb[t0 - lane] = Yb - Ytop;
        load_rows(t0 - nbk);  // the next block's, with the serial part to arrive
        lds_barrier();
        if ((tid >> 4) < C) {  // 512 threads: source label, column
            double b = 0.0;
#pragma unroll
            for (int w = 0; w < 8; ++w) b += bp[(w * C + (tid >> 4)) * 16 + j];
            bL[((j & 3) * 4 + (j >> 2)) * CPB + (tid >> 4)] = b;
        }
        lds_barrier();
        if (chain) {
            // ---- finish the positions one after the other
            double bf[DX_MB], ie[DX_MB], es[DX_MB], v[DX_MB];
#pragma unroll
            for (int i = 0; i < DX_MB; ++i) {
                bf[i] = bL[qo + i * CPB + cc0];
                ie[i] = ieL[qo + i * CPB + cc0];
                es[i] = esL[qo + i * CPB + cc0];
            }
#pragma unroll
            for (int i = 0; i < DX_MB; ++i) {
                v[i] = 0.0;
                if (i < nbk) {  // uniform
                    double b = bf[i];
#pragma unroll
                    for (int k = 1; k <= i; ++k)  // ends at position i - k of the block, finished before
                        b += R::product(cv ? ie[i] * v[i - k] : 0.0, Ek + (k - 1) * R::HC);
                    b = cv ? b : 0.0;
                    v[i] = b * es[i];
                    blast = b;
                    if (owner) {
                        bL[qo + i * CPB + c] = b;
                        Vq[c * W + r0 - i] = v[i];
                    }
                }
            }
        } else {
            // meanwhile, sums over the source labels of a_t G[k], k = 1 .. 3, for what durations inside the block add to the
            // mass that starts at a position: one product of the sixteen rows per (duration, label tile)
            double ar[2 * SF2];
#pragma unroll
            for (int s = 0; s < 2 * SF2; ++s) ar[s] = avL[((j & 3) * 4 + (j >> 2)) * CPB + 4 * s + g4];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                const int tile = q + 4 * u;
                if (tile >= NSH) break;  // uniform
                dx_d4 w = {0.0, 0.0, 0.0, 0.0};
#pragma unroll
                for (int s = 0; s < 2 * SF2; ++s) w = __builtin_amdgcn_mfma_f64_16x16x4f64(ar[s], Ek[u * 2 * SF2 + s], w, 0, 0, 0);
#pragma unroll
                for (int v = 0; v < 4; ++v)  // row 4 v + g4: task g4, position v
                    wL[(((tile / MT) * 4 + g4) * 4 + v) * CPB + (tile % MT) * 16 + j] = w[v];
            }
        }
        lds_barrier();
        // ---- the block's rows.  A position without one goes to a sink: the number of stores behind the next block's loads is then
        // known, and waiting for those is not waiting for these.  Lanes that own no label store what the owner of theirs, or of label 0,
        // stores.  A block of the warm-up has no rows and forms none: with sums and stores to the sink there too, long warm-ups (few labels,
        // short segments) took longer than without any of this; a call, before | with them | so, us: 16 x 2000, K = 8, C = 4
        // 618 | 632 | 597; C = 1 586 | 609 | 572; K = 16, C = 5 841 | 861 | 802; K = 16, C = 16 242 | 225 | 221; 2 x 1704, K = 77, C = 4
        // 258 | 260 | 251; 4 x 100 000, K = 64, C = 24 3307 | 3161 | 3164.
        if (!chain && nbk > 0 && t0 - nbk + 1 < hi) {  // uniform
            constexpr int OS = 16 * CPB;
            const double *vr = Vq + cc0 * W + r0;
            double v[DX_MB];
#pragma unroll
            for (int i = 0; i < DX_MB; ++i) v[i] = vr[-i];
#pragma unroll
            for (int i = 0; i < DX_MB; ++i) {
                const int tt = t0 - i, o = qo + i * CPB + cc0;
                double out = (oL[o] + oL[o + OS]) + (oL[o + 2 * OS] + oL[o + 3 * OS]);
#pragma unroll
                for (int k = 1; k <= i; ++k) out = fma(wL[(k - 1) * OS + o], v[i - k], out);
                const bool row = i < nbk && tt < hi;  // uniform
                const size_t at = (size_t)tt * C + cc0;
                *(row ? rowV + at : p.sink + tid) = v[i];
                *(row ? rowD + at : p.sink + tid) = out * ieL[o] - (tt >= 1 ? avL[o] * bL[o] : 0.0);
            }
        }
        const int tlast = t0 - nbk + 1, rlast = r0 - nbk + 1;
        t0 -= nbk;
        r0 -= nbk;
        if (rec) {
            // (window rows are not written again before the next block's first barrier)
            auto record = [&](double *ck, double *ckY) {
                for (int cl = wave >> 2; cl < C; cl += 2)
                    for (int d = lane; d < K; d += 64)  // position tlast + d
                        ck[(size_t)((tlast + d) % K) * C + cl] = Vq[cl * W + rlast + d];
                if (chain && owner) ck[KC + c] = blast;
                if (chain && lane == 0) *ckY = Yb;
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
// Running emission-gradient sums per interval, of both families' scans (for fin_seq_body): one workgroup per (sequence,
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
    // scale of the forward rows: the interval's first position is the last of the task before (a look-up with a division per
    // position and lane cost a sixth of the launch: 75.8 -> 63.5 us at the genomic shape)
    const double yin = ckYA[jv], yfirst = ckYA[max(jv - 1, 0)];
    // absolute scales of the stored rows for k_dx_acc, split into a factor in [1, 2) and an exponent:
    // 2^YA(t) / Z and 2^YB(t)
    if (p.dtMA) {
        for (int tt = lo + (int)threadIdx.x; tt < hi || (tt == L && hi == L); tt += NT) {
            const double yb = tt == L ? 0.0 : ytop + rowYb[tt];
            const double ya = tt == L ? 0.0 : (tt == lo ? yfirst : yin) + rowY[tt] - logZ * LOG2E;
            const double fa = floor(ya), fb = floor(yb);
            p.dtMA[row0 + tt] = exp2(ya - fa);
            p.dtMB[row0 + tt] = exp2(yb - fb);
            p.dtE[row0 + tt] = make_int2(whole_exponent(fa), whole_exponent(fb));
        }
    }
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
                y[i] = (tt == lo ? yfirst : yin) + rowY[tt] + ytop + rowYb[tt];
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
// Work is handed out in pieces of at most this many positions of an interval: whole intervals would leave the
// persistent workgroups with unequal shares.
constexpr int DXA_PIECE = 64;
__host__ __device__ constexpr int dxa_pieces(int Delta) { return (Delta + DXA_PIECE - 1) / DXA_PIECE; }
// LDS doubles: a rows, per wave the label's 1/ES and v rows
__host__ __device__ constexpr size_t dxa_lds_doubles(int mt) { return (size_t)DT_TG * (16 * mt + 1) + (size_t)DXA_W * (DT_TG + DXA_VR); }

// A group of positions (at most DT_TG, inside one scaling block) goes through LDS; the rows of the next group are
// requested before the products of this one.  Scales: k_dx_emis has left them as factor and exponent, all exponents
// are combined before anything is formed, so that an empty row stays zero and nothing passes through infinity.
template <int MT, int KT>  // KT: duration tiles of sixteen with anything in them (four where K > 64)
__global__ __launch_bounds__(64 * DXA_W, 4) void k_dx_acc(Params p)
{
    extern __shared__ double lds_raw[];
    constexpr int AS = 16 * MT + 1;
    constexpr int AE = DT_TG * 16 * MT / (64 * DXA_W);  // a elements per thread
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int g4 = lane >> 4, j = lane & 15;
    const int K = p.K, C = p.C, CC = C * C, N = p.N, Delta = p.Delta;
    const int kgs = (K + DXA_K - 1) / DXA_K;
    const int item = blockIdx.y * DXA_W + wave;
    const bool mine = item < C * kgs;
    const int c = mine ? item / kgs : 0, kA = mine ? (item % kgs) * DXA_K : 0;  // durations kA + 1 .. kA + 64
    double *Arow = lds_raw;                            // [DT_TG][AS]  a_t(c') w_b 2^YA(t) / Z in the group's scale
    double *IEw = Arow + DT_TG * AS + wave * (DT_TG + DXA_VR);  // [DT_TG] 1/ES of the wave's label
    double *Vw = IEw + DT_TG;                          // [DXA_VR] v of the wave's label from position group + kA + 1 on
    dx_d4 acc[MT][KT];
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int k = 0; k < KT; ++k) acc[m][k] = dx_d4{0.0, 0.0, 0.0, 0.0};

    const int pieces = dxa_pieces(Delta), nitem = p.B * N * pieces;
    int it = blockIdx.x, tg0 = 0, tg1 = 0, hi = 0, L = 0, Jl = 0;
    size_t row0 = 0;
    double wb = 1.0;
    // the next group: false when there is none
    auto advance = [&]() {
        tg0 = tg1;
        while (tg0 >= hi) {
            if (it >= nitem) return false;
            const int task = it / pieces, b = task / N, chunk = task % N;
            const int lo = chunk * Delta + (it % pieces) * DXA_PIECE;
            const SeqHdr h = p.hdr[b];
            L = h.L;
            Jl = 31 - __clz(h.J);
            hi = min(min(lo + DXA_PIECE, (chunk + 1) * Delta), L);
            tg0 = lo;
            row0 = (size_t)b * (p.T + 1);
            wb = p.grad_logz ? (double)p.grad_logz[b] : 1.0;
            it += gridDim.x;
        }
        tg1 = min(min(hi, ((tg0 >> Jl) + 1) << Jl), tg0 + DT_TG);
        return true;
    };
    double ar[AE], am[AE], vr[2], vm[2], ie = 0.0;
    int ae[AE], vs[2], nbt = 0, eA0 = 0;
    auto request = [&]() {
        const int *nb = p.nbase + row0 * C + c;
        nbt = nb[(size_t)(tg0 >> Jl) * C];
        eA0 = p.dtE[row0 + tg0].x;
#pragma unroll
        for (int u = 0; u < AE; ++u) {
            const int i = tid + u * 64 * DXA_W, r = i / (16 * MT), o = i % (16 * MT);
            const size_t t = row0 + min(tg0 + r, tg1 - 1);
            ar[u] = p.dtA[t * C + min(o, C - 1)];
            am[u] = p.dtMA[t];
            ae[u] = p.dtE[t].x;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int s = min(tg0 + kA + 1 + lane + 64 * u, L);
            vr[u] = p.dtV[(row0 + s) * C + c];
            vm[u] = p.dtMB[row0 + s];
            vs[u] = p.dtE[row0 + s].y + nb[(size_t)(s >> Jl) * C];
        }
        ie = p.EI[(row0 + min(tg0 + (lane & 31), L)) * C + c].y;
    };
    bool more = advance();
    if (more) request();
    while (more) {  // uniform
        const int ng = tg1 - tg0;
        __syncthreads();  // the previous group is done with the staged rows
#pragma unroll
        for (int u = 0; u < AE; ++u) {
            const int i = tid + u * 64 * DXA_W, r = i / (16 * MT), o = i % (16 * MT);
            Arow[r * AS + o] = (r < ng && o < C) ? ldexp(ar[u] * wb * am[u], ae[u] - eA0) : 0.0;
        }
        if (lane < DT_TG) IEw[lane] = (mine && lane < ng) ? ie : 0.0;
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int r = lane + 64 * u, s = tg0 + kA + 1 + r;
            double v = 0.0;
            if (mine && s <= L && r < ng + DXA_K && kA + r < ng + K) v = fmin(ldexp(vr[u] * vm[u], vs[u] + eA0 - nbt), DBL_MAX);
            if (r < DXA_VR) Vw[r] = v;
        }
        __syncthreads();
        more = advance();
        if (more) request();
        for (int i0 = 0; i0 < ng; i0 += 4) {  // positions i0 .. i0+3 (zero rows beyond the group)
            double A[MT];
#pragma unroll
            for (int m = 0; m < MT; ++m) A[m] = Arow[(i0 + g4) * AS + 16 * m + j];
            const double iet = IEw[i0 + g4];
            double bv[KT];
#pragma unroll
            for (int k = 0; k < KT; ++k) bv[k] = iet * Vw[i0 + g4 + 16 * k + j];
#pragma unroll
            for (int k = 0; k < KT; ++k)
#pragma unroll
                for (int m = 0; m < MT; ++m) acc[m][k] = __builtin_amdgcn_mfma_f64_16x16x4f64(A[m], bv[k], acc[m][k], 0, 0, 0);
        }
    }
    if (!mine) return;
    // Partial tables as [source label][label][duration], so that sixteen lanes store a line, and without the factor G, which
    // k_dt_fin applies once: with a load of it before each of 32 stores of single doubles a genomic call takes 3125 us, so 3081.
    double *pg = p.partG + (size_t)blockIdx.x * K * CC;
    const int kd = kA + j;
    int first = (g4 * C + c) * K + kd;
    asm volatile("" : "+v"(first));  // (formed here: ahead of the loop it and what is added to it would cost registers there)
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int k = 0; k < KT; ++k)
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const int o = 16 * m + 4 * v;
                if (o + g4 < C && 16 * k < K - kd) pg[first + (o * C * K + 16 * k)] = acc[m][k][v];
            }
}
