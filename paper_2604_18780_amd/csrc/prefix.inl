// Eq. 1 and Eq. 2: tables, per-sequence baseline, centred prefix sums, block exponents and the (ES, 1/ES) pairs.
// Included by semicrf.hip inside its anonymous namespace (after common.h); not a translation unit of its own.

// ---------------------------------------------------------------------------
// exp(dur), exp(trans) in fp64 and the maxima that bound per-step growth.  The table entries are spread over
// p.ntab workgroups (TAB_ITEMS entries each); every one leaves the two maxima of its share.
// ---------------------------------------------------------------------------
constexpr int TAB_ITEMS = 8 * NT;
inline int tables_blocks(const Params &p)
{
    if (!p.dur || (!p.trans && !p.trans3)) return 1;
    const size_t n = (size_t)p.K * p.C + (size_t)p.C * p.C * (p.trans3 ? (size_t)p.K : 1);
    const size_t w = (n + TAB_ITEMS - 1) / TAB_ITEMS;
    return (int)(w < (size_t)TAB_BLOCKS_MAX ? w : (size_t)TAB_BLOCKS_MAX);
}

__device__ __forceinline__ void tables_body(const Params &p, const int blk)
{
    __shared__ double red[2 * (NT / 64)];
    const int tid = threadIdx.x;
    const int KC = p.K * p.C, CC = p.C * p.C;
    if (!p.dur || (!p.trans && !p.trans3)) {  // prefix sums only: growth is bounded by the emissions alone
        if (tid < 2) p.tabmax[tid] = 0.0;
        return;
    }
    double mxd = -DBL_MAX, mxt = -DBL_MAX;
    const int first = blk * NT + tid, step = p.ntab * NT;
    if (p.trans3) {  // one transition matrix per duration: only the maxima are needed here
        for (int i = first; i < KC; i += step) mxd = fmax(mxd, (double)p.dur[i]);
#pragma unroll 8
        for (int i = first; i < p.K * CC; i += step) mxt = fmax(mxt, (double)p.trans3[i]);
    } else {
#pragma unroll 4
        for (int i = first; i < KC + CC; i += step) {
            const bool isd = i < KC;
            const double v = (double)(isd ? p.dur[i] : p.trans[i - KC]);
            (isd ? p.W : p.Etr - KC)[i] = exp(v);
            mxd = fmax(mxd, isd ? v : -DBL_MAX);
            mxt = fmax(mxt, isd ? -DBL_MAX : v);
        }
    }
    // maxima: inside each wave, then over the waves (any order)
    mxd = wave_max(mxd);
    mxt = wave_max(mxt);
    if ((tid & 63) == 0) {
        red[tid >> 6] = mxd;
        red[NT / 64 + (tid >> 6)] = mxt;
    }
    __syncthreads();
    if (tid < 2) {
        double m = red[tid * (NT / 64)];
        for (int i = 1; i < NT / 64; ++i) m = fmax(m, red[tid * (NT / 64) + i]);
        p.tabmax[2 * blk + tid] = m;
    }
}

// ---------------------------------------------------------------------------
// Eq. 1, stage 1: per-chunk column sums (fp64) and what bounds the growth inside a scaling block.  grid (NCH, B).
// An item is (32 positions, label), labels fastest: 32 loads in flight, and the running sum along the positions gives the
// furthest that the prefix sum of a label gets from its value at the first of them (JMAX = 32 is the longest block; a
// shorter one lies inside such a group).  The baseline nu is not known yet: it moves that by at most 31 |nu|.
// Bound by the latency of its loads: 9.3 us with rows dealt out over the threads (eight loads in flight, no excursions),
// 7.0 us so (B = 32, T = 2000, C = 64, bfloat16); 11.8 us both ways at 4 x 100 000 x 24, 27.0 and 26.8 us with projections,
// which are read 16 bytes at a time where they are aligned (30.2 us one by one).
// ---------------------------------------------------------------------------
constexpr int COL_NG = PREP_CH / JMAX;

// the smallest float that is not below x >= 0 (two bounds of a chunk in the place of one double)
__device__ __forceinline__ float float_above(const double x)
{
    const float q = (float)x;
    return (double)q < x ? nextafterf(q, INFINITY) : q;
}

// The emissions of one item, n of them (o: offset of the first), zeros beyond: their sum, and into mx and ex the largest and the
// largest excursion.
template <int ET>
__device__ __forceinline__ double col_item(const Params &p, const size_t o, const int n, double &mx, double &ex)
{
    const int C = p.C;
    double f[JMAX];
    if (n == JMAX) {
#pragma unroll
        for (int i = 0; i < JMAX; ++i) f[i] = emis_at<ET>(p, o + (unsigned)(i * C));
    } else if (n > 0) {  // the sequence's last: rows beyond its end are replaced by its last one, so that nothing waits in a branch
#pragma unroll
        for (int i = 0; i < JMAX; ++i) {
            const double v = emis_at<ET>(p, o + (unsigned)(min(i, n - 1) * C));
            f[i] = i < n ? v : 0.0;
        }
    } else {
#pragma unroll
        for (int i = 0; i < JMAX; ++i) f[i] = 0.0;
    }
    double s = 0.0;
#pragma unroll
    for (int i = 0; i < JMAX; ++i) {
        mx = fmax(mx, fabs(f[i]));
        s += f[i];
        if (i < JMAX - 1) ex = fmax(ex, fabs(s));
    }
    return s;
}

// The largest entry of rows u0 .. u1-1 of a projection (0 without one), this thread's share.
__device__ __forceinline__ float rows_absmax(const Params &p, const float *a, const int b, const int u0, const int u1)
{
    float m = 0.f;
    if (!a || u1 <= u0) return m;
    a += ((size_t)b * p.T + u0) * p.C;  // one after the other
    const int n = (u1 - u0) * p.C, n4 = ((uintptr_t)a & 15) == 0 ? n / 4 : 0;
#pragma unroll 4
    for (int i = threadIdx.x; i < n4; i += NT) {
        const float4 v = ((const float4 *)a)[i];
        m = fmaxf(fmaxf(fmaxf(m, fabsf(v.x)), fmaxf(fabsf(v.y), fabsf(v.z))), fabsf(v.w));
    }
#pragma unroll 4
    for (int i = 4 * n4 + threadIdx.x; i < n; i += NT) m = fmaxf(m, fabsf(a[i]));
    return m;
}

template <int ET>
__device__ __forceinline__ void colsum_body(const Params &p, const int b, const int ch)
{
    __shared__ double red[COL_NG * 256];  // C <= 256
    __shared__ double redm[NT / 64], redx[NT / 64];
    __shared__ float reds[NT / 64], rede[NT / 64], redc[NT / 64];
    const int tid = threadIdx.x;
    const int C = p.C, L = seq_len(p, b);
    const int u0 = ch * PREP_CH;
    const int u1 = min(u0 + PREP_CH, L);
    const double smp = p.warm_model ? warm_load<ET>(p, b, ch, L) : 0.0;
    double mx = 0.0, ex = 0.0;
    for (int it = tid; it < COL_NG * C; it += NT) {
        const int t0 = u0 + it / C * JMAX, n = min(L - t0, JMAX);
        red[it] = col_item<ET>(p, ((size_t)b * p.T + t0) * C + it % C, n, mx, ex);
    }
    // the boundary projections move a message like an emission does: their maxima are added
    float mps = rows_absmax(p, p.proj_start, b, u0, u1), mpe = rows_absmax(p, p.proj_end, b, u0, u1);
    // the maxima first inside each wave (a maximum does not care for order)
    mx = wave_max(mx);
    ex = wave_max(ex);
    if (p.proj_start) mps = (float)wave_max((double)mps);
    if (p.proj_end) mpe = (float)wave_max((double)mpe);
    const float con = p.warm_model ? warm_sample(p, ch, L, smp) : 0.f;
    if ((tid & 63) == 0) {
        redc[tid >> 6] = con;
        redm[tid >> 6] = mx;
        redx[tid >> 6] = ex;
        reds[tid >> 6] = mps;
        rede[tid >> 6] = mpe;
    }
    __syncthreads();
    if (tid < C) {
        double s = 0.0;
#pragma unroll
        for (int i = 0; i < COL_NG; ++i) s += red[i * C + tid];
        p.chsum[((size_t)b * p.NCH + ch) * C + tid] = s;
    }
    if (tid == 0) {
        for (int i = 1; i < NT / 64; ++i) {
            mx = fmax(mx, redm[i]);
            ex = fmax(ex, redx[i]);
            mps = fmaxf(mps, reds[i]);
            mpe = fmaxf(mpe, rede[i]);
        }
        p.chmax[(size_t)b * p.NCH + ch] = make_float2(float_above(mx + (double)mps + (double)mpe), float_above(ex));
        if (p.warm_model) p.contrast[(size_t)b * p.NCH + ch] = ((redc[0] + redc[1]) + redc[2]) + redc[3];
    }
}

// One launch: the first p.ntab workgroups build the tables, workgroup p.ntab + b*NCH + ch sums a chunk, what favour_blocks adds
// looks at the durations of pairs of labels.
template <int ET>
__global__ __launch_bounds__(NT) void k_colsum(Params p)
{
    if ((int)blockIdx.x < p.ntab) {
        tables_body(p, blockIdx.x);
        return;
    }
    const int id = blockIdx.x - p.ntab;
    if (id >= p.NCH * p.B) favour_body(p, id - p.NCH * p.B);
    else colsum_body<ET>(p, id / p.NCH, id % p.NCH);
}

// Scaling block length J and the range flag of a sequence: fm = max |f - nu| over its positions and labels, boundary
// terms included; ex = largest excursion of the sums of f inside JMAX aligned positions, nm = max |nu|.  tabmax: the maxima of the
// p.ntab table workgroups.
__device__ __forceinline__ SeqHdr seq_header(const Params &p, const int L, const double fm, const double ex, const double nm,
                                             const double dmax, const double tmax)
{
    double grow = fm + fmax(dmax, 0.0) + fmax(tmax, 0.0) + p.logKC;
    double shrink = fm + fmax(-dmax, 0.0) + fmax(-tmax, 0.0);
    double r = fmax(fmax(grow, shrink), 1e-9);
    int J = 1, flags = 0;
    if (!(r <= RANGE_NATS)) flags = 1;  // also catches NaN
    // excursion of the centred sums inside JMAX aligned positions; between two positions of a shorter block it can be
    // twice that.  A boundary term is part of the pair of its position.
    const double exc = ex + (double)(JMAX - 1) * nm;
    const double term = (p.proj_start || p.proj_end || p.pi_start || p.pi_end) ? fm : 0.0;
    for (int n = 2; n <= JMAX; n *= 2) {
        const double E = fmin((double)(n - 1) * fm, n == JMAX ? exc : 2.0 * exc) + term;
        if (!((double)(n + 1) * r + E <= BLOCK_NATS)) break;
        J = n;
    }
    SeqHdr h;
    h.L = L; h.J = J; h.flags = flags; h.pad = 0; h.logZ = 0.0; h.logZb = 0.0;
    return h;
}
// The same with the maxima that k_colsum has left.
__device__ __forceinline__ SeqHdr seq_header(const Params &p, const int L, const double fm, const double ex, const double nm)
{
    double dmax = p.tabmax[0], tmax = p.tabmax[1];
    for (int i = 1; i < p.ntab; ++i) {
        dmax = fmax(dmax, p.tabmax[2 * i]);
        tmax = fmax(tmax, p.tabmax[2 * i + 1]);
    }
    return seq_header(p, L, fm, ex, nm, dmax, tmax);
}

// ---------------------------------------------------------------------------
// Eq. 1, stage 2, for sequences of many chunks: nu = mean over valid positions; chunk sums -> exclusive
// offsets of the centred prefix sum; scaling block length J.  grid B.
// ---------------------------------------------------------------------------
constexpr int PREP_NT = 1024;  // one workgroup per sequence: as many threads as a workgroup may have
__global__ __launch_bounds__(PREP_NT) void k_prep_seq(Params p)
{
    // The chunks are split into G = PREP_NT/C contiguous ranges, one per thread group; range sums
    // are combined in range order (a fixed order for a given problem).
    __shared__ double gsum[PREP_NT];
    __shared__ double red[PREP_NT / 64], redx[PREP_NT / 64];
    __shared__ double nu_s[256];  // C <= 256
    const int b = blockIdx.x, tid = threadIdx.x;
    const int C = p.C, L = seq_len(p, b), NCH = p.NCH;
    const int G = PREP_NT / C;
    const int g = tid / C, c = tid % C;
    const bool act = g < G;
    const int per = (NCH + G - 1) / G;
    const int c0 = min(g * per, NCH), c1 = min(c0 + per, NCH);
    double *cs = p.chsum + ((size_t)b * NCH) * C + c;
    double loc = 0.0;
    if (act) {
#pragma unroll 8
        for (int ch = c0; ch < c1; ++ch) loc += cs[(size_t)ch * C];
    }
    gsum[tid] = loc;
    __syncthreads();
    if (tid < C) {
        double total = 0.0;
        for (int gg = 0; gg < G; ++gg) total += gsum[gg * C + tid];
        const double nu = (p.center && L > 0) ? total / (double)L : 0.0;
        p.nu[(size_t)b * C + tid] = nu;
        nu_s[tid] = nu;
    }
    __syncthreads();
    if (act) {
        const double mynu = nu_s[c];
        double pref = 0.0;  // raw prefix sum at the start of this range
        for (int gg = 0; gg < g; ++gg) pref += gsum[gg * C + c];
#pragma unroll 8
        for (int ch = c0; ch < c1; ++ch) {
            const double sum = cs[(size_t)ch * C];
            const int nvalid = min(ch * PREP_CH, L);
            cs[(size_t)ch * C] = pref - (double)nvalid * mynu;
            pref += sum;
        }
    }
    // bounds on |f - nu| and on the excursions
    double fm = 0.0, ex = 0.0;
#pragma unroll 4
    for (int ch = tid; ch < NCH; ch += PREP_NT) {
        const float2 m = p.chmax[(size_t)b * NCH + ch];
        fm = fmax(fm, (double)m.x);
        ex = fmax(ex, (double)m.y);
    }
    fm = wave_max(fm);
    ex = wave_max(ex);
    if ((tid & 63) == 0) {
        red[tid >> 6] = fm;
        redx[tid >> 6] = ex;
    }
    __syncthreads();
    if (tid == 0) {
        for (int i = 0; i < PREP_NT / 64; ++i) {
            fm = fmax(fm, red[i]);
            ex = fmax(ex, redx[i]);
        }
        double nm = 0.0, npi = 0.0;
        for (int i = 0; i < C; ++i) {
            nm = fmax(nm, fabs(nu_s[i]));
            if (p.pi_start) npi = fmax(npi, fabs((double)p.pi_start[i]));
            if (p.pi_end) npi = fmax(npi, fabs((double)p.pi_end[i]));
        }
        p.hdr[b] = seq_header(p, L, fm + nm + 2.0 * npi, ex, nm);
    }
}

// ---------------------------------------------------------------------------
// Eq. 2: centred prefix sums S[t,c] (fp64), the per-block exponents n_j(c) and the pair
// (ES, 1/ES), ES = exp(S - n ln2).  grid (NCH, B), 256 threads; a workgroup takes one chunk of PREP_CH positions.
//
// INLINE: the workgroup also does what k_prep_seq does, for its own chunk: it reads ALL chunk sums of its sequence
// (label totals -> nu, the part before its chunk -> offset) and the chunk maxima (-> J); the first chunk's workgroup
// leaves nu and the header for the later kernels.  That is NCH*C doubles per workgroup from L2 instead of a launch of
// one workgroup per sequence (9 us at 391 chunks, 6 us at 2), and it grows like NCH^2: up to PREP_INLINE chunks.
//
// A chunk is cut into 32 segments of PREP_SEG = 8 positions; an item is (segment, label), labels fastest, so that a
// wave reads and writes whole cache lines.  An item loads its 8 emissions at once and adds them up, the segment sums
// of a label are scanned by one thread, then every item walks its 8 positions from its exact start.  (Segments of 32
// positions walked with one dependent load each took 25 us for a single chunk, all of it latency.)
// ---------------------------------------------------------------------------
constexpr int PREP_SEG = 8;
constexpr int PREP_NSEG = PREP_CH / PREP_SEG;
constexpr int PREP_INLINE = 512;
static_assert(PREP_CH % JMAX == 0 && JMAX % PREP_SEG == 0 && NT == 256 && PREP_NSEG == 32, "k_prefix geometry");

// 1/x to the last bit or two: hardware estimate and two Newton steps (x is a finite positive exp)
__device__ __forceinline__ double recip(const double x)
{
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}

// exp by the reduction x = n ln2 + r, |r| <= ln2 / 2, and the Taylor polynomial of degree 13 (remainder below 5e-18);
// without the library's special cases: finite arguments beyond +-708 overflow to inf or 0 in the scaling, infinite ones are not
// for it, NaN stays NaN.
__device__ __forceinline__ double exp_inner(const double x)
{
    constexpr double LN2_HI = 0x1.62e42fefa39efp-1, LN2_LO = 0x1.abc9e3b39803fp-56;  // ln 2 in two parts
    const double n = rint(x * LOG2E);
    const double r = fma(n, -LN2_LO, fma(n, -LN2_HI, x));
    double q = 1.0 / 6227020800.0;
    q = fma(q, r, 1.0 / 479001600.0);
    q = fma(q, r, 1.0 / 39916800.0);
    q = fma(q, r, 1.0 / 3628800.0);
    q = fma(q, r, 1.0 / 362880.0);
    q = fma(q, r, 1.0 / 40320.0);
    q = fma(q, r, 1.0 / 5040.0);
    q = fma(q, r, 1.0 / 720.0);
    q = fma(q, r, 1.0 / 120.0);
    q = fma(q, r, 1.0 / 24.0);
    q = fma(q, r, 1.0 / 6.0);
    q = fma(q, r, 0.5);
    q = fma(q, r, 1.0);
    q = fma(q, r, 1.0);
    return ldexp(q, (int)n);
}

// The same for any argument: 0 for -infinity and what is too small, infinity for what is too large, NaN for NaN.  (Boundary
// terms are added to the prefix sum, and -infinity is how a caller forbids a start or an end.)
__device__ __forceinline__ double exp_any(const double x)
{
    return exp_inner(x < -746.0 ? -746.0 : (x > 710.0 ? 710.0 : x));
}

// BTERMS: any boundary term of Eq. 4 present, or the log-domain pair of the max semiring; ET: emission storage type
// MODE: what has been done before.  PREP_OFFSETS: k_colsum and k_prep_seq; PREP_SUMS: k_colsum (INLINE above); PREP_NOTHING: the
// workgroup adds up its whole sequence itself, and one of them builds the tables, see prep_alone.
constexpr int PREP_OFFSETS = 0, PREP_SUMS = 1, PREP_NOTHING = 2;
constexpr int PREP_ALONE = 3;   // chunks
constexpr int PREP_ROUNDS = 2;  // items of 32 positions per thread
// Short sequences with small tables: the launch of k_colsum and the gap behind it cost more than sums that every workgroup of a
// sequence forms for itself, as long as these are few.  Time of a whole call with two launches over that with one, least .. most of
// training, scores and best segmentations with 4 .. 44 labels, T = 250 .. 760 (calls of 45 .. 1800 us):
//   sequences                     1             4             16            64            256          1024
//   one chunk                1.01 .. 1.08  1.01 .. 1.09  1.02 .. 1.09  1.03 .. 1.10  1.01 .. 1.06  1.00 .. 1.05
//   more, an item a thread   1.01 .. 1.07  1.03 .. 1.07  1.02 .. 1.06  1.02 .. 1.06  1.01 .. 1.04  1.00 .. 1.03
//   ... two items             .99 .. 1.05  1.01 .. 1.09  1.01 .. 1.04  1.02 .. 1.06  1.00 .. 1.03   .95 .. 1.03
//   ... three items and more  .98 .. 1.05   .99 .. 1.06  1.00 .. 1.04  1.00 .. 1.05   .99 .. 1.02   .98 .. 1.03
// With two items and three chunks it turns between 256 and 340 sequences (1.00 .. 1.03, .98 .. 1.01).  Start and end projections are
// read by every workgroup of the sequence, too; with those (replayed from a graph: host work is longer than the smallest of these calls)
//   one chunk                1.00 .. 1.02  1.01 .. 1.02  1.02 .. 1.13  1.02 .. 1.06  1.00 .. 1.03
//   two chunks                .98 .. 1.01   .99 .. 1.01  1.01 .. 1.09  1.00 .. 1.03   .99 .. 1.00
//   three chunks              .96 .. 1.01   .98 .. 1.05   .99 .. 1.07   .98 .. 1.02   .99 .. 1.01
inline bool prep_alone(const Params &p)
{
    if (p.NCH > PREP_ALONE || p.ntab != 1 || !p.dur || !p.trans || p.trans3) return false;
    const int items = (p.T + JMAX - 1) / JMAX * p.C, chunks = p.B * p.NCH;  // (no overflow: C <= 44 with one share of tables)
    if (items > PREP_ROUNDS * NT) return false;
    if (p.NCH == 1) return true;
    if (p.proj_start || p.proj_end) return p.NCH == 2 && chunks >= 32 && chunks <= 128;
    return items <= NT || chunks <= 768;
}

template <bool BTERMS, int ET, int MODE>
__global__ __launch_bounds__(NT) void k_prefix(Params p)
{
    constexpr bool INLINE = MODE != PREP_OFFSETS;
    extern __shared__ double lds_raw[];  // [PREP_NSEG][C] segment sums, then starts; INLINE: + [C] nu
    __shared__ double red2[2 * NT];
    __shared__ double redm[NT / 64], redx[NT / 64];
    __shared__ SeqHdr hs;
    // the first workgroup of a sequence chooses its first warm-up, where that comes from the model
    const int b = blockIdx.y, ch = (int)blockIdx.x - (p.warm_model ? 1 : 0), tid = threadIdx.x;
    const int C = p.C, NCH = p.NCH;
    if (ch < 0) {
        __shared__ float smp[PREP_ALONE * (NT / 64)];
        const int len = seq_len(p, b);
        double v[PREP_ALONE];
#pragma unroll
        for (int i = 0; i < PREP_ALONE; ++i) v[i] = MODE == PREP_NOTHING && i < NCH ? warm_load<ET>(p, b, i, len) : -INFINITY;
        warm_plan(p, b, lds_raw, red2, MODE == PREP_NOTHING ? smp : nullptr, [&]() {
#pragma unroll
            for (int i = 0; i < PREP_ALONE; ++i) {
                const float s = i < NCH ? warm_sample(p, i, len, v[i]) : 0.f;
                if ((tid & 63) == 0) smp[i * (NT / 64) + (tid >> 6)] = s;
            }
        });
        return;
    }
    constexpr int NTB = MODE == PREP_NOTHING ? TAB_ITEMS / NT : 1;
    float tab[NTB];  // this thread's entries of the tables, before exp (duration biases first)
    const int KC = p.K * C;
    double *seg = lds_raw, *nus = lds_raw + PREP_NSEG * C;
    const size_t f0 = (size_t)b * p.T * C;
    int L, J;
    double off = 0.0;  // threads tid < C: centred prefix sum at the chunk's first position
    if (INLINE) {
        L = seq_len(p, b);
        const int G = NT / C, g = tid / C, c = tid % C;
        const double *cs = p.chsum + (size_t)b * NCH * C + c;
        double tot = 0.0, pre = 0.0, fm = 0.0, ex = 0.0, mxd = -DBL_MAX, mxt = -DBL_MAX;
        if (MODE == PREP_NOTHING) {
            __shared__ double csum[PREP_ROUNDS * NT];
            const int ngr = (L + JMAX - 1) / JMAX;  // groups of positions
#pragma unroll
            for (int u = 0; u < NTB; ++u) {
                const int i = min(u * NT + tid, KC + C * C - 1);
                tab[u] = *(i < KC ? p.dur + i : p.trans + (i - KC));
            }
            const bool proj = BTERMS && (p.proj_start || p.proj_end);
            double mc[PREP_ALONE] = {};  // with projections: the largest emission of each chunk
            for (int it = tid; it < ngr * C; it += NT) {
                const int g32 = it / C;
                double m = 0.0;
                csum[it] = col_item<ET>(p, f0 + (size_t)g32 * JMAX * C + it % C, min(L - g32 * JMAX, JMAX), m, ex);
                if (proj) {
#pragma unroll
                    for (int i = 0; i < PREP_ALONE; ++i) mc[i] = fmax(mc[i], g32 / COL_NG == i ? m : 0.0);
                } else {
                    fm = fmax(fm, m);
                }
            }
            if (proj) {  // the largest sum of a chunk's three maxima, not the sum of the sequence's: see colsum_body
                constexpr int NW = NT / 64;
#pragma unroll
                for (int i = 0; i < PREP_ALONE; ++i) {
                    const int u0 = i * PREP_CH, u1 = min(u0 + PREP_CH, L);
                    const double m[3] = {wave_max(mc[i]), wave_max((double)rows_absmax(p, p.proj_start, b, u0, u1)),
                                         wave_max((double)rows_absmax(p, p.proj_end, b, u0, u1))};
                    if ((tid & 63) == 0) {
#pragma unroll
                        for (int j = 0; j < 3; ++j) red2[(i * 3 + j) * NW + (tid >> 6)] = m[j];
                    }
                }
                __syncthreads();
#pragma unroll
                for (int i = 0; i < PREP_ALONE; ++i) {
                    double sum = 0.0;
#pragma unroll
                    for (int j = 0; j < 3; ++j) {
                        const double *r = red2 + (i * 3 + j) * NW;
                        sum += fmax(fmax(r[0], r[1]), fmax(r[2], r[3]));
                    }
                    fm = fmax(fm, sum);
                }
            }
#pragma unroll
            for (int u = 0; u < NTB; ++u) {
                const int i = u * NT + tid;
                mxd = fmax(mxd, i < KC ? (double)tab[u] : -DBL_MAX);
                mxt = fmax(mxt, i >= KC ? (double)tab[u] : -DBL_MAX);
            }
            mxd = wave_max(mxd);
            mxt = wave_max(mxt);
            __syncthreads();
            if (tid < C) {
                for (int i = 0; i * COL_NG < ngr; ++i) {  // chunk by chunk
                    double s = 0.0;
#pragma unroll
                    for (int q = 0; q < COL_NG; ++q) s += i * COL_NG + q < ngr ? csum[min(i * COL_NG + q, ngr - 1) * C + tid] : 0.0;
                    tot += s;
                    pre += i < ch ? s : 0.0;
                }
            }
        } else if (g < G) {
#pragma unroll 8
            for (int i = g; i < NCH; i += G) {
                const double v = cs[(size_t)i * C];
                tot += v;
                pre += i < ch ? v : 0.0;
            }
        }
        if (MODE == PREP_SUMS) {
            for (int i = tid; i < NCH; i += NT) {
                const float2 m = p.chmax[(size_t)b * NCH + i];
                fm = fmax(fm, (double)m.x);
                ex = fmax(ex, (double)m.y);
            }
            red2[tid] = tot;
            red2[NT + tid] = pre;
            __syncthreads();
        }
        double nm = 0.0;
        if (tid < C) {
            if (MODE == PREP_SUMS) {
                tot = 0.0;
                for (int gg = 0; gg < G; ++gg) {
                    tot += red2[gg * C + tid];
                    off += red2[NT + gg * C + tid];
                }
            } else {
                off = pre;
            }
            const double nu = (p.center && L > 0) ? tot / (double)L : 0.0;
            off -= (double)min(ch * PREP_CH, L) * nu;
            nus[tid] = nu;
            if (ch == 0) p.nu[(size_t)b * C + tid] = nu;
            nm = fabs(nu);
        }
        // maxima of |f|, of the excursions, of |nu| and of the scalar boundaries: inside each wave, then over the waves
        double npi = 0.0;
        if (BTERMS && tid < C) {
            if (p.pi_start) npi = fabs((double)p.pi_start[tid]);
            if (p.pi_end) npi = fmax(npi, fabs((double)p.pi_end[tid]));
        }
        fm = wave_max(fm);
        ex = wave_max(ex);
        nm = wave_max(nm);
        if (BTERMS) npi = wave_max(npi);
        if (MODE == PREP_SUMS) __syncthreads();
        if ((tid & 63) == 0) {
            redm[tid >> 6] = fm;
            redx[tid >> 6] = ex;
            red2[tid >> 6] = nm;
            red2[NT + (tid >> 6)] = npi;
            if (MODE == PREP_NOTHING) {
                red2[8 + (tid >> 6)] = mxd;
                red2[16 + (tid >> 6)] = mxt;
            }
        }
        __syncthreads();
        if (tid == 0) {
            for (int i = 0; i < NT / 64; ++i) {
                fm = fmax(fm, redm[i]);
                ex = fmax(ex, redx[i]);
                nm = fmax(nm, red2[i]);
                npi = fmax(npi, red2[NT + i]);
                if (MODE == PREP_NOTHING) {
                    mxd = fmax(mxd, red2[8 + i]);
                    mxt = fmax(mxt, red2[16 + i]);
                }
            }
            // (single precision upwards, as k_colsum leaves them)
            hs = MODE == PREP_NOTHING ? seq_header(p, L, (double)float_above(fm) + nm + 2.0 * npi, (double)float_above(ex), nm, mxd, mxt)
                                      : seq_header(p, L, fm + nm + 2.0 * npi, ex, nm);
            if (ch == 0) p.hdr[b] = hs;
        }
    } else {
        const SeqHdr h = p.hdr[b];
        L = h.L;
        J = h.J;
        if (tid < C) {
            nus[tid] = p.nu[(size_t)b * C + tid];
            off = p.chsum[((size_t)b * NCH + ch) * C + tid];
        }
    }
    __syncthreads();
    if (INLINE) J = hs.J;
    const int Jm = J - 1;
    const int tc = ch * PREP_CH;
    const size_t row0 = (size_t)b * (p.T + 1);
    const int items = PREP_NSEG * C;
    if (MODE == PREP_NOTHING && b == 0 && ch == NCH - 1) {
#pragma unroll
        for (int u = 0; u < NTB; ++u) {
            const int i = u * NT + tid;
            if (i < KC + C * C) (i < KC ? p.W : p.Etr - KC)[i] = exp((double)tab[u]);
        }
    }
    auto load = [&](const int t0, const int c, double (&f)[PREP_SEG]) {
        const size_t o = f0 + (size_t)t0 * C + c;
        if (t0 + PREP_SEG <= L) {
#pragma unroll
            for (int i = 0; i < PREP_SEG; ++i) f[i] = emis_at<ET>(p, o + (unsigned)(i * C));
        } else {
#pragma unroll
            for (int i = 0; i < PREP_SEG; ++i) f[i] = t0 + i < L ? emis_at<ET>(p, o + (unsigned)(i * C)) : 0.0;
        }
    };
    for (int it = tid; it < items; it += NT) {
        const int s = it / C, c = it - s * C;
        const int t0 = tc + s * PREP_SEG;
        double f[PREP_SEG];
        load(t0, c, f);
        const double sum = ((f[0] + f[1]) + (f[2] + f[3])) + ((f[4] + f[5]) + (f[6] + f[7]));
        seg[it] = fma(-(double)max(0, min(PREP_SEG, L - t0)), nus[c], sum);
    }
    __syncthreads();
    if (tid < C) {
        double v[PREP_NSEG];
#pragma unroll
        for (int s = 0; s < PREP_NSEG; ++s) v[s] = seg[s * C + tid];
        double S = off;
#pragma unroll
        for (int s = 0; s < PREP_NSEG; ++s) {
            seg[s * C + tid] = S;
            S += v[s];
        }
    }
    __syncthreads();
    const int bmask = ~((J < PREP_SEG ? 1 : J / PREP_SEG) - 1), logJ = 31 - __clz(J);
    for (int it = tid; it < items; it += NT) {
        const int s = it / C, c = it - s * C;
        const int t0 = tc + s * PREP_SEG;
        if (t0 > p.T) break;
        double f[PREP_SEG];
        load(t0, c, f);
        const double nu = nus[c];
        double S = seg[it];
        // exponent of the scaling block that position t0 lies in: from the sum at the block's first position, which
        // is the start of a segment of this chunk (blocks longer than a segment), or t0 itself (shorter ones)
        double n = rint(seg[(s & bmask) * C + c] * LOG2E);
        double base = n * LN2;
        double2 *E = p.EI + (row0 + t0) * C + c;
        if (!BTERMS && J >= PREP_SEG && t0 + PREP_SEG <= L && !p.cum) {
            if ((t0 & Jm) == 0) p.nbase[(row0 + (size_t)(t0 >> logJ)) * C + c] = (int)n;
#pragma unroll
            for (int i = 0; i < PREP_SEG; ++i) {
                const double es = exp_inner(S - base);
                E[(unsigned)(i * C)] = make_double2(es, recip(es));
                S += f[i] - nu;
            }
            continue;
        }
        const bool inside = J >= PREP_SEG && t0 + PREP_SEG <= L && !p.cum;
        if (BTERMS && (MODE == PREP_NOTHING ? __all(inside) : inside)) {
            // The same for a segment inside the sequence: all projections are requested at once and nothing is decided per
            // position (genomic analysis 662 -> 654 us, this kernel 109 -> 104).  In the single launch of short sequences, where one wave at a sequence's
            // end that takes both ways is as long as the launch, only where the whole wave can (decoding, 6 x 750, K = 4,
            // C = 5: 69.7 us without this path, 70.8 with it in every lane that can, 70.2; 64 x 256, K = 16, C = 24 84.6, 81.8, 82.1).
            if ((t0 & Jm) == 0) p.nbase[(row0 + (size_t)(t0 >> logJ)) * C + c] = (int)n;
            const size_t o = f0 + (size_t)t0 * C + c;
            float fs[PREP_SEG], fe[PREP_SEG];
#pragma unroll
            for (int i = 0; i < PREP_SEG; ++i) {
                fs[i] = p.proj_start ? p.proj_start[o + (unsigned)(i * C)] : 0.f;
                fe[i] = p.proj_end ? p.proj_end[t0 + i >= 1 ? o + (unsigned)(i * C) - C : o] : 0.f;
            }
#pragma unroll
            for (int i = 0; i < PREP_SEG; ++i) {
                double ps = (double)fs[i], pe = (double)fe[i];
                if (i == 0 && t0 == 0) {
                    pe = 0.0;
                    if (p.pi_start) ps += (double)p.pi_start[c];
                }
                E[(unsigned)(i * C)] = p.logpair ? make_double2(S + pe, ps - S)
                                                 : make_double2(exp_any((S - base) + pe), exp_any(ps - (S - base)));
                S += f[i] - nu;
            }
            continue;
        }
        // boundary terms: start score of token t, end score of token t-1
        double xs[PREP_SEG], xe[PREP_SEG];
        if (BTERMS) {
            const size_t o = f0 + (size_t)t0 * C + c;
#pragma unroll
            for (int i = 0; i < PREP_SEG; ++i) {
                xs[i] = (p.proj_start && t0 + i < L) ? (double)p.proj_start[o + (unsigned)(i * C)] : 0.0;
                xe[i] = (p.proj_end && t0 + i >= 1 && t0 + i <= L) ? (double)p.proj_end[o + (unsigned)(i * C) - C] : 0.0;
            }
            if (t0 == 0 && L > 0 && p.pi_start) xs[0] += (double)p.pi_start[c];
            if (p.pi_end) {
#pragma unroll
                for (int i = 0; i < PREP_SEG; ++i)
                    if (t0 + i == L && L >= 1) xe[i] += (double)p.pi_end[c];
            }
        }
#pragma unroll
        for (int i = 0; i < PREP_SEG; ++i) {
            const int t = t0 + i;
            if (t <= L) {
                if ((t & Jm) == 0) {
                    n = rint(S * LOG2E);
                    p.nbase[(row0 + (size_t)(t >> logJ)) * C + c] = (int)n;
                    base = n * LN2;
                }
                const double x = S - base;
                double2 pr;
                if (!BTERMS) {
                    const double es = exp_inner(x);
                    pr = make_double2(es, recip(es));
                } else {
                    // (ES * exp(end score of token t-1), exp(start score of token t) / ES): every message
                    // that arrives at position t is multiplied by the first, every one that leaves by the second;
                    // max semiring: the same pair in the log domain, (S + end score, start score - S)
                    pr = p.logpair ? make_double2(S + xe[i], xs[i] - S)
                                   : make_double2(exp_any(x + xe[i]), exp_any(xs[i] - x));
                }
                E[(unsigned)(i * C)] = pr;
                if (p.cum) p.cum[(row0 + t) * C + c] = S;
                if (t < L) S += f[i] - nu;
            } else if (p.cum && t <= p.T) {
                p.cum[(row0 + t) * C + c] = 0.0;
            }
        }
    }
}

// Dynamic LDS of k_prefix.
inline size_t prefix_lds(const int C) { return ((size_t)PREP_NSEG * C + C) * sizeof(double); }
