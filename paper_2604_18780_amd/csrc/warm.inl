// The first warm-up of the chunk-parallel scans, from the model and the scores.
// Included by semicrf.hip inside its anonymous namespace (after common.h); not a translation unit of its own.

// ---------------------------------------------------------------------------
// How many positions a scan task needs before its interval until its start is forgotten, per sequence.
//
// A message entry that leaves position s with label c reaches every later position t with the weight W[t-s, c], so what an
// old entry still adds there is measured against what the newer entries add.  Where a label keeps being fed (by itself and
// by detours through other labels) with g per position, the entries of its window grow like lambda^t with
// g sum_k W[k,c] lambda^-k = 1, and what was in the window n positions ago has become lambda^-n of it.  The slowest label
// decides.  g comes from the transition matrix: Etr[c,c] for the label itself, plus r Etr[c,o] Etr[o,c] for a detour of
// one position through o, where r is how far the other labels' scores lie below the best one (the mean over every
// WARM_EVERY-th position of log sum_c exp(score - best), sampled by k_colsum, or by k_prefix itself).
//
// Growth is not all: the labels' shares must settle, too.  They settle as fast where the transitions are about alike, and ever more
// slowly the sharper these are, most of all where the scores tell nothing (r near 1), while the detours' sum grows.  So a
// detour counts for 1 at most, and the length grows with s, the standard deviation of the transition scores that are not
// forbidden (or by how much a label's own is above the others', where that is more): 1.15 + (0.02 + r) s^2 + (0.04 + 0.3 r) s^4
// times what the growth asks for.  Where that factor is above 2.4 it varies too much from model to model to be worth less than
// half of the default length.  Models in which a label reaches another only over several steps (forbidden transitions) forget
// more slowly, about in proportion to the steps.
//
// The length only decides how long the scan takes: whether it was enough is checked at every interval boundary
// (k_spec_cmp).  Found in a replay of the recurrences at 24 boundaries of each of 10 752 random models: C = 3 .. 64, K = 8 .. 300,
// transitions N(0, s^2), s = 0.1 .. 3, as they are, with 40 % or all beyond a band of 2 forbidden, with the labels' own
// forbidden or raised by 1 or 2, all lowered by 2; scores that tell much, little and nothing; durations favoured by up to
// 0.2 a position.  Positions until the mismatch is below 1e-13, in units of log(1e15) / log(lambda), at most (means of 2 and noise of
// 1 | noise of 0.1 alone): 1.2 | 1.0 at s = 0.1, 1.1 | 1.4 at 0.5, 1.3 | 2.3 at 1, 1.7 | 5 at 1.3, 3.9 | 11 at 2; per step where
// a band is all that is allowed, mostly 0.5 .. 0.8 | 1.7 .. 4.  Without a band the choice sufficed at all 24 boundaries for every
// model up to s = 1 whose scores tell anything, but for 0 .. 10 % of those with the labels' own raised by 2,
// 0 .. 12 % by 1, 0 .. 2 % with 40 % forbidden; where they tell nothing but for 0 .. 4 %; up to s = 1.6 but for 0 .. 22 % (25 %); with means of 2 it was 47 positions
// on average, of 179 by default.  Of a thousand boundaries one or two take longer, mostly in long runs of one label: those are mended.
//
// A longer warm-up than K + (that) is never needed for the windows to agree entry by entry; a shorter one leaves the older
// entries of the window different, in places where they no longer matter.  negl[c] = 1 / (K R), with R the largest ratio of
// the weight of a longer duration to that of a shorter one: an entry below negl[c] times a newer entry of its label adds,
// at every later position, less than 1/K of what the newer one adds there.
// ---------------------------------------------------------------------------
constexpr int WARM_EVERY = 64;      // one position in so many is sampled: one per wave and chunk
constexpr int WARM_TERMS = 16;      // durations that enter lambda (a growth that needs more of them is slow anyway)
constexpr int WARM_PER = 16;        // most window entries per thread of the comparison that ignores negligible ones
constexpr double WARM_NATS = 34.5;  // log(1e15): a hundredth of the bound on states after a chosen warm-up
constexpr double WARM_FACTOR = 2.4; // largest factor for sharpness with which any length below the default is chosen
static_assert(PREP_CH == WARM_EVERY * (NT / 64), "every wave takes one sample of a chunk");

// The contrast of a chunk's scores: every wave takes one position, a label per lane.  warm_load is called early, so that
// the score is there when warm_sample needs it.
template <int ET>
__device__ __forceinline__ double warm_load(const Params &p, const int b, const int ch, const int L)
{
    const int lane = threadIdx.x & 63, t = ch * PREP_CH + (threadIdx.x >> 6) * WARM_EVERY;
    if (t >= L) return -INFINITY;  // (the same for the whole wave; positions beyond the sequence are never read)
    const double v = emis_at<ET>(p, ((size_t)b * p.T + t) * p.C + min(lane, p.C - 1));
    return lane < p.C ? v : -INFINITY;
}
__device__ __forceinline__ float warm_sample(const Params &p, const int ch, const int L, const double v)  // per wave
{
    const float e = __expf((float)(v - wave_max(v)));
    const float l = __logf((float)wave_sum((double)e));
    const int t = ch * PREP_CH + (threadIdx.x >> 6) * WARM_EVERY;
    return t < L && l > 0.f && l < 100.f ? l : 0.f;  // scores that are not numbers count as certain
}

// One matrix per duration: the largest log weight of a longer duration over a shorter one for sixteen pairs of labels, left in
// the place of the table (which is built later).  Sixteen ranges of durations a pair, then over the ranges in order.  (In warm_plan, by
// a single workgroup, it took 20 us longer than the prefix sums it runs beside: K = 64, C = 24, T = 100 000 52 -> 72 us.)
constexpr int WARM_PAIRS = NT / 16;
__device__ __forceinline__ void favour_body(const Params &p, const int blk)
{
    __shared__ float red[3][NT / 64][WARM_PAIRS];
    const int tid = threadIdx.x, g = tid / WARM_PAIRS, K = p.K, C = p.C, CC = C * C;
    const int pair = blk * WARM_PAIRS + tid % WARM_PAIRS, pr = min(pair, CC - 1);
    const int per = (K + NT / WARM_PAIRS - 1) / (NT / WARM_PAIRS), k0 = min(g * per, K), k1 = min(k0 + per, K);
    float mn = INFINITY, mx = -INFINITY, best = 0.f;
#pragma unroll 8
    for (int k = k0; k < k1; ++k) {
        const float v = p.dur[(size_t)k * C + pr % C] + p.trans3[(size_t)k * CC + pr];
        best = fmaxf(best, v - mn);
        mn = fminf(mn, v);
        mx = fmaxf(mx, v);
    }
    auto then = [&](const float mn2, const float mx2, const float best2) {  // a later range
        best = fmaxf(best, fmaxf(best2, mx2 - mn));
        mn = fminf(mn, mn2);
        mx = fmaxf(mx, mx2);
    };
#pragma unroll
    for (int off = WARM_PAIRS; off < 64; off <<= 1) then(__shfl_down(mn, off), __shfl_down(mx, off), __shfl_down(best, off));
    if ((tid & 63) < WARM_PAIRS) {
        red[0][tid >> 6][tid & 63] = mn;
        red[1][tid >> 6][tid & 63] = mx;
        red[2][tid >> 6][tid & 63] = best;
    }
    __syncthreads();
    if (g != 0 || pair >= CC) return;
#pragma unroll
    for (int i = 1; i < NT / 64; ++i) then(red[0][i][tid], red[1][i][tid], red[2][i][tid]);
    ((float *)p.G3)[pair] = best;
}
inline int favour_blocks(const Params &p) { return p.warm_model && p.trans3 ? (p.C * p.C + WARM_PAIRS - 1) / WARM_PAIRS : 0; }

// One workgroup per sequence, next to those of k_prefix; it should not take longer than they do (64 sequences of a
// chunk of 24 labels: the launch takes 15.2 us without, 15.8 with it; with 4 labels and two chunks it does: 6.9 without, 10.8).  So
// everything that comes from memory is requested before anything is done with it, and the transition matrix is worked on in
// LDS by four threads per label.  lds: (PREP_NSEG + 1) C doubles, buf: 2 NT.
// smp: place in LDS for the samples of the sequence's chunks, NT / 64 each, which sample() takes; without, p.contrast holds their sums.
template <class Sample>
__device__ __forceinline__ void warm_plan(const Params &p, const int b, double *lds, double *buf, const float *smp, Sample sample)
{
    // buf, one after the other: ranges of durations [3 * NT]; detours (all, counted for 1 at most) and best successors, [4][64]
    // each; successors [4][64]
    float *red = (float *)buf, *part = (float *)buf, *part1 = part + NT, *best4 = part + 2 * NT;
    unsigned long long *succ = (unsigned long long *)buf;
    __shared__ double cons[NT / 64], off[3][NT / 64];
    static_assert(NT == 4 * 64, "four threads per label");
    const int tid = threadIdx.x, lane = tid & 63, wv = tid >> 6;
    const int K = p.K, C = p.C, CC = C * C;
    const bool dt = p.trans3 != nullptr;
    const float *t1 = dt ? p.trans3 : p.trans;  // transitions (with one matrix per duration: of duration 1)
    const int ts = C + 1;                       // row stride of their copy
    float *tl = (float *)lds;                   // [C][ts]
    const int lc = min(lane, C - 1), n = min(K, WARM_TERMS);
    // ---- requests: transitions, the first durations of the lane's label, this thread's range of durations, contrast
    constexpr int NTR = (64 * 64 + NT - 1) / NT, NWR = (64 * WARM_TERMS + NT - 1) / NT;
    float tr[NTR], wq[NWR], dq[NWR], du[WARM_PER];
#pragma unroll
    for (int i = 0; i < NTR; ++i) tr[i] = i * NT < CC ? t1[min(i * NT + tid, CC - 1)] : 0.f;
#pragma unroll
    for (int i = 0; i < NWR; ++i) {
        const int e = min(i * NT + tid, n * C - 1);
        wq[i] = p.dur[e];
        dq[i] = dt ? p.trans3[(size_t)(e / C) * CC + e % C * (C + 1)] : 0.f;
    }
    const int G = NT / C, g = tid / C, per = (K + G - 1) / G, k0 = g * per, k1 = g < G ? min(k0 + per, K) : k0;
#pragma unroll
    for (int u = 0; u < WARM_PER; ++u) du[u] = p.dur[(size_t)min(k0 + u, K - 1) * C + tid % C];
    float fv[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 4; ++i)
        if (dt) fv[i] = ((const float *)p.G3)[min(i * NT + tid, CC - 1)];
    // contrast: of this sequence alone, so that what happens to it does not depend on the others of its batch
    double con = 0.0;
    if (smp) {
        sample();
    } else {
#pragma unroll 8
        for (int i = tid; i < p.NCH; i += NT) con += (double)p.contrast[(size_t)b * p.NCH + i];
    }
    const double cnt = (double)((seq_len(p, b) + WARM_EVERY - 1) / WARM_EVERY);
    // ---- largest log weight of a longer duration over a shorter one, per label (and source label where they have
    // matrices of their own): ranges of durations, then over the ranges in order
    float favour = 0.f;  // lanes of the first wave: that of their label
    if (!dt) {
        float mn = INFINITY, mx = -INFINITY, best = 0.f;
#pragma unroll
        for (int u = 0; u < WARM_PER; ++u) {
            if (k0 + u < k1) {
                const float v = du[u];
                best = fmaxf(best, v - mn);
                mn = fminf(mn, v);
                mx = fmaxf(mx, v);
            }
        }
        red[tid] = mn;
        red[NT + tid] = mx;
        red[2 * NT + tid] = best;
        __syncthreads();
        if (tid < C) {
#pragma unroll 4
            for (int gg = 1; gg < G; ++gg) {
                best = fmaxf(best, fmaxf(red[2 * NT + gg * C + tid], red[NT + gg * C + tid] - mn));
                mn = fminf(mn, red[gg * C + tid]);
            }
            favour = best;
            // weights below exp(-700) are zero in the tables: nothing is negligible next to them
            if (p.logpair) p.negl[(size_t)b * C + tid] = (double)best * 1.000001;
            else p.negl[(size_t)b * C + tid] = best < 600.f ? exp(-1.001 * (double)best) / (double)K : 0.0;  // (differences are rounded)
        }
    } else {  // (by pairs of labels, from k_colsum)
#pragma unroll
        for (int i = 0; i < 4; ++i) red[i * NT + tid] = fv[i];
        __syncthreads();
        if (tid < C) {
            float best = red[tid];
#pragma unroll 8
            for (int o = 1; o < C; ++o) best = fmaxf(best, red[o * C + tid]);
            favour = best;
            p.negl[(size_t)b * C + tid] = best < 600.f ? exp(-1.001 * (double)best) / (double)K : 0.0;  // (differences are rounded)
        }
    }
#pragma unroll
    for (int i = 0; i < NTR; ++i) {
        const int e = i * NT + tid;
        if (e < CC) tl[e / C * ts + e % C] = tr[i];
    }
    // (added up as k_colsum does it, so that both prefix stages choose the same length)
    if (smp && tid < p.NCH) con = (double)(((smp[4 * tid] + smp[4 * tid + 1]) + smp[4 * tid + 2]) + smp[4 * tid + 3]);
    con = wave_sum(con);
    __syncthreads();  // (the ranges above have been read)
    if (lane == 0) cons[wv] = con;
    // ---- detours of a label and its best successor, four threads per label
    const float stay = tl[lc * ts + lc];
    float det = 0.f, det1 = 0.f, mx = -INFINITY;
    const int o0 = wv * ((C + 3) / 4), o1 = min(o0 + (C + 3) / 4, C);
#pragma unroll 4
    for (int o = o0; o < o1; ++o) {
        const float out = tl[lc * ts + o], d = o == lc ? 0.f : __expf(out + tl[o * ts + lc]);
        det += d;
        det1 += fminf(d, 1.f);
        mx = fmaxf(mx, out);
    }
    part[wv * 64 + lane] = det;
    part1[wv * 64 + lane] = det1;
    best4[wv * 64 + lane] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(best4[lane], best4[64 + lane]), fmaxf(best4[128 + lane], best4[192 + lane]));
    det = ((part[lane] + part[64 + lane]) + part[128 + lane]) + part[192 + lane];
    det1 = ((part1[lane] + part1[64 + lane]) + part1[128 + lane]) + part1[192 + lane];
    __syncthreads();
    unsigned long long reach = 0;        // successors within eight nats of the best one
    double os = 0.0, oss = 0.0, on = 0.0;  // scores of the other labels (forbidden ones apart): sum, of squares, number
#pragma unroll 4
    for (int o = o0; o < o1; ++o) {
        const float v = tl[lc * ts + o];
        reach |= (unsigned long long)(v > mx - 8.f) << o;
        const double x = lane < C && o != lc && v > mx - 50.f ? (double)v : 0.0;
        os += x;
        oss += x * x;
        on += lane < C && o != lc && v > mx - 50.f ? 1.0 : 0.0;
    }
    succ[wv * 64 + lane] = reach;
    os = wave_sum(os);
    oss = wave_sum(oss);
    on = wave_sum(on);
    if (lane == 0) off[0][wv] = os, off[1][wv] = oss, off[2][wv] = on;
    __syncthreads();
    float *wl = tl;  // [2][WARM_TERMS][C], in the place of the transitions: durations, own transitions of each
#pragma unroll
    for (int i = 0; i < NWR; ++i) {
        if (i * NT + tid < n * C) {
            wl[i * NT + tid] = wq[i];
            wl[WARM_TERMS * C + i * NT + tid] = dq[i];
        }
    }
    __syncthreads();
    if (wv != 0) return;
    con = ((cons[0] + cons[1]) + cons[2]) + cons[3];
    const float r = cnt > 0.0 ? (__expf((float)(con / cnt)) - 1.f) / (float)(C - 1) : 0.f;
    // ---- how sharp the transitions are: s^2
    double sharp;
    {
        const bool own = lane < C && stay > mx - 50.f;
        const double so = own ? (double)stay : 0.0, sn = wave_sum(own ? 1.0 : 0.0), st = wave_sum(so), sst = wave_sum(so * so);
        os = ((off[0][0] + off[0][1]) + off[0][2]) + off[0][3];
        oss = ((off[1][0] + off[1][1]) + off[1][2]) + off[1][3];
        on = ((off[2][0] + off[2][1]) + off[2][2]) + off[2][3];
        const double mean = (os + st) / (on + sn), raised = on > 0.0 && sn > 0.0 ? fmax(st / sn - os / on, 0.0) : 0.0;
        sharp = fmax((oss + sst) / (on + sn) - mean * mean, raised * raised);
    }
    // ---- steps from a label to every other
    reach = (succ[lane] | succ[64 + lane]) | (succ[128 + lane] | succ[192 + lane]);
    const unsigned long long full = C >= 64 ? ~0ull : (1ull << C) - 1ull;
    int hops = 1;
    if (__ballot(reach != full)) {
        unsigned long long *const adj = succ;
        adj[lane] = reach;
        lds_wave_fence();
        unsigned long long front = reach;
        while (hops < 64 && __ballot(reach != full)) {
            unsigned long long nx = 0;
            while (front) {
                nx |= adj[__ffsll(front) - 1];
                front &= front - 1;
            }
            front = nx & ~reach;
            if (!__ballot(front != 0)) hops = 64;  // some label is never reached
            else ++hops;
            reach |= nx;
        }
    }
    favour = (float)wave_max((double)favour);
    if (p.logpair) {
        // Best score: what decides is how soon all best paths into a window have met, which takes an emission that tells
        // the labels apart, but not for certain, and a label change or a split that pays.  In a replay of 12 boundaries of each of 3 504
        // models (C = 3 .. 48, K = 24 .. 128, transitions N(0, s^2)) the share of models where not all had met after these lengths,
        // and after 2 K: r = 0.12 .. 0.4, s up to 1.5 0.2 % (up to 98 positions), 0; s = 2 0.9 %, 0; r = 0.35 .. 0.56, s up to 1 0, 0, s = 1.5 11 %, 7 %;
        // r = 0.58 .. 0.88 0 .. 63 %, 0 .. 44 %; r = 0.03 .. 0.05 4 .. 26 %, 0 .. 4 %; own transitions or others forbidden 0 .. 63 %, 0 .. 89 %.
        if (lane != 0) return;
        const int deflt = vit_warmup(K), shrt = C >= 16 ? 40 : (C >= 8 ? 48 : (C >= 5 ? 64 : 96));
        const bool plain = hops == 1 && favour < 4.f && r > 0.08f && r < 0.45f && sharp < 1.7 * 1.7;
        p.wlen[b].x = plain ? min(shrt, deflt) : deflt;
        return;
    }
    // ---- growth of the label: y = 1 / lambda
    float y1 = 1.f;
    {
        const float q = r * (hops > 2 ? det : det1);  // (steps are counted for themselves)
        float w[WARM_TERMS];
#pragma unroll
        for (int k = 0; k < WARM_TERMS; ++k) {
            const float *wk = wl + min(k, n - 1) * C + lc;
            w[k] = k < n ? __expf(wk[0]) * (__expf(dt ? wk[WARM_TERMS * C] : stay) + q) : 0.f;
        }
        float y0 = 0.f;
        for (int it = 0; it < 12; ++it) {
            const float y = 0.5f * (y0 + y1);
            float s0 = 0.f, s1 = 0.f;  // even and odd durations, two chains
#pragma unroll
            for (int k = WARM_TERMS - 2; k >= 0; k -= 2) {
                s0 = fmaf(s0, y * y, w[k]);
                s1 = fmaf(s1, y * y, w[k + 1]);
            }
            if (fmaf(s1, y, s0) * y > 1.f) y1 = y;
            else y0 = y;
        }
    }
    double lam = lane < C ? (double)-__logf(y1) : INFINITY;  // log(lambda); 0 where there is no growth
    lam = -wave_max(lam == lam ? -lam : 0.0);
    if (lane != 0) return;
    const double deflt = (double)sum_warmup(K);
    double wd = deflt;
    if (lam > 0.01 && hops < 64) {
        // a few positions say little about the contrast; entries that later durations favour must have fallen further
        const double m = (WARM_NATS + (double)favour) / lam * (1.0 + 0.25 / sqrt(fmax(cnt, 1.0)));
        if (hops > 2) {
            const double far = (0.55 + 1.5 * (double)r) * m * (double)hops;
            if (far > deflt) wd = fmin(far, (double)p.warm_long);
            else if (sharp < 1.6 * 1.6) wd = fmin(deflt, fmax(16.0, far) + 4.0);
        } else if (sharp < 2.2 * 2.2) {
            const double factor = 1.15 + (0.02 + (double)r) * sharp + (0.04 + 0.3 * (double)r) * sharp * sharp;
            const double n = fmax(16.0, factor * m) + 4.0;
            if (n < (factor <= WARM_FACTOR ? deflt : 0.5 * deflt)) wd = n;
            // sharp transitions and windows that will hardly agree entry by entry after the default length
            else if (factor <= WARM_FACTOR && sharp > 0.36 && (double)K + 0.5 * n > deflt) wd = fmin(n, 1.5 * deflt);
        }
    }
    if (!(p.warm_model & WARM_SHORTER)) wd = hops > 2 ? fmax(wd, deflt) : deflt;
    p.wlen[b] = make_int4(wd == deflt ? sum_warmup(K) : ((int)wd + 3) & ~3, p.warm_long, p.warm_long, hops > 2 && wd > deflt);
}

// The first warm-up of a scan task of sequence b; deflt: what it is without a model.
__device__ __forceinline__ int first_warm(const Params &p, const int b, const int deflt)
{
    return p.warm_model ? p.wlen[b].x : deflt;
}

// The same for the scans with duration-dependent transitions, whose second attempt's warm-up k_spec_fix leaves.
__device__ __forceinline__ int dt_warm(const Params &p, const int b, const int dir, const int tier, const int deflt)
{
    if (!p.warm_model) return deflt;
    const int4 w = p.wlen[b];
    return tier == 0 ? w.x : (dir ? w.z : w.y);
}

// Warm-up of the second attempt where the first, of `warm` positions, left the mismatch `worst`.  The mismatch falls
// geometrically, so the length that brings it to 1e-12 follows; a quarter and half a segment length on top for
// stretches that forget more slowly, never less than the default.  What follows overshoots where the mismatch has hardly
// begun to fall (K = 34, C = 12, transitions N(0, 2^2) .. N(0, 3^2): 272 positions suffice where 350 .. 480 follow, 195 -> 280 us a
// call), so eight segment lengths, or twice what was tried, are the most, and what hopeless cases take; the third attempt goes further.
__device__ __forceinline__ int second_warm(const Params &p, const int warm, const double worst)
{
    const double most = p.warm_model ? fmin((double)max(long_warmup(p.K), 2 * warm), (double)p.warm_long) : (double)p.warm_long;
    double w = most;
    if (worst > 0.0 && worst < 0.1) w = fmin(w, 1.25 * (double)warm * (-27.7 / log(worst)) + 0.5 * (double)p.K);
    if (p.warm_model) w = fmax(w, (double)sum_warmup(p.K));
    return ((int)w + 3) & ~3;
}

// The same for the scans with duration-dependent transitions, whose second attempt is the last before the whole sequence is
// scanned: eight segment lengths, or twice a first warm-up that was chosen longer than the default.
__device__ __forceinline__ int last_warm(const Params &p, const int warm)
{
    return warm > sum_warmup(p.K) ? min(max(long_warmup(p.K), 2 * warm), p.warm_long) : long_warmup(p.K);
}
