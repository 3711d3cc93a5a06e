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
// WARM_EVERY-th position of log sum_c exp(score - best), sampled by k_colsum).  Models in which a label reaches
// another only over several steps (forbidden transitions) forget more slowly, about in proportion to the steps.
//
// The length only decides how long the scan takes: whether it was enough is checked at every interval boundary
// (k_spec_cmp).  Measured in a replay of the recurrences on 96 random models of C = 3 .. 64, K = 4 .. 512, transitions N(0, s^2),
// s = 0.1 .. 1: the mismatch falls below 1e-10 after 0.6 .. 1.8 times log(1e12) / log(lambda) positions (12 at C = 64, 16 .. 20
// at C = 24, 28 at C = 8, 40 .. 56 at C = 3; 1.5 K before), 0.3 .. 0.8 of that per step where transitions are forbidden.
//
// A longer warm-up than K + (that) is never needed for the windows to agree entry by entry; a shorter one leaves the older
// entries of the window different, in places where they no longer matter.  negl[c] = 1 / (K R), with R the largest ratio of
// the weight of a longer duration to that of a shorter one: an entry below negl[c] times a newer entry of its label adds,
// at every later position, less than 1/K of what the newer one adds there.
// ---------------------------------------------------------------------------
constexpr int WARM_EVERY = 64;      // one position in so many is sampled: one per wave and chunk
constexpr int WARM_TERMS = 16;      // durations that enter lambda (a growth that needs more of them is slow anyway)
constexpr int WARM_PER = 16;        // most window entries per thread of the comparison that ignores negligible ones
constexpr double WARM_NATS = 27.6;  // log(1e12): a hundredth of the bound of the comparison
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

// One workgroup per sequence, next to those of k_prefix; it must not take longer than they do (12 us at two chunks).  So
// everything that comes from memory is requested before anything is done with it, and the transition matrix is worked on in
// LDS by four threads per label.  lds: (PREP_NSEG + 1) C doubles, buf: 2 NT.
__device__ void warm_plan(const Params &p, const int b, double *lds, double *buf)
{
    // buf, one after the other: ranges of durations [3 * NT]; then detours, successors and best successors, [4][64] each
    float *red = (float *)buf, *part = (float *)buf, *best4 = (float *)(buf + 3 * NT / 2);
    unsigned long long *succ = (unsigned long long *)(buf + NT / 2);
    __shared__ double cons[NT / 64];
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
    float tr[NTR], wq[NWR], du[WARM_PER];
#pragma unroll
    for (int i = 0; i < NTR; ++i) tr[i] = i * NT < CC ? t1[min(i * NT + tid, CC - 1)] : 0.f;
#pragma unroll
    for (int i = 0; i < NWR; ++i) {
        const int e = min(i * NT + tid, n * C - 1);
        wq[i] = p.dur[e];
        if (dt) wq[i] += p.trans3[(size_t)(e / C) * CC + e % C * (C + 1)];
    }
    const int G = NT / C, g = tid / C, per = (K + G - 1) / G, k0 = g * per, k1 = g < G ? min(k0 + per, K) : k0;
#pragma unroll
    for (int u = 0; u < WARM_PER; ++u) du[u] = p.dur[(size_t)min(k0 + u, K - 1) * C + tid % C];
    // contrast: of this sequence alone, so that what happens to it does not depend on the others of its batch
    double con = 0.0;
#pragma unroll 8
    for (int i = tid; i < p.NCH; i += NT) con += (double)p.contrast[(size_t)b * p.NCH + i];
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
    } else {
        for (int p0 = 0; p0 < CC; p0 += NT) {
            const int np = min(CC - p0, NT), G3 = NT / np, g3 = tid / np, pr = p0 + tid % np;
            const int per3 = (K + G3 - 1) / G3, q0 = min(g3 * per3, K), q1 = g3 < G3 ? min(q0 + per3, K) : q0;
            float mn = INFINITY, mx = -INFINITY, best = 0.f;
#pragma unroll 16
            for (int k = q0; k < q1; ++k) {
                const float v = p.dur[(size_t)k * C + pr % C] + p.trans3[(size_t)k * CC + pr];
                best = fmaxf(best, v - mn);
                mn = fminf(mn, v);
                mx = fmaxf(mx, v);
            }
            red[tid] = mn;
            red[NT + tid] = mx;
            red[2 * NT + tid] = best;
            __syncthreads();
            if (tid < np) {
                for (int gg = 1; gg < G3; ++gg) {
                    best = fmaxf(best, fmaxf(red[2 * NT + gg * np + tid], red[NT + gg * np + tid] - mn));
                    mn = fminf(mn, red[gg * np + tid]);
                }
                lds[pr] = (double)best;
            }
            __syncthreads();
        }
        if (tid < C) {
            double best = lds[tid];
            for (int o = 1; o < C; ++o) best = fmax(best, lds[o * C + tid]);
            p.negl[(size_t)b * C + tid] = best < 600.f ? exp(-1.001 * (double)best) / (double)K : 0.0;  // (differences are rounded)
        }
        __syncthreads();
    }
#pragma unroll
    for (int i = 0; i < NTR; ++i) {
        const int e = i * NT + tid;
        if (e < CC) tl[e / C * ts + e % C] = tr[i];
    }
    con = wave_sum(con);
    __syncthreads();  // (the ranges above have been read)
    if (lane == 0) cons[wv] = con;
    // ---- detours of a label and its best successor, four threads per label
    const float stay = tl[lc * ts + lc];
    float det = 0.f, mx = -INFINITY;
    const int o0 = wv * ((C + 3) / 4), o1 = min(o0 + (C + 3) / 4, C);
#pragma unroll 4
    for (int o = o0; o < o1; ++o) {
        const float out = tl[lc * ts + o];
        det += o == lc ? 0.f : __expf(out + tl[o * ts + lc] - stay);
        mx = fmaxf(mx, out);
    }
    part[wv * 64 + lane] = det;
    best4[wv * 64 + lane] = mx;
    __syncthreads();
    mx = fmaxf(fmaxf(best4[lane], best4[64 + lane]), fmaxf(best4[128 + lane], best4[192 + lane]));
    unsigned long long reach = 0;  // successors within eight nats of the best one
#pragma unroll 4
    for (int o = o0; o < o1; ++o) reach |= (unsigned long long)(tl[lc * ts + o] > mx - 8.f) << o;
    succ[wv * 64 + lane] = reach;
    __syncthreads();
    float *wl = tl;  // [WARM_TERMS][C], in the place of the transitions
#pragma unroll
    for (int i = 0; i < NWR; ++i)
        if (i * NT + tid < n * C) wl[i * NT + tid] = wq[i];
    __syncthreads();
    if (wv != 0) return;
    con = ((cons[0] + cons[1]) + cons[2]) + cons[3];
    const float r = cnt > 0.0 ? (__expf((float)(con / cnt)) - 1.f) / (float)(C - 1) : 0.f;
    det = ((part[lane] + part[64 + lane]) + part[128 + lane]) + part[192 + lane];
    // ---- growth of the label: y = 1 / lambda
    float y1 = 1.f;
    {
        float w[WARM_TERMS];
#pragma unroll
        for (int k = 0; k < WARM_TERMS; ++k) w[k] = k < n ? __expf(wl[min(k, n - 1) * C + lc] + (dt ? 0.f : stay)) : 0.f;
        const float q = 1.f + r * det;
        float y0 = 0.f;
        for (int it = 0; it < 12; ++it) {
            const float y = 0.5f * (y0 + y1);
            float s0 = 0.f, s1 = 0.f;  // even and odd durations, two chains
#pragma unroll
            for (int k = WARM_TERMS - 2; k >= 0; k -= 2) {
                s0 = fmaf(s0, y * y, w[k]);
                s1 = fmaf(s1, y * y, w[k + 1]);
            }
            if (q * fmaf(s1, y, s0) * y > 1.f) y1 = y;
            else y0 = y;
        }
    }
    double lam = lane < C ? (double)-__logf(y1) : INFINITY;  // log(lambda); 0 where there is no growth
    lam = -wave_max(lam == lam ? -lam : 0.0);
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
    if (lane != 0) return;
    if (p.logpair) {
        // Best score: what decides is how soon all best paths into a window have met, which takes an emission that tells
        // the labels apart and a label change or a split that pays.  In a replay of 8 x 800 and 40 x 150 .. 400 boundaries of
        // random models (C = 3 .. 54, K = 8 .. 423, transitions N(0, s^2), s = 0.1 .. 1) all had met after 32 positions where
        // there are eight labels or more, after 64 but for 2 where there are three or four (2 K before, 128 .. 846).
        // Models out of that range keep that length.
        const int deflt = vit_warmup(K), shrt = C >= 16 ? 40 : (C >= 8 ? 48 : (C >= 5 ? 64 : 96));
        p.wlen[b].x = hops == 1 && favour < 4.f && r > 0.02f ? min(shrt, deflt) : deflt;
        return;
    }
    double wd = (double)sum_warmup(K);
    if (lam > 0.01 && hops < 64) {
        const double m = WARM_NATS / lam;
        const double slow = 0.85 * m * (double)hops;
        // longer than the default only where labels are far apart; sure scores forget faster than the growth of their runs says
        if (hops > 2 && slow > wd) wd = fmin(slow, (double)p.warm_long);
        else wd = fmin(wd, fmax(16.0, fmax(2.0 * m, slow) + 4.0));
    }
    if (!(p.warm_model & WARM_SHORTER)) wd = fmax(wd, (double)sum_warmup(K));
    p.wlen[b] = make_int4(((int)wd + 3) & ~3, p.warm_long, p.warm_long, hops > 2 && wd > (double)sum_warmup(K));
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
// stretches that forget more slowly.  Hopeless cases take eight segment lengths, or twice what was tried.
__device__ __forceinline__ int second_warm(const Params &p, const int warm, const double worst)
{
    double w = (double)max(max(8 * p.K, 64), 2 * warm);
    if (worst > 0.0 && worst < 0.1) w = 1.25 * (double)warm * (-27.7 / log(worst)) + 0.5 * (double)p.K;
    return ((int)fmin(w, (double)p.warm_long) + 3) & ~3;
}
