// Fixed-order reductions of the gradient formulas: per-sequence sums, the emission gradient and the position marginals.
// Included by semicrf.hip inside its anonymous namespace (after common.h); not a translation unit of its own.

// ---------------------------------------------------------------------------
// Finalisation (fixed-order reductions).
// ---------------------------------------------------------------------------
// Positions per partial sum of sequence b: an interval, or a part of one where the one-wave stored-row marginals
// took the sequence (the condition under which that kernel works on it).
__device__ __forceinline__ int stat_delta(const Params &p, const int b)
{
    return (p.msplit > 1 && p.spec_ok[b * 2] && p.spec_ok[b * 2 + 1]) ? p.Delta / p.msplit : p.Delta;
}

// carry[b,i,c] = sum_{i'<=i} tot[b,i',c] and the sums behind mean[b,c] = (1/L) sum_u pm[b,u,c].  FIN_FS workgroups
// per sequence, each a contiguous slice of the sequence's partial sums (it first adds up, label by label, what
// lies before its slice).  Inside a workgroup the partial sums are split into G = NT/C contiguous chunks, one per
// thread group; chunk sums are combined in chunk order, so the result does not depend on the launch shape.
// mean is left as FIN_FS sums per label; k_fin_emis adds them and divides.
constexpr int FIN_FS = FIN_SLICES;
__device__ __forceinline__ void fin_seq_body(const Params &p, const int b, const int s)
{
    __shared__ double gsum[NT];
    __shared__ double gtot[NT];
    const int C = p.C, N = p.NP, tid = threadIdx.x;
    const int L = p.hdr[b].L;
    const int Ds = stat_delta(p, b);
    const int nint = (L + Ds - 1) / Ds;
    const int G = NT / C;
    const int g = tid / C, c = tid % C;
    const bool act = g < G;
    const int per_s = (nint + FIN_FS - 1) / FIN_FS;
    const int s0 = min(s * per_s, nint), s1 = min(s0 + per_s, nint);
    const double *tot = p.tot + ((size_t)b * N) * C + c;
    // what lies before the slice
    {
        const int per = (s0 + G - 1) / G;
        const int a0 = min(g * per, s0), a1 = min(a0 + per, s0);
        double pre = 0.0;
        if (act) {
#pragma unroll 8
            for (int i = a0; i < a1; ++i) pre += tot[(size_t)i * C];
        }
        gsum[tid] = pre;
    }
    __syncthreads();
    double run = 0.0;
    if (act)
        for (int gg = 0; gg < G; ++gg) run += gsum[gg * C + c];
    __syncthreads();
    // the slice
    const int per = (s1 - s0 + G - 1) / G;
    const int i0 = min(s0 + g * per, s1), i1 = min(i0 + per, s1);
    double loc = 0.0;
    if (act) {
#pragma unroll 8
        for (int i = i0; i < i1; ++i) loc += tot[(size_t)i * C];
    }
    gsum[tid] = loc;
    __syncthreads();
    double total = 0.0;
    if (act) {
        for (int gg = 0; gg < g; ++gg) run += gsum[gg * C + c];
#pragma unroll 8
        for (int i = i0; i < i1; ++i) {
            const size_t o = ((size_t)b * N + i) * C + c;
            run += p.tot[o];
            p.carry[o] = run;
            const int n = min(Ds, L - i * Ds);
            total += (double)n * run - p.sumR[o];
        }
    }
    gtot[tid] = total;
    __syncthreads();
    if (tid < C) {
        double t = 0.0;
        for (int gg = 0; gg < G; ++gg) t += gtot[gg * C + tid];
        p.mean[((size_t)b * FIN_FS + s) * C + tid] = t;
    }
    // boundary posterior: certain at both ends of the sequence, nothing beyond it (the interval
    // kernels wrote positions 1 .. L-1)
    if (p.bdy_post && s == 0) {
        float *bd = p.bdy_post + (size_t)b * (p.T + 1);
        if (tid == 0) bd[0] = 1.f;
        for (int t = max(L, 1) + tid; t <= p.T; t += NT) bd[t] = t == L ? 1.f : 0.f;
    }
}

// Gradients of the scalar sequence boundaries: sums over sequences, in sequence order, of the
// mass of the segments that start at position 0 / end at position L.  One workgroup.
__device__ __forceinline__ void fin_pi_body(const Params &p)
{
    const int c = threadIdx.x;
    if (c >= p.C) return;
    double gs = 0.0, ge = 0.0;
    for (int b = 0; b < p.B; ++b) {
        if (p.hdr[b].L < 1) continue;
        const double w = p.grad_logz ? (double)p.grad_logz[b] : 1.0;
        gs = fma(w, p.out0[(size_t)b * p.C + c], gs);
        ge = fma(w, p.inL[(size_t)b * p.C + c], ge);
    }
    if (p.g_pi_start) p.g_pi_start[c] = (float)gs;
    if (p.g_pi_end) p.g_pi_end[c] = (float)ge;
}

// grad_emis / pos_marg, elementwise over (u,c) of one sequence.  grid (blocks, B).
// V = 4: four labels of one position per thread as 16-byte accesses (C a multiple of 4, outputs 16-byte aligned,
// fewer than 2^31 elements per sequence); V = 1: the general form.
template <int V>
__global__ __launch_bounds__(NT) void k_fin_emis(Params p)
{
    const int b = blockIdx.y, C = p.C;
    const int L = p.hdr[b].L;
    const double w = p.grad_logz ? (double)p.grad_logz[b] : 1.0;
    const size_t n = (size_t)p.T * C;  // elements of one sequence
    const size_t base = (size_t)b * n;
    const double *carry = p.carry + ((size_t)b * p.NP) * C;
    const int Ds = stat_delta(p, b);
    __shared__ double mean[GRAD_CMAX];
    if ((int)threadIdx.x < C) {
        double t = 0.0;
        for (int s = 0; s < FIN_FS; ++s) t += p.mean[((size_t)b * FIN_FS + s) * C + threadIdx.x];
        mean[threadIdx.x] = (p.center && L > 0) ? t / (double)L : 0.0;
    }
    __syncthreads();
    if (V == 4) {
        const unsigned Cq = (unsigned)C / 4u, nq = (unsigned)(n / 4), step = gridDim.x * NT;
        float4 *ge4 = (float4 *)(p.grad_emis + base);
        float4 *pm4 = p.pos_marg ? (float4 *)(p.pos_marg + base) : nullptr;
        for (unsigned q = blockIdx.x * NT + threadIdx.x; q < nq; q += step) {
            const unsigned u = q / Cq, c = (q - u * Cq) * 4u;
            float4 ge = make_float4(0.f, 0.f, 0.f, 0.f), pmv = ge;
            if ((int)u < L) {
                const double *cr = carry + (size_t)(u / (unsigned)Ds) * C + c;
                const float4 r = ge4[q];
                const double pm0 = cr[0] - (double)r.x, pm1 = cr[1] - (double)r.y;
                const double pm2 = cr[2] - (double)r.z, pm3 = cr[3] - (double)r.w;
                ge = make_float4((float)(w * (pm0 - mean[c])), (float)(w * (pm1 - mean[c + 1])),
                                 (float)(w * (pm2 - mean[c + 2])), (float)(w * (pm3 - mean[c + 3])));
                pmv = make_float4((float)pm0, (float)pm1, (float)pm2, (float)pm3);
            }
            ge4[q] = ge;
            if (pm4) pm4[q] = pmv;
            if ((int)u >= L - 1) {  // boundary projections, as below
                const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
                if (p.g_proj_start && (int)u >= L) ((float4 *)(p.g_proj_start + base))[q] = zero;
                if (p.g_proj_end) {
                    float4 x = zero;
                    if ((int)u == L - 1) {
                        const double *in = p.inL + (size_t)b * C + c;
                        x = make_float4((float)(w * in[0]), (float)(w * in[1]), (float)(w * in[2]), (float)(w * in[3]));
                    }
                    ((float4 *)(p.g_proj_end + base))[q] = x;
                }
            }
        }
        return;
    }
    auto one = [&](const size_t idx, const int u, const int c) {
        float ge = 0.f, pmv = 0.f;
        if (u < L) {
            const int i = u / Ds;
            const double pm = carry[(size_t)i * C + c] - (double)p.grad_emis[base + idx];
            ge = (float)(w * (pm - mean[c]));
            pmv = (float)pm;
        }
        p.grad_emis[base + idx] = ge;
        if (p.pos_marg) p.pos_marg[base + idx] = pmv;
        // boundary projections: rows beyond the sequence are zero; the last token's end score
        // belongs to the segments that end at position L
        if (p.g_proj_start && u >= L) p.g_proj_start[base + idx] = 0.f;
        if (p.g_proj_end && u >= L - 1)
            p.g_proj_end[base + idx] = u == L - 1 ? (float)(w * p.inL[(size_t)b * C + c]) : 0.f;
    };
    if (n < ((size_t)1 << 31)) {  // 32-bit index arithmetic
        const unsigned n32 = (unsigned)n, step = gridDim.x * NT;
        for (unsigned idx = blockIdx.x * NT + threadIdx.x; idx < n32; idx += step) {
            const unsigned u = idx / (unsigned)C;
            one(idx, (int)u, (int)(idx - u * (unsigned)C));
        }
    } else {
        for (size_t idx = (size_t)blockIdx.x * NT + threadIdx.x; idx < n; idx += (size_t)gridDim.x * NT)
            one(idx, (int)(idx / C), (int)(idx % C));
    }
}

// Launch of k_fin_emis in the form the sizes and outputs allow.
inline void launch_fin_emis(const Params &p, hipStream_t st)
{
    const size_t n = (size_t)p.T * p.C;
    const bool vec = p.C % 4 == 0 && n < ((size_t)1 << 31) &&
                     (((uintptr_t)p.grad_emis | (uintptr_t)p.pos_marg | (uintptr_t)p.g_proj_start |
                       (uintptr_t)p.g_proj_end) & 15) == 0;
    size_t blocks = ((vec ? n / 4 : n) + NT - 1) / NT;
    if (blocks > 16384) blocks = 16384;
    if (vec) hipLaunchKernelGGL(k_fin_emis<4>, dim3((unsigned)blocks, p.B), dim3(NT), 0, st, p);
    else hipLaunchKernelGGL(k_fin_emis<1>, dim3((unsigned)blocks, p.B), dim3(NT), 0, st, p);
}

// grad_trans[c',c] = Etr[c',c] * sum_b w_b sum_i partTr;  grad_dur[k,c] = sum_b w_b sum_i partD.
// One workgroup per FIN_PO outputs; its NT / FIN_PO thread groups take the partial sums of all sequences in turn and
// their sums are combined in group order (fixed order for a given problem).  Sixteen of a group's partial sums are
// requested before the first is added: taken sequence by sequence, a batch of short ones (16 partial sums for 64 groups
// each) cost a memory latency per four sequences with half of the groups idle, 30 us for B = 64, T = 256.
// Outputs are dealt so that neighbouring ones, which share lines, fall to workgroups of one chiplet (blocks go round the
// eight of them).
constexpr int FIN_PO = 4;  // small: the partial sums of a long sequence are many, the outputs few
inline __host__ __device__ int fin_param_blocks(const int K, const int C)
{
    return ((C * C + K * C + FIN_PO - 1) / FIN_PO + 7) & ~7;
}
__device__ __forceinline__ void fin_params_body(const Params &p, const int blk)
{
    __shared__ double red[NT];
    constexpr int NG = NT / FIN_PO, UB = 16;
    const int C = p.C, CC = C * C, KC = p.K * C, N = p.NP, tid = threadIdx.x;
    const int o = tid % FIN_PO, g = tid / FIN_PO;
    const int idx = ((blk & 7) * (fin_param_blocks(p.K, C) >> 3) + (blk >> 3)) * FIN_PO + o;
    const bool ok = idx < CC + KC;
    __shared__ int npart[NT];  // partial sums of the first NT sequences, and their weights
    __shared__ double weight[NT];
    auto count = [&](const int b) {
        const int Ds = stat_delta(p, b);
        return (p.hdr[b].L + Ds - 1) / Ds;
    };
    auto factor = [&](const int b) { return p.grad_logz ? (double)p.grad_logz[b] : 1.0; };
    if (tid < p.B) {
        npart[tid] = count(tid);
        weight[tid] = factor(tid);
    }
    __syncthreads();
    const size_t stride = idx < CC ? (size_t)CC : (size_t)KC;
    const double *q0 = idx < CC ? p.partTr + idx : p.partD + (idx - CC);  // partial sum i of sequence b at (b*N + i)*stride
    double acc = 0.0;
    if (ok) {
        int b = g / N, i = g % N;  // the group's next partial sum
        const int db = NG / N, di = NG % N;
        while (b < p.B) {
            double v[UB], w[UB];
#pragma unroll
            for (int u = 0; u < UB; ++u) {
                v[u] = w[u] = 0.0;
                if (b < p.B && i < (b < NT ? npart[b] : count(b))) {
                    v[u] = q0[((size_t)b * N + i) * stride];
                    w[u] = b < NT ? weight[b] : factor(b);
                }
                b += db;
                i += di;
                if (i >= N) {
                    i -= N;
                    ++b;
                }
            }
#pragma unroll
            for (int u = 0; u < UB; ++u) acc = fma(w[u], v[u], acc);
        }
    }
    red[tid] = acc;
    __syncthreads();
    if (ok && g == 0) {
        double t = 0.0;
        for (int gg = 0; gg < NG; ++gg) t += red[gg * FIN_PO + o];
        if (idx < CC) p.grad_trans[idx] = (float)(t * p.Etr[idx]);
        else p.grad_dur[idx - CC] = (float)t;
    }
}

// One launch for the two independent reductions: FIN_FS workgroups per sequence, the rest
// per FIN_PO parameter gradients.
__global__ __launch_bounds__(NT) void k_fin_seq(Params p)
{
    const int nparam = fin_param_blocks(p.K, p.C);
    const int nseq = p.B * FIN_FS;
    if ((int)blockIdx.x < nseq) fin_seq_body(p, blockIdx.x / FIN_FS, blockIdx.x % FIN_FS);
    else if ((int)blockIdx.x < nseq + nparam) fin_params_body(p, blockIdx.x - nseq);
    else fin_pi_body(p);
}

// Entropies of the posteriors (the paper's boundary-entropy paragraph): per sequence,
//   h_pos = (1/L) sum_{u<L} -sum_c pm[u,c] ln pm[u,c]          (mean per-position label entropy)
//   h_bdy = -sum_{u<L} ph_u ln ph_u,  ph_u = bdy[u] / sum_{u'<L} bdy[u']   (entropy of the normalised
//           segment-start distribution; a segment starts at token u iff a boundary falls at position u)
// One workgroup per sequence; thread partial sums are combined in thread order.
__global__ __launch_bounds__(NT) void k_entropies(const float *pos_marg, const float *bdy_post,
                                                  const int32_t *lengths, int T, int C, float *h_pos,
                                                  float *h_bdy)
{
    __shared__ double red[NT];
    const int b = blockIdx.x, tid = threadIdx.x;
    int L = lengths ? lengths[b] : T;
    L = L < 0 ? 0 : (L > T ? T : L);
    auto block_sum = [&](double v) {
        red[tid] = v;
        __syncthreads();
        double s = 0.0;
        if (tid == 0)
            for (int i = 0; i < NT; ++i) s += red[i];
        __syncthreads();
        if (tid == 0) red[0] = s;
        __syncthreads();
        s = red[0];
        __syncthreads();
        return s;
    };
    if (h_pos) {
        const float *pm = pos_marg + (size_t)b * T * C;
        double acc = 0.0;
        for (size_t i = tid; i < (size_t)L * C; i += NT) {
            const double x = (double)pm[i];
            if (x > 0.0) acc -= x * log(x);
        }
        const double tot = block_sum(acc);
        if (tid == 0) h_pos[b] = L > 0 ? (float)(tot / (double)L) : 0.f;
    }
    if (h_bdy) {
        const float *bd = bdy_post + (size_t)b * (T + 1);
        double acc = 0.0;
        for (int u = tid; u < L; u += NT) acc += (double)bd[u];
        const double norm = block_sum(acc);
        acc = 0.0;
        for (int u = tid; u < L; u += NT) {
            const double x = (double)bd[u] / norm;
            if (x > 0.0) acc -= x * log(x);
        }
        const double tot = block_sum(acc);
        if (tid == 0) h_bdy[b] = L > 0 ? (float)tot : 0.f;
    }
}


// The same with a workspace: any number of workgroups per sequence, ENT_TOK tokens each, and one more launch that adds
// their sums up in token order.  Three sums suffice in one pass over the data: with n = sum bdy,
// h_bdy = log n - (sum bdy log bdy) / n.  Bound by the fp64 log per element; genomic shape (4 x 100 000 x 24):
// 4.53 ms for k_entropies (four workgroups on the whole chip) -> 0.05 ms, and 14 us less with the logarithm below in the
// place of log() (genomic analysis as a whole 684 -> 670 us).
constexpr int ENT_TOK = 512;
// x log x of a float, in 64 bits.  x = 2^e m with m in [sqrt(1/2), sqrt(2)): m has 24 bits, so m - 1 and m + 1 are exact, and
// log m = 2 atanh(s), s = (m - 1) / (m + 1), |s| < 0.1716: the odd series up to s^21 leaves out less than s^23 / 11, 2e-18 of the sum.
// What the quotient's rounding leaves out, the terms from s^3 on and the low part of e ln 2 (its high part has 42 bits, so that
// its product with e is exact) are added up first, so that the logarithm is rounded about once: 1.13e-16 relative at most over
// 20 million floats against 80-bit logarithms (the host's log() 1.11e-16; 2.3e-16 without those parts).
__device__ __forceinline__ double xlogx(const float v)
{
    constexpr double LN2_HIGH = 0x1.62e42fefa38p-1, LN2_REST = 0x1.ef35793c7673p-45;
    const double x = (double)v;
    int e = __builtin_amdgcn_frexp_exp(x);
    double m = __builtin_amdgcn_frexp_mant(x);  // [1/2, 1)
    const bool low = m < 0.70710678118654752;
    m = low ? m + m : m;
    e -= low ? 1 : 0;
    const double n = m - 1.0, d = m + 1.0;
    double r = __builtin_amdgcn_rcp(d);
    r = fma(fma(-d, r, 1.0), r, r);
    r = fma(fma(-d, r, 1.0), r, r);
    double s = n * r;
    s = fma(fma(-d, s, n), r, s);
    const double left = fma(-d, s, n) * r;
    const double z = s * s;
    double q = 1.0 / 21.0;
#pragma unroll
    for (int i = 19; i >= 3; i -= 2) q = fma(q, z, 1.0 / (double)i);
    const double a = (double)e * LN2_HIGH, c = 2.0 * s, h = a + c;  // |a| > |c| or a = 0: c - (h - a) is exact
    const double l = h + ((c - (h - a)) + fma(c * z, q, fma((double)e, LN2_REST, 2.0 * left)));
    return x > 0.0 ? x * (x < INFINITY ? l : x) : 0.0;
}
template <int N>
__device__ __forceinline__ double ent_block_sum(double v, double *red)  // every thread of N; sum in thread 0
{
    for (int off = 32; off; off >>= 1) v += __shfl_down(v, off);
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    double s = 0.0;
    if (threadIdx.x == 0)
        for (int i = 0; i < N / 64; ++i) s += red[i];
    return s;
}

// Sixteen bytes per load, four loads at a time, and six waves per SIMD instead of three at the genomic shape: both launches 38.7 -> 32.5
// us, the arithmetic of 9.6 million logarithms.  A workgroup has as many threads as its ENT_TOK tokens of C marginals keep busy, and no more:
// both launches, us, one number per load and 256 threads | 128 | 256 | 512 threads (launches alone take 15.5):
//   64 x 100 000   C = 1 36 | 33 | 40 | 58; C = 2 46 | 43 | 46 | 62; C = 4 67 | 65 | 66 | 79; C = 6 88 | 86 | 86 | 95
//   1024 x 2000    C = 1 17 | 16 | 18 | 24; C = 4 28 | 34 | 28 | 31; C = 8 43 | 49 | 46 | 43; C = 24 101 | 108 | 96 | 96
//   64 x 20 000    C = 2 16 | 20 | 16 | 17; C = 6 26 | 27 | 24 | 25; C = 8 30 | 32 | 28 | 29; C = 24 69 | 76 | 63 | 63
//   4 x 100 000    C = 8 16 | 16 | 16 | 16; C = 12 20 | 20 | 19 | 19; C = 24 35 | 36 | 31 | 30; C = 64 81 | 81 | 70 | 65
inline int ent_threads(const int C) { return C < 2 ? 128 : (C < 8 ? 256 : 512); }
template <int N>
__global__ __launch_bounds__(N) void k_ent_part(const float *pos_marg, const float *bdy_post, const int32_t *lengths,
                                                int T, int C, int want_pos, int want_bdy, double *part)
{
    __shared__ double red[N / 64];
    const int b = blockIdx.y, tid = threadIdx.x;
    int L = lengths ? lengths[b] : T;
    L = L < 0 ? 0 : (L > T ? T : L);
    const int u0 = blockIdx.x * ENT_TOK, n = min(L - u0, ENT_TOK);  // n <= 0 beyond the sequence: sums are 0
    double a = 0.0, s = 0.0, e = 0.0;
    if (want_pos && n > 0) {
        const float *pm = pos_marg + ((size_t)b * T + u0) * C;
        const int m = n * C, head = min((int)(-((uintptr_t)pm >> 2) & 3), m), body = (m - head) >> 2;  // (4-byte aligned at least)
        const float4 *pm4 = (const float4 *)(pm + head);
#pragma unroll 4
        for (int i = tid; i < body; i += N) {
            const float4 v = pm4[i];
            a -= (xlogx(v.x) + xlogx(v.y)) + (xlogx(v.z) + xlogx(v.w));
        }
        if (tid < head) a -= xlogx(pm[tid]);
        const int tail = head + 4 * body + tid;
        if (tail < m) a -= xlogx(pm[tail]);
    }
    if (want_bdy) {
        const float *bd = bdy_post + (size_t)b * (T + 1) + u0;
        for (int i = tid; i < n; i += N) {
            s += (double)bd[i];
            e += xlogx(bd[i]);
        }
    }
    a = ent_block_sum<N>(a, red);
    s = ent_block_sum<N>(s, red);
    e = ent_block_sum<N>(e, red);
    if (tid == 0) {
        double *o = part + ((size_t)b * gridDim.x + blockIdx.x) * 3;
        o[0] = a;
        o[1] = s;
        o[2] = e;
    }
}

__global__ __launch_bounds__(NT) void k_ent_fin(const double *part, const int32_t *lengths, int T, int npart,
                                                float *h_pos, float *h_bdy)
{
    __shared__ double red[NT / 64];
    const int b = blockIdx.x;
    int L = lengths ? lengths[b] : T;
    L = L < 0 ? 0 : (L > T ? T : L);
    double v[3] = {0.0, 0.0, 0.0};
    for (int i = threadIdx.x; i < npart; i += NT)
#pragma unroll
        for (int j = 0; j < 3; ++j) v[j] += part[((size_t)b * npart + i) * 3 + j];
#pragma unroll
    for (int j = 0; j < 3; ++j) v[j] = ent_block_sum<NT>(v[j], red);
    if (threadIdx.x != 0) return;
    if (h_pos) h_pos[b] = L > 0 ? (float)(v[0] / (double)L) : 0.f;
    // (no mass: no distribution, entropy 0, as k_entropies gives it)
    if (h_bdy) h_bdy[b] = L > 0 && v[1] > 0.0 && v[1] < DBL_MAX ? (float)(log(v[1]) - v[2] / v[1]) : 0.f;
}
