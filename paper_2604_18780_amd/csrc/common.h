// Declarations shared by the translation units of libsemicrf: sizes, the kernel parameter block,
// small device helpers, and the launchers one unit offers to another.
#ifndef SEMICRF_COMMON_H
#define SEMICRF_COMMON_H

#include <hip/hip_runtime.h>
#include <float.h>
#include <math.h>
#include <stdint.h>
#include <stdlib.h>
#include <type_traits>
#include <utility>

#include "semicrf.h"
#include "geometry.h"
#include "plan.h"

namespace semicrf_impl {

constexpr double LN2 = 0.6931471805599453094;
constexpr double LOG2E = 1.4426950408889634074;
constexpr double RANGE_NATS = 300.0;  // per-position growth that is supported (2x this < ln DBL_MAX)
// What a scaling block of J positions may reach, as a logarithm.  With r the most a position changes a message by and E the
// furthest the centred prefix sum of a label gets from its value at the block's first position:
//   a message of one scan, or the product of a forward and a backward one    e^((J + 1) r)   (each is 1 in sum at its end
//                                                                             of the block; both together cross it once)
//   the same times a prefix factor ES or 1/ES (q, v, a v, q exp(Y + Y'))      e^((J + 1) r + E)
// and no kernel forms anything larger, so that stays below ln DBL_MAX = 709.8 (and above ln DBL_MIN = -708.4).
// E is at most (J - 1) max|f - nu|, but with noisy scores far less: k_colsum measures it (genomic shape, J = 32: 96 nats
// measured, 212 by the bound, next to 33 r = 488; the window is read and written once per block only to be scaled).
constexpr double BLOCK_NATS = 690.0;

constexpr int WARM_LONGER = 1, WARM_SHORTER = 2;  // Params::warm_model

struct SeqHdr {
    int L;          // clamped length
    int J;          // scaling block length (power of two <= JMAX)
    int flags;      // bit 0: scores exceed the supported per-position range
    int pad;
    double logZ;    // from the forward scan
    double logZb;   // from the backward scan (diagnostic: must equal logZ)
};
static_assert(sizeof(SeqHdr) == SEQ_HDR_BYTES, "the plan sizes the header array with SEQ_HDR_BYTES");

struct Params {
    // problem
    const void *emis;   // [B][T][C] float, or 2-byte IEEE half / bfloat16 (emis_type 1 / 2)
    int emis_type;
    const int32_t *lengths;
    const float *trans;
    const float *dur;
    const float *grad_logz;
    // optional boundary terms of Eq. 4 (any of them may be null)
    const float *proj_start;  // [B][T][C]  start score of a segment whose first token is t
    const float *proj_end;    // [B][T][C]  end score of a segment whose last token is t
    const float *pi_start;    // [C]        scalar boundary of the sequence's first segment
    const float *pi_end;      // [C]        scalar boundary of the sequence's last segment
    int B, T, K, C;
    int Delta, N;       // checkpoint interval and intervals per padded sequence
    int NCH;            // prefix-sum chunks per sequence (covers t = 0..T)
    int center;
    int want_grad;
    int nslot;
    // workspace
    SeqHdr *hdr;        // [B]
    double *nu;         // [B][C]
    double *chsum;      // [B][NCH][C] chunk sums, then exclusive chunk offsets
    float2 *chmax;      // [B][NCH] .x = largest |f| (boundary terms added), .y = largest excursion (see k_colsum)
    double *tabmax;     // [ntab][2]: max dur, max trans of each table workgroup's share
    double logKC;       // log(K * C)
    int ntab;           // workgroups that build the tables
    double *W;          // [K][C]
    double *Etr;        // [C][C]
    double2 *EI;        // [B][T+1][C]  .x = ES = exp(S - n ln2), .y = 1/ES
    int *nbase;         // [B][T+1][C] (row j = scaling block j)
    double *ckA;        // [B][N+1][K*C + C]
    double *ckB;        // [B][N+1][K*C + C]
    double *ckYA;       // [B][N+1]
    double *ckYB;       // [B][N+1]
    // chunk-parallel scan: states reached at the END of a chunk (compared with the next
    // chunk's warm-up state), their scales, per-boundary log2 scale ratios and mismatches
    double *ckA2;       // [B][N+1][K*C + C]
    double *ckB2;       // [B][N+1][K*C + C]
    double *ckYA2;      // [B][N+1]
    double *ckYB2;      // [B][N+1]
    double *spec_lr;    // [B][2][N+1]
    double *spec_err;   // [B][2][N+1]
    double *spec_rep;   // [B][2] largest mismatch of the last verification (-1: not attempted), for the report
    int *spec_ok;       // [B][2]  1: the chunk-parallel scan of (sequence, direction) was accepted
    int logpair;        // k_prefix stores the log-domain pair (S + end score, start score - S): Viterbi
    double *vv;         // [B][T+1][C] Viterbi: V_t(c) = best score arriving at position t
    double *vrt;        // [B][C][T+1] Viterbi: r_t(c) = best score leaving position t
    int *vbest;         // [B] Viterbi: label of the last segment
    int *vbp;           // [B][T+1][C] Viterbi back-pointers: (duration << 8) | predecessor label
    int *vpar[2];       // [B][T+1][C] parent node (position * C + label) and its doublings (ping-pong)
    int4 *vtile[2];     // [B][tiles] what the first pass and the retry of the trace-back left of a tile: nodes by which the
                        // path enters and leaves it, start of the segment it leaves by, segments that start in it
    unsigned char *vmark;  // [B][T+1][C] 1: the node lies on the best path
    float *vscore;      // Viterbi outputs
    int32_t *vlabels, *vstarts, *vnseg;
    int spec;           // chunk-parallel scan enabled for this call
    int mscan;          // its tasks may run sixteen at a time in lock step on the matrix cores
    double *sink;       // [1536] target of stores that must be issued but whose value nobody wants
    int spec2;          // chunk-parallel scan tasks with two waves each (tip + helper): 0 where it pays, 1 always, 2 never
    int lowmem;         // low-memory plan: interval at the spacing of Algorithm 1, a few row slots per sequence
    int warm_long;      // longest warm-up length
    int warm_model;     // the first warm-up of a sequence comes from its model and scores (warm_plan): WARM_LONGER if that is
                        // longer than the default, WARM_SHORTER also if it is shorter (windows are then compared by what
                        // their entries can still contribute, and may be incomplete otherwise); 0: always the default
    double *negl;       // [B][C] see warm_plan
    int4 *wlen;         // [B] first warm-up; duration-dependent transitions: warm-ups of the second attempt (forward, backward);
                        // 1 where the first is longer than the default because labels are steps apart
    float *contrast;    // [B][NCH] sum over the sampled positions of a chunk of log sum_c exp(score - largest score)
    int warm0;          // first warm-up length of the chunk-parallel scans asked for by the caller (0 = default)
    int marg_route;     // 0 automatic, 1 marginals from the stored rows of both scans, 2 per-interval recurrence
    int vit_global;     // Viterbi trace-back by pointer doubling over all nodes (test of the fallback route)
    int fuse;           // its forward tasks also store the interval stage's forward rows (one slot per task)
    double *aloc;       // [nslot][Delta][2C]
    double *alocY;      // [nslot][Delta]
    double *bloc;       // [nslot][Delta][2C] backward rows (p_t, v_t) of the chunk-parallel backward tasks
    double *blocY;      // [nslot][Delta]     their scale relative to the interval's upper end
    int bterms;         // the call has boundary terms among its inputs or outputs
    int marg;           // marginals from the stored rows of both scans (no recurrence in the interval stage)
    int msplit;         // parts per interval of the one-wave stored-row marginals; a sequence they handle has its partial
                        // sums per part (index interval*msplit + part), any other per interval (index interval)
    int NP;             // N * msplit: partial sums of a sequence in partD, partTr, tot, sumR, carry
    double *partD;      // [B][NP][K][C]
    double *partTr;     // [B][NP][C][C]
    double *tot;        // [B][NP][C]
    double *sumR;       // [B][NP][C]
    double *carry;      // [B][NP][C]
    double *mean;       // [B][FIN_SLICES][C]  sums behind the per-label mean of the position marginals
    double *out0;       // [B][C]  mass of the segments that start at position 0, per label
    double *inL;        // [B][C]  mass of the segments that end at position L, per label
    // outputs
    double *cum;        // optional [B][T+1][C]
    float *logz;
    float *grad_emis;
    float *grad_trans;
    float *grad_dur;
    float *pos_marg;
    float *g_proj_start;  // optional [B][T][C]
    float *g_proj_end;    // optional [B][T][C]
    float *g_pi_start;    // optional [C]
    float *g_pi_end;      // optional [C]
    float *bdy_post;      // optional [B][T+1]
    // duration-dependent transitions (null / unused otherwise)
    const float *trans3;  // [K][C][C] trans3[k-1][c'][c] in place of trans[c'][c]
    double *G3;           // [K][C][C] exp(dur[k-1,c] + trans3[k-1,c',c])
    double *GF, *GB, *GS; // the same in the operand order of the matrix-core scans (forward, backward, durations 1 .. 3)
    double *dtA;          // [B][T+1][C] forward messages a_t(c), scaled
    double *dtY;          // [B][T+1]    log2 scale of that row relative to its interval's first position
    double *dtV;          // [B][T+1][C] backward messages v_t(c) = b_t(c) ES_t(c), scaled
    double *dtD;          // [B][T+1][C] (mass of the segments that start at t) - (that end at t), scaled
    double *dtYb;         // [B][T+1]    log2 scale of those two rows relative to the interval's upper end
    double *dtMA, *dtMB;  // [B][T+1] factors in [1, 2) of 2^YA / Z and 2^YB (matrix-core marginals; dtMA null otherwise)
    int2 *dtE;            // [B][T+1] their exponents
    double *partG;        // [dt_nwg][K][C][C] per-workgroup sums of the weighted segment marginals
    double *sumG;         // [K][C][C] their fixed-order total
    int dt_nwg;
    float *grad_trans3;   // output [K][C][C]
};

// emission i of the [B][T][C] array; ET = storage type (0 float, 1 IEEE half, 2 bfloat16)
template <int ET>
__device__ __forceinline__ double emis_at(const Params &p, size_t i)
{
    if (ET == 0) return (double)((const float *)p.emis)[i];
    if (ET == 1) return (double)(float)((const _Float16 *)p.emis)[i];
    return (double)__uint_as_float((uint32_t)((const uint16_t *)p.emis)[i] << 16);  // bfloat16: upper half of a float
}

__device__ __forceinline__ int seq_len(const Params &p, int b)
{
    int L = p.lengths ? p.lengths[b] : p.T;
    L = L < 0 ? 0 : L;
    return L > p.T ? p.T : L;
}

__device__ __forceinline__ int safe_exponent(double m)
{
    if (!(m > 0.0) || !(m < DBL_MAX)) return 0;
    int e;
    (void)frexp(m, &e);
    return e;
}

// A whole number of a stored scale, or of a sum of them, as an integer.  Scales are relative to an end of their interval or of the
// sequence: each is as large as what all the positions to there gain (up to 433 bits a position), and only what they add up to lies
// near a double's range.  So the limit is the integers' (met by scores outside the supported range alone), and no part of an exponent
// is cut off before the others are added.
__device__ __forceinline__ int whole_exponent(const double e) { return (int)fmin(fmax(e, -0x1p30), 0x1p30); }

__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// The tip's end-of-step barrier: no s_waitcnt.  The only LDS write of the step that
// other waves read (the ring entry) is not read by them before the NEXT barrier.
__device__ __forceinline__ void tip_step_barrier()
{
    asm volatile("s_barrier" ::: "memory");
}

// orders LDS accesses of one wave (LDS executes a wave's instructions in order)
__device__ __forceinline__ void lds_wave_fence()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// v + (v of the lane 32 away), in every lane: rows 2,3 of one copy are swapped with
// rows 0,1 of the other (a row is 16 lanes), then the copies are added.
__device__ __forceinline__ double add_across_32(double v)
{
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return __hiloint2double((int)b[0], (int)a[0]) + __hiloint2double((int)b[1], (int)a[1]);
}

// A stored row (two doubles) that a later kernel reads once: written past the caches.
__device__ __forceinline__ void store_row(double2 *dst, const double a, const double b)
{
    typedef double d2_t __attribute__((ext_vector_type(2)));
    __builtin_nontemporal_store(d2_t{a, b}, (d2_t *)dst);
}

// Stores of the rows of a block of positions in which some lanes have nothing to store (they own no label, or the block has no
// rows): through a buffer that holds just the block's rows, whose range check drops what lies beyond.  A store under a lane condition
// makes the compiler wait for all loads in flight where the condition ends, and one to a place nobody reads costs its traffic: with
// 40 of 64 lanes on the same kilobyte, 0.5 GB of the genomic shape's scans.
constexpr unsigned ROW_NOWHERE = 0xc0000000u;  // beyond every block
struct RowStore {
    __amdgpu_buffer_rsrc_t rows;
    __device__ __forceinline__ RowStore(void *base, const int bytes)  // base: the same in every lane
        : rows(__builtin_amdgcn_make_buffer_rsrc(base, 0, bytes, 0x00020000)) {}
    __device__ __forceinline__ void pair(const unsigned lane_bytes, const int row_bytes, const double a, const double b) const
    {
        typedef double d2_t __attribute__((ext_vector_type(2)));
        typedef int i4_t __attribute__((ext_vector_type(4)));
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(i4_t, (d2_t{a, b})), rows, (int)lane_bytes, row_bytes, 2);  // non-temporal
    }
    __device__ __forceinline__ void one(const unsigned lane_bytes, const int row_bytes, const double a) const
    {
        typedef int i2_t __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(i2_t, a), rows, (int)lane_bytes, row_bytes, 2);
    }
};

// The value lanes 0..31 hold (-> lo_half) and the one lanes 32..63 hold (-> hi_half), lane l paired with lane
// l + 32, both delivered to both lanes.
__device__ __forceinline__ void both_halves(const double v, double &lo_half, double &hi_half)
{
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    lo_half = __hiloint2double((int)b[0], (int)a[0]);
    hi_half = __hiloint2double((int)b[1], (int)a[1]);
}

// v + (v of the lane 16 away): odd rows of one copy are swapped with even rows of the other
__device__ __forceinline__ double add_across_16(double v)
{
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return __hiloint2double((int)b[0], (int)a[0]) + __hiloint2double((int)b[1], (int)a[1]);
}

// v + (v of the lane 8 away inside a row of 16): DPP row rotate by 8
__device__ __forceinline__ double add_across_8(double v)
{
    const int lo = __double2loint(v), hi = __double2hiint(v);
    const int lo2 = __builtin_amdgcn_update_dpp(0, lo, 0x128, 0xf, 0xf, false);
    const int hi2 = __builtin_amdgcn_update_dpp(0, hi, 0x128, 0xf, 0xf, false);
    return v + __hiloint2double(hi2, lo2);
}

// sum over the 64/CTP lanes of a wave that share lane % CTP; every lane gets the total
template <int CTP>
__device__ __forceinline__ double group_sum(double v)
{
    if (CTP <= 8) v = add_across_8(v);
    if (CTP <= 16) v = add_across_16(v);
    if (CTP <= 32) v = add_across_32(v);
    return v;
}

// ---- products of a message vector with the transition matrix inside one wave, without LDS.
// v_fmac_f64 with the DPP control row_newbcast:n multiplies by the value lane n of the own row of 16 lanes holds, so
// a vector that lies one entry per lane along a row is contracted by one instruction per entry.  (Through LDS, a
// store, six 16-byte broadcast reads and their waits: 250 clocks of a position's chain against 160, and half of the
// scan kernels' LDS traffic.)  The leading s_nop covers the two wait states a DPP read needs after a vector write.
#define SEMICRF_FD(acc, n, op) "v_fmac_f64_dpp %" #acc ", %2, %" #op " row_newbcast:" #n " row_mask:0xf bank_mask:0xf\n\t"
__device__ __forceinline__ void row_dot4(const double y, const double *e, double &z0, double &z1)
{
    asm("s_nop 1\n\t" SEMICRF_FD(0, 0, 3) SEMICRF_FD(1, 1, 4) SEMICRF_FD(0, 2, 5) SEMICRF_FD(1, 3, 6)
        : "+&v"(z0), "+&v"(z1) : "v"(y), "v"(e[0]), "v"(e[1]), "v"(e[2]), "v"(e[3]));
}

__device__ __forceinline__ void row_dot8(const double y, const double *e, double &z0, double &z1)
{
    asm("s_nop 1\n\t" SEMICRF_FD(0, 0, 3) SEMICRF_FD(1, 1, 4) SEMICRF_FD(0, 2, 5) SEMICRF_FD(1, 3, 6)
        SEMICRF_FD(0, 4, 7) SEMICRF_FD(1, 5, 8) SEMICRF_FD(0, 6, 9) SEMICRF_FD(1, 7, 10)
        : "+&v"(z0), "+&v"(z1)
        : "v"(y), "v"(e[0]), "v"(e[1]), "v"(e[2]), "v"(e[3]), "v"(e[4]), "v"(e[5]), "v"(e[6]), "v"(e[7]));
}

__device__ __forceinline__ void row_dot12(const double y, const double *e, double &z0, double &z1)
{
    asm("s_nop 1\n\t" SEMICRF_FD(0, 0, 3) SEMICRF_FD(1, 1, 4) SEMICRF_FD(0, 2, 5) SEMICRF_FD(1, 3, 6)
        SEMICRF_FD(0, 4, 7) SEMICRF_FD(1, 5, 8) SEMICRF_FD(0, 6, 9) SEMICRF_FD(1, 7, 10)
        SEMICRF_FD(0, 8, 11) SEMICRF_FD(1, 9, 12) SEMICRF_FD(0, 10, 13) SEMICRF_FD(1, 11, 14)
        : "+&v"(z0), "+&v"(z1)
        : "v"(y), "v"(e[0]), "v"(e[1]), "v"(e[2]), "v"(e[3]), "v"(e[4]), "v"(e[5]), "v"(e[6]), "v"(e[7]), "v"(e[8]),
          "v"(e[9]), "v"(e[10]), "v"(e[11]));
}

__device__ __forceinline__ void row_dot16(const double y, const double *e, double &z0, double &z1)
{
    asm("s_nop 1\n\t" SEMICRF_FD(0, 0, 3) SEMICRF_FD(1, 1, 4) SEMICRF_FD(0, 2, 5) SEMICRF_FD(1, 3, 6)
        SEMICRF_FD(0, 4, 7) SEMICRF_FD(1, 5, 8) SEMICRF_FD(0, 6, 9) SEMICRF_FD(1, 7, 10)
        SEMICRF_FD(0, 8, 11) SEMICRF_FD(1, 9, 12) SEMICRF_FD(0, 10, 13) SEMICRF_FD(1, 11, 14)
        SEMICRF_FD(0, 12, 15) SEMICRF_FD(1, 13, 16) SEMICRF_FD(0, 14, 17) SEMICRF_FD(1, 15, 18)
        : "+&v"(z0), "+&v"(z1)
        : "v"(y), "v"(e[0]), "v"(e[1]), "v"(e[2]), "v"(e[3]), "v"(e[4]), "v"(e[5]), "v"(e[6]), "v"(e[7]), "v"(e[8]),
          "v"(e[9]), "v"(e[10]), "v"(e[11]), "v"(e[12]), "v"(e[13]), "v"(e[14]), "v"(e[15]));
}
#undef SEMICRF_FD

// the value lane N of the own row of 16 lanes holds
template <int N>
__device__ __forceinline__ double row_bcast(const double v)
{
    return __builtin_amdgcn_update_dpp(v, v, 0x150 + N, 0xf, 0xf, true);
}

// z0, z1 = running maxima of y(n) + e[n] over the even and the odd lanes n of the own row
template <int... I>
__device__ __forceinline__ void row_max(const double y, const double *e, double &z0, double &z1,
                                        std::integer_sequence<int, I...>)
{
    (((I & 1 ? z1 : z0) = fmax(I & 1 ? z1 : z0, row_bcast<I>(y) + e[I])), ...);
}

// the larger of v and the v of the lane 32, 16 or (inside a row of 16) 8 away
__device__ __forceinline__ double max_across_32(double v)
{
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto a = __builtin_amdgcn_permlane32_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane32_swap(hi, hi, false, false);
    return fmax(__hiloint2double((int)b[0], (int)a[0]), __hiloint2double((int)b[1], (int)a[1]));
}

__device__ __forceinline__ double max_across_16(double v)
{
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    return fmax(__hiloint2double((int)b[0], (int)a[0]), __hiloint2double((int)b[1], (int)a[1]));
}

// the larger of v and the v of the lane N places on in the own row of 16 (cyclically)
template <int N>
__device__ __forceinline__ double max_row_ror(double v)
{
    const int lo = __double2loint(v), hi = __double2hiint(v);
    const int lo2 = __builtin_amdgcn_update_dpp(0, lo, 0x120 + N, 0xf, 0xf, false);
    const int hi2 = __builtin_amdgcn_update_dpp(0, hi, 0x120 + N, 0xf, 0xf, false);
    return fmax(v, __hiloint2double(hi2, lo2));
}

// max over the 64/CTP lanes of a wave that share lane % CTP; every lane gets the result
template <int CTP>
__device__ __forceinline__ double group_max(double v)
{
    if (CTP <= 8) v = max_row_ror<8>(v);
    if (CTP <= 16) v = max_across_16(v);
    if (CTP <= 32) v = max_across_32(v);
    return v;
}

template <int N>
__device__ __forceinline__ double add_row_ror(const double v)  // v + the v of the lane N places on in its row of 16
{
    const int lo = __double2loint(v), hi = __double2hiint(v);
    const int lo2 = __builtin_amdgcn_update_dpp(0, lo, 0x120 + N, 0xf, 0xf, true);
    const int hi2 = __builtin_amdgcn_update_dpp(0, hi, 0x120 + N, 0xf, 0xf, true);
    return v + __hiloint2double(hi2, lo2);
}

// sum over the wave, in every lane
__device__ __forceinline__ double wave_sum(const double v)
{
    return add_across_32(add_across_16(add_row_ror<1>(add_row_ror<2>(add_row_ror<4>(add_row_ror<8>(v))))));
}

// max over the wave, in every lane
__device__ __forceinline__ double wave_max(double v)
{
    v = max_row_ror<8>(v);
    v = max_row_ror<4>(v);
    v = max_row_ror<2>(v);
    v = max_row_ror<1>(v);
    return max_across_32(max_across_16(v));
}

// rows 0,2 of v in rows 0,1,2,3 as 0,0,2,2 (-> even) and rows 1,3 as 1,1,3,3 (-> odd)
__device__ __forceinline__ void both_row_parities(const double v, double &even, double &odd)
{
    const unsigned lo = (unsigned)__double2loint(v), hi = (unsigned)__double2hiint(v);
    const auto a = __builtin_amdgcn_permlane16_swap(lo, lo, false, false);
    const auto b = __builtin_amdgcn_permlane16_swap(hi, hi, false, false);
    even = __hiloint2double((int)b[0], (int)a[0]);
    odd = __hiloint2double((int)b[1], (int)a[1]);
}

// Lane organisation of a wave for CT labels and the transition product in it.  Lane -> (label, group): 64 lanes hold
// every label GW times.  Labels lie along rows of 16 lanes: one row holds 16 labels (CT = 16, 32, 64), 12 (CT = 24,
// four lanes idle), or 8 twice (CT = 8).  The matrix column of a lane is split over the two halves of the wave
// (CT <= 32): half h takes the inputs h*HC .. h*HC+HC-1, which must then lie at lanes 0 .. HC-1 of its rows.
template <int CT>
struct RowMap {
    static constexpr int CTP = CT <= 8 ? 8 : (CT <= 16 ? 16 : (CT <= 32 ? 32 : 64));
    static constexpr int H = CT <= 32 ? 2 : 1;
    static constexpr int HC = CT / H;  // inputs per lane
    static __device__ __forceinline__ int label(const int lane)  // labels >= C and idle lanes: not used
    {
        if (CT == 24) {
            const int i = lane & 15;
            return i < 12 ? ((lane >> 4) & 1) * 12 + i : 24 + (i - 12);  // idle lanes: numbers beyond every label
        }
        return lane % CTP;
    }
    static __device__ __forceinline__ int group(const int lane) { return lane / CTP; }

    // y: entry of the vector at the lane's own label, the same in every group.  Returns sum_o y(o) e[o] with e the
    // lane's part of its column: e[i] belongs to input (lane >> 5) * HC + i (CT <= 32), i (CT = 64).
    static __device__ __forceinline__ double product(const double y, const double *e)
    {
        double z0 = 0.0, z1 = 0.0;
        if (CT == 64) {
            double lo, hi, y0, y1, y2, y3;
            both_halves(y, lo, hi);
            both_row_parities(lo, y0, y1);
            both_row_parities(hi, y2, y3);
            row_dot16(y0, e, z0, z1);
            row_dot16(y1, e + 16, z0, z1);
            row_dot16(y2, e + 32, z0, z1);
            row_dot16(y3, e + 48, z0, z1);
            return z0 + z1;
        }
        const double in = half_inputs(y);
        if (CT == 8) row_dot4(in, e, z0, z1);
        else if (CT == 16) row_dot8(in, e, z0, z1);
        else if (CT == 24) row_dot12(in, e, z0, z1);
        else row_dot16(in, e, z0, z1);
        return add_across_32(z0 + z1);
    }

    // max_o (y(o) + e[o]), as product() (lanes and labels alike; an e of -infinity leaves an input out).
    static __device__ __forceinline__ double max_product(const double y, const double *e)
    {
        double z0 = -INFINITY, z1 = -INFINITY;
        if (CT == 64) {
            constexpr std::make_integer_sequence<int, 16> seq;
            double lo, hi, y0, y1, y2, y3;
            both_halves(y, lo, hi);
            both_row_parities(lo, y0, y1);
            both_row_parities(hi, y2, y3);
            row_max(y0, e, z0, z1, seq);
            row_max(y1, e + 16, z0, z1, seq);
            row_max(y2, e + 32, z0, z1, seq);
            row_max(y3, e + 48, z0, z1, seq);
            return fmax(z0, z1);
        }
        row_max(half_inputs(y), e, z0, z1, std::make_integer_sequence<int, HC <= 16 ? HC : 16>());
        return max_across_32(fmax(z0, z1));
    }

    // sum of the vector, the same value in every lane (labels >= C must hold zeros)
    static __device__ __forceinline__ double total(const double y)
    {
        double one[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) one[i] = 1.0;
        double z0 = 0.0, z1 = 0.0;
        if (CT == 64) {
            row_dot16(y, one, z0, z1);
            return add_across_16(add_across_32(z0 + z1));
        }
        const double in = half_inputs(y);
        if (CT == 8) row_dot4(in, one, z0, z1);
        else if (CT == 16) row_dot8(in, one, z0, z1);
        else if (CT == 24) row_dot12(in, one, z0, z1);
        else row_dot16(in, one, z0, z1);
        return add_across_32(z0 + z1);
    }

private:
    // the inputs of the lane's half at lanes 0 .. HC-1 of its row
    static __device__ __forceinline__ double half_inputs(const double y)
    {
        if (CT == 24 || CT == 32) {  // rows hold labels A, B, A, B; the lower half needs A, the upper B
            double even, odd;
            both_row_parities(y, even, odd);
            return (__lane_id() & 32) ? odd : even;
        }
        // every row holds all labels: the upper half's rows are rotated by HC lanes
        constexpr int ROR = 0x120 + (16 - HC);  // row_ror: lane i gets lane (i - n) mod 16, n = 16 - HC
        const int lo = __double2loint(y), hi = __double2hiint(y);
        const int lo2 = __builtin_amdgcn_update_dpp(lo, lo, ROR, 0xc, 0xf, false);
        const int hi2 = __builtin_amdgcn_update_dpp(hi, hi, ROR, 0xc, 0xf, false);
        return __hiloint2double(hi2, lo2);
    }
};

// ---- the lock-step scan on the matrix cores (mscan.hip)
constexpr int MS_JMIN = 16;  // shortest scaling block that kernel handles; shorter ones are left to the one-wave scan
bool mscan_applies(int K, int C, int Delta);
// enqueues the kernel; SEMICRF_OK or SEMICRF_ELAUNCH
int launch_mscan(const Params &p, hipStream_t st, bool both, int warm, int tier);

}  // namespace semicrf_impl

#endif  // SEMICRF_COMMON_H
