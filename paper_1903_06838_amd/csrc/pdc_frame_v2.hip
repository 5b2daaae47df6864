// Persistent frame kernel for gfx950.
//
// One workgroup (8 waves, two workgroups a compute unit) owns a strip of rows
// (which may cross one tile edge) for a range of frames.  A group of L lanes
// holds a bank-row (B pixels of one row) in registers, V values a lane, with
// its dark and 1/gain, which stay there for every frame; only the 2-byte raw
// words stream from HBM.  Per frame:
//   phase 1 (each wave, its own bank-rows): the raw words (loaded a frame
//     ahead) are corrected in registers (Fig. b), every bank-row's lower median
//     is found, exactly, by a bracketing count search (common mode, Fig. c), and
//     Frames2 goes to LDS; the same lanes test their values against the seed
//     threshold and append the seed pixels to a workgroup list;
//   phase 2 (over the pooled seeds): 3x3 local maximum with the raster
//     tie-break, masked 3x3 charge sum, photon count (Fig. e and the charge
//     summing section); hits mark a per-bank-row column bitmap;
//   phase 3 (one wave): staging chunk claim;
//   phase 4: each hit's raster position = bank-row prefix + number of hits
//     left of it in its bank-row (bitmap popcount).
//
// What bounds it: VALU instructions.  On the 10,000-frame CSPAD batch at
// occupancy 0.01 it issues about 6,100 wave instructions per strip-frame of 30
// own rows (the form before this one 8,000: 16 waves of four 16-lane groups,
// values through LDS) and the VALUs are busy about 80 % of the time (66 %);
// the kernel takes 23.7 ms, 38.1 ms before.
// What the two changes behind that give:
//   - few lanes a bank-row: a wave searches 8 (194-pixel banks) or 16 (96)
//     medians at once, so the search's reductions, control and sort, as many
//     instructions as the work on the values, are paid for twice the bank-rows;
//   - a bank-row's values never leave its lanes' registers between the raw
//     words and the seeds, so one wave's medians wait for no other wave's
//     corrections, and the two workgroups of a compute unit fill each other's
//     waits at the barriers.
#include <hip/hip_runtime.h>
#include <math.h>

#include "pdc_device.h"
#include "pdc_exact.h"
#include "pdc_internal.h"

#pragma clang fp contract(off)

namespace pdc {

#ifdef PDC_PHASE_TIMERS
// Tracing build only (PDC_PHASE_TIMERS): shader-clock cycles each wave spends
// in each phase of the persistent kernel's frame loop, summed over the launch:
// [wave][0 A, 1 wait at barrier 1, 2 medians, 3 seeds, 4 wait at barrier 2,
// 5 local maxima, 6 hit writes, 7 unused].
__device__ unsigned long long g_phase_cycles[kV2Waves * 8];
#endif


// Number of set bits of m below this lane.
__device__ __forceinline__ int mbcnt(uint64_t m)
{
    return (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0));
}

// Workgroup barrier for LDS only: it waits for the wave's own LDS accesses,
// while its global loads (the next frame's words) and stores stay in flight.
// Nothing a wave writes to global memory inside the frame loop is read by
// another wave of the workgroup.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Orders this wave's LDS accesses before the ones that follow, without
// waiting for its global loads (a wave's LDS instructions complete in order;
// the compiler must not move them across).
__device__ __forceinline__ void wave_lds_order()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// Inclusive prefix sum over the 64 lanes (DPP row shifts, then row
// broadcasts); all lanes must be active.
__device__ __forceinline__ uint32_t wave_incl_scan(uint32_t x)
{
    int v = (int)x;
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);  // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);  // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);  // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);  // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false); // row_bcast:15
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false); // row_bcast:31
    return (uint32_t)v;
}

// Group reductions over aligned groups of L lanes (L = 2, 4, 8 or 16; the
// groups lie inside 16-lane DPP rows).  Every lane of a group receives the
// group's result.  All lanes of the wave must be active.
template <int L>
__device__ __forceinline__ int gsum_i(int v)
{
    v += __builtin_amdgcn_update_dpp(0, v, 0xB1, 0xF, 0xF, false);                // quad_perm 1,0,3,2
    if (L >= 4) v += __builtin_amdgcn_update_dpp(0, v, 0x4E, 0xF, 0xF, false);    // quad_perm 2,3,0,1
    if (L >= 8) v += __builtin_amdgcn_update_dpp(0, v, 0x141, 0xF, 0xF, false);   // row_half_mirror
    if (L >= 16) v += __builtin_amdgcn_update_dpp(0, v, 0x140, 0xF, 0xF, false);  // row_mirror
    return v;
}

template <int L>
__device__ __forceinline__ float gsum_f(float x)
{
#define PDC_GS(ctrl) x += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), ctrl, 0xF, 0xF, false))
    PDC_GS(0xB1);
    if (L >= 4) PDC_GS(0x4E);
    if (L >= 8) PDC_GS(0x141);
    if (L >= 16) PDC_GS(0x140);
#undef PDC_GS
    return x;
}

// Mask of the lane's values below p: bit v is set when x[v] < p.  For finite
// p, x < p exactly when fl(x - p) has its sign bit set (a nonzero difference
// never rounds to +0, x == p gives +0, x = +inf gives +inf); p is clamped to
// the finite range, which changes no answer because the values are bounded far
// below FLT_MAX.  Each value costs a subtraction and an alignbit that shifts
// its sign bit in; the count is one popcount of the mask.
template <int V>
__device__ __forceinline__ uint32_t lane_mask(const float (&x)[V], float p)
{
    const float pc = __builtin_amdgcn_fmed3f(p, -3.40282347e38f, 3.40282347e38f);
    uint32_t m = 0;
#pragma unroll
    for (int v = V - 1; v >= 0; --v) m = __builtin_amdgcn_alignbit(m, __float_as_uint(__fsub_rn(x[v], pc)), 31);
    return m;
}

// [lo, hi) holds a single float (adjacent keys, both bounds finite or not).
__device__ __forceinline__ bool done_single(float lo, float hi)
{
    return (uint32_t)(f2key(hi) - f2key(lo)) <= 1u;
}

// Rough location of an L-lane group's median: medians of three of each lane's
// values (up to eight triples, of columns far apart: a photon's cloud covers
// neighbours), averaged over the group.  Dense banks (no +inf
// inside the first B columns) take the triples that every lane holds; with
// invalid pixels (SPARSE) each lane takes the finite ones.  Only the work of
// the searches below depends on it, never their result.
template <int V, int L, bool SPARSE>
__device__ __forceinline__ float group_estimate(const float (&x)[V], bool full)
{
    static_assert(V >= 3, "the start estimate takes triples of values per lane");
    constexpr int NT = V / 3 < 8 ? V / 3 : 8;
    if (!SPARSE && full) {  // uniform: every lane's NT triples lie inside the bank
        float s3 = __builtin_amdgcn_fmed3f(x[0], x[NT], x[2 * NT]);
#pragma unroll
        for (int t = 1; t < NT; ++t) s3 += __builtin_amdgcn_fmed3f(x[t], x[t + NT], x[t + 2 * NT]);
        return gsum_f<L>(s3) * (1.0f / (float)(NT * L));
    }
    float s3 = 0.0f;
    int n3 = 0;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        const float a = x[t];
        const float b = x[t + NT] < INFINITY ? x[t + NT] : a;
        const float c = x[t + 2 * NT] < INFINITY ? x[t + 2 * NT] : b;
        if (a < INFINITY) {
            s3 += __builtin_amdgcn_fmed3f(a, b, c);
            ++n3;
        }
    }
    const float ssum = gsum_f<L>(s3);
    const int nl = gsum_i<L>(n3);
    return nl > 0 ? ssum * __builtin_amdgcn_rcpf((float)nl) : 0.0f;
}

// The sides of the compare-exchanges below: e[j] is -inf for a lane whose
// bit j of its place in the group is clear (it keeps the smaller value of a
// pair) and +inf otherwise.  Made once per kernel and kept in registers (an
// opaque copy, so that the compiler does not recompute them per use).
template <int L>
struct SortSides {
    static constexpr int N = L == 4 ? 2 : (L == 8 ? 3 : 4);
    float e[N];
};

template <int L>
__device__ __forceinline__ SortSides<L> sort_sides()
{
    const int gl = __lane_id() & (L - 1);
    SortSides<L> sd;
#pragma unroll
    for (int j = 0; j < SortSides<L>::N; ++j) {
        sd.e[j] = (gl >> j) & 1 ? INFINITY : -INFINITY;
        asm volatile("" : "+v"(sd.e[j]));
    }
    return sd;
}

template <int CTRL>
__device__ __forceinline__ float dpp_f(float x)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(x), CTRL, 0xF, 0xF, false));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kMirror4 = 0x1B, kMirror8 = 0x141, kMirror16 = 0x140;

// Compare-exchange of every register with the same (REV: the mirrored)
// register of the partner lane: a median of three with the lane's side keeps
// the smaller or the larger value (no NaN is present).
template <int S, int CTRL, bool REV>
__device__ __forceinline__ void cx_lanes(float (&y)[S], float e)
{
    float p[S];
#pragma unroll
    for (int s = 0; s < S; ++s) p[s] = dpp_f<CTRL>(y[REV ? S - 1 - s : s]);
#pragma unroll
    for (int s = 0; s < S; ++s) y[s] = __builtin_amdgcn_fmed3f(y[s], p[s], e);
}
// Compare-exchange of registers a < b of one lane.
__device__ __forceinline__ void cx_regs(float &a, float &b)
{
    float lo, hi;
    asm("v_min_f32 %0, %1, %2" : "=v"(lo) : "v"(a), "v"(b));
    asm("v_max_f32 %0, %1, %2" : "=v"(hi) : "v"(a), "v"(b));
    a = lo;
    b = hi;
}
// The rest of a merge inside a lane: half-cleaners of distances S/2 .. 1, for
// S = 3 (the half-cleaners across lanes split any even length) a sort.
template <int S>
__device__ __forceinline__ void cx_inner(float (&y)[S])
{
    if constexpr (S == 4) {
        cx_regs(y[0], y[2]);
        cx_regs(y[1], y[3]);
        cx_regs(y[0], y[1]);
        cx_regs(y[2], y[3]);
    } else if constexpr (S == 3) {
        cx_regs(y[0], y[1]);
        cx_regs(y[1], y[2]);
        cx_regs(y[0], y[1]);
    } else {
        cx_regs(y[0], y[1]);
    }
}

// Ascending bitonic sort of the S L values of an aligned L-lane group (value
// j in register j % S of lane j / S), then value r (group-uniform) broadcast
// to the group.  Merges start with the mirror partner inside the block, then
// halve with xor partners.  The pick is an OR over the group of the chosen
// lane's bits and zeros elsewhere.  All lanes must be active.
template <int L, int S>
__device__ __forceinline__ float group_sort_pick(float (&y)[S], int r, const SortSides<L> &sd)
{
    static_assert((S == 2 || S == 3 || S == 4) && (L == 4 || L == 8 || L == 16), "compiled layouts");
    const int gl = __lane_id() & (L - 1);
    if constexpr (S == 4) {
        cx_regs(y[0], y[1]);
        cx_regs(y[2], y[3]);
        cx_regs(y[0], y[3]);
        cx_regs(y[1], y[2]);
        cx_regs(y[0], y[1]);
        cx_regs(y[2], y[3]);
    } else {
        cx_inner(y);
    }
    cx_lanes<S, kXor1, true>(y, sd.e[0]);  // merge across 2 lanes
    cx_inner(y);
    cx_lanes<S, kMirror4, true>(y, sd.e[1]);  // across 4
    cx_lanes<S, kXor1, false>(y, sd.e[0]);
    cx_inner(y);
    if constexpr (L >= 8) {
        cx_lanes<S, kMirror8, true>(y, sd.e[2]);
        cx_lanes<S, kXor2, false>(y, sd.e[1]);
        cx_lanes<S, kXor1, false>(y, sd.e[0]);
        cx_inner(y);
    }
    if constexpr (L >= 16) {
        cx_lanes<S, kMirror16, true>(y, sd.e[3]);
        // xor 4 = xor 3 (quad mirror) then xor 7 (half-row mirror)
        float p[S];
#pragma unroll
        for (int s = 0; s < S; ++s) p[s] = dpp_f<kMirror8>(dpp_f<kMirror4>(y[s]));
#pragma unroll
        for (int s = 0; s < S; ++s) y[s] = __builtin_amdgcn_fmed3f(y[s], p[s], sd.e[2]);
        cx_lanes<S, kXor2, false>(y, sd.e[1]);
        cx_lanes<S, kXor1, false>(y, sd.e[0]);
        cx_inner(y);
    }
    // value r is register r - S (r / S) of lane r / S (r < S L <= 32, or group-
    // uniform rubbish that no lane picks)
    const int rl = S == 3 ? (r * 43) >> 7 : r / S;
    float z = y[0];
#pragma unroll
    for (int s = 1; s < S; ++s) z = r - S * rl == s ? y[s] : z;
    int rb = gl == rl ? __float_as_int(z) : 0;
#define PDC_GX(ctrl) rb |= __builtin_amdgcn_update_dpp(0, rb, ctrl, 0xF, 0xF, false);
    PDC_GX(kXor1)
    PDC_GX(kXor2)
    if (L >= 8) PDC_GX(kMirror8)
    if (L >= 16) PDC_GX(kMirror16)
#undef PDC_GX
    return __int_as_float(rb);
}

// Slot v of a lane: offset from the lane's first column of its bank-row (the
// first 8 Q slots are chunks of 8 columns, 8 L apart; the R after them single
// columns, L apart, from column 8 L Q + gl).
template <int L, int Q, int R>
__device__ __forceinline__ int slot_off(int v, int gl)
{
    const int o = v + (v & ~7) * (L - 1);
    if (R == 0) return o;
    return v < 8 * Q ? o : 8 * L * Q - 7 * gl + L * (v - 8 * Q);
}

// Exact element of rank k (0-based, ascending) among the nval finite values
// held by an L-lane group (V = 8 Q + R values per lane, absent values +inf,
// slot v also at src[slot_off(v)] in LDS); every group of the wave searches
// its own bank at once.  Bracketing search on counts, count(x < lo) <= k <
// count(x < hi) throughout, with the lane masks of both bounds kept: the first
// bracket is the estimate and a bound placed from its count (widening until
// they bracket), later steps interpolate the pivot from the bracket counts and
// bisect in key space when the interpolated pivot is not strictly inside or
// the bracket stopped halving.  Once at most S L values remain in [lo, hi)
// (the lane's are the bits of mhi & ~mlo) they are gathered from LDS into the
// group's lanes, S a lane, sorted across them, and the answer is read off; a
// bracket that holds a single float (possibly many copies of it) gives that
// float.  Groups with act false return an unspecified value.  gsc: the
// group's S L floats of LDS scratch.
//
// S and the margin of the second bound.  The work of a step is paid by the
// whole wave while any of its 64 / L groups needs it, so the bracket that is
// left to the sort is wide enough that few groups miss it or overfill it.  Counts
// beyond the first two, a wave, in a model of this search at occupancy 0.01:
// CSPAD's 194 columns on 8 lanes 0.83 with 16 values left to the sort, 0.29 with
// 24 and a margin of 6 ranks (4: 0.37, 7: 0.33), 0.14 with 32 and 7 (a longer
// sort for every wave; margins of 5 to 10 measured within 0.5 %); 96 columns on 4
// lanes 0.73 with 16 and 4 (3: 0.76, 5: 0.80), where more values would cost
// registers in the sort; 256 columns on 16 lanes 0.09 with 32 and 7.
template <int L, int Q, int R, int S, bool SPARSE>
__device__ __forceinline__ float group_median(const float (&x)[8 * Q + R], const float *src, int nval, int k, float rw,
                                              bool act, float *gsc, bool full, const SortSides<L> &sd)
{
    constexpr int V = 8 * Q + R, CAP = S * L, MARGIN = CAP >= 32 ? 7 : (CAP >= 24 ? 6 : 4);
    const float est = group_estimate<V, L, SPARSE>(x, full);

    // First bracket in two counts: the count below the estimate gives its
    // rank error e, and the second bound goes e + MARGIN rank widths beyond it
    // on the side of rank k
    float lo, hi;
    uint32_t mlo, mhi;
    int clo, chi;
    {
        const uint32_t m1 = lane_mask<V>(x, est);
        const int c1 = gsum_i<L>(__popc(m1));
        const bool up = c1 <= k;  // rank k lies at or above the estimate
        const float d = (float)((up ? k + 1 - c1 : c1 - k) + MARGIN) * rw;
        const float p2 = up ? est + d : est - d;
        const uint32_t m2 = lane_mask<V>(x, p2);
        const int c2 = gsum_i<L>(__popc(m2));
        lo = up ? est : p2;
        hi = up ? p2 : est;
        mlo = up ? m1 : m2;
        mhi = up ? m2 : m1;
        clo = up ? c1 : c2;
        chi = up ? c2 : c1;
    }
    bool ok = !act || (clo <= k && k < chi);
    // widening: a start bracket that misses by m ranks moves its violated
    // bound (m + 3) rank widths beyond, doubling the step on repeated misses
    float sc = rw;
    for (int it = 0; it < 40; ++it) {
        if (__ballot(!ok) == 0) break;
        const bool down = clo > k;
        const float d = (float)((down ? clo - k : k + 1 - chi) + 3) * sc;
        sc = sc + sc;
        const float p = it < 38 ? (down ? lo - d : hi + d) : (down ? -INFINITY : INFINITY);
        const uint32_t mp = lane_mask<V>(x, p);
        const int cp = gsum_i<L>(__popc(mp));
        if (!ok) {
            if (down) {
                hi = lo;
                chi = clo;
                mhi = mlo;
                lo = p;
                clo = cp;
                mlo = mp;
            } else {
                lo = hi;
                clo = chi;
                mlo = mhi;
                hi = p;
                chi = cp;
                mhi = mp;
            }
            ok = clo <= k && k < chi;
        }
    }

    int last_n = 4 * nval;
    bool done = !act || chi - clo <= CAP;
    for (int it = 0; it < 200; ++it) {
        if (__ballot(!done) == 0) break;
        const int n = chi - clo;
        float q = lo + (hi - lo) * (((float)(k - clo) + 0.5f) * __builtin_amdgcn_rcpf((float)n));
        // q is NaN or not strictly inside when a bound is infinite
        const bool interp = 2 * n <= last_n && q > lo && q < hi;
        bool single = false;  // [lo, hi) holds one float only (never when interp holds)
        if (!interp) {
            // bisect in key space: at most 32 such steps reach a bracket that
            // holds a single float, whatever the scale (a value-space midpoint
            // would halve a bracket [0, h) through the whole exponent range)
            const int32_t klo = f2key(lo), khi = f2key(hi);
            single = (uint32_t)(khi - klo) <= 1u;
            q = key2f((klo >> 1) + (khi >> 1) + (klo & khi & 1));
        }
        done = done || single;
        last_n = interp ? n : 4 * nval;
        const uint32_t mq = lane_mask<V>(x, q);
        const int cq = gsum_i<L>(__popc(mq));
        if (!done) {
            if (cq <= k) {
                lo = q;
                clo = cq;
                mlo = mq;
            } else {
                hi = q;
                chi = cq;
                mhi = mq;
            }
            done = chi - clo <= CAP;
        }
    }
    // Finish: the n <= S L values in [lo, hi) are gathered from LDS into the
    // group's lanes (in lane order), sorted across them, and value k - clo is
    // the answer.  A bracket that holds a single float (n > S L possible) has
    // the answer lo.
    const int gl = __lane_id() & (L - 1);
    const int n = chi - clo;
    const bool gather = n <= CAP && !done_single(lo, hi);
    uint32_t cm = gather ? mhi & ~mlo : 0u;
    const int c = __popc(cm);
    int incl = c;
    // (a shift from outside the 16-lane row reads 0, so with L = 16 the
    // group edge needs no test)
#define PDC_SCAN(ctrl, sh)                                                                       \
    {                                                                                            \
        const int o = __builtin_amdgcn_update_dpp(0, incl, ctrl, 0xF, 0xF, true);                 \
        incl += (L == 16 || gl >= sh) ? o : 0;                                                   \
    }
    PDC_SCAN(0x111, 1)
    PDC_SCAN(0x112, 2)
    if (L >= 8) PDC_SCAN(0x114, 4)
    if (L >= 16) PDC_SCAN(0x118, 8)
#undef PDC_SCAN
    float *dst = gsc + (incl - c);
    while (cm) {
        // two at a time, both read before either is stored
        const int v0 = __builtin_ctz(cm);
        cm &= cm - 1u;
        const bool two = cm != 0;
        const int v1 = two ? __builtin_ctz(cm) : v0;
        cm &= cm - 1u;
        const float t0 = src[slot_off<L, Q, R>(v0, gl)], t1 = src[slot_off<L, Q, R>(v1, gl)];
        dst[0] = t0;
        if (two) dst[1] = t1;
        dst += 2;
    }
    wave_lds_order();
    float y[S];
#pragma unroll
    for (int s = 0; s < S; ++s) y[s] = gsc[S * gl + s];
#pragma unroll
    for (int s = 0; s < S; ++s) y[s] = (gather && S * gl + s < n) ? y[s] : INFINITY;
    wave_lds_order();
    // exactly one value of the group (k - clo < n <= S L) is the answer
    const float pick = group_sort_pick<L, S>(y, k - clo, sd);
    return gather ? pick : lo;
}

struct V2Layout {
    uint32_t v, bits, cnt, seed, hl, hl_stride, nseed, hcnt, total;  // float offsets
};

// LDS of one workgroup (floats).  v holds one frame (Frames1 while a wave
// searches its medians, then Frames2); the hit lists
// (charge and strip position of each local maximum), bitmaps and counts are
// double-buffered by frame parity, the seed counts kept for four frames (frame
// mod 4).  Seeds and hits name their pixel by its position in the strip's
// loaded rows (16 bits).  The median finish scratch (4 to 8 KiB) lies in the
// hit list of the frame's own parity, which is not in use then.
__device__ __host__ __forceinline__ V2Layout v2_layout(int rmax, int W, int B, int nb, int seed_cap, int hit_cap)
{
    V2Layout L;
    // W + 1 floats before v: phase 2 reads a seed's neighbours at fixed
    // offsets from the row above, column left, without clamping (what lies
    // outside the rows or the tile is read and then masked)
    uint32_t o = ((uint32_t)W + 4u) & ~3u;
    L.v = o;
    o += (uint32_t)rmax * W;
    L.bits = o;
    o += 2u * rmax * nb * ((uint32_t)(B + 31) / 32u);
    L.cnt = o;
    o += 2u * rmax * nb;
    L.nseed = o;
    o += 4;
    L.hcnt = o;
    o += 2;
    L.seed = o;
    o += ((uint32_t)seed_cap + 1u) / 2u;
    o = (o + 3u) & ~3u;
    L.hl = o;
    // per parity: hit_cap charges, then hit_cap 16-bit positions
    L.hl_stride = ((uint32_t)hit_cap + ((uint32_t)hit_cap + 1u) / 2u + 3u) & ~3u;
    o += 2u * L.hl_stride;
    L.total = o;
    return L;
}

size_t frame_kernel_v2_lds_bytes(int rmax, int W, int B, int nb, int seed_cap, int hit_cap)
{
    return (size_t)v2_layout(rmax, W, B, nb, seed_cap, hit_cap).total * 4;
}

// Item (frame group, strip) of block b among n: blocks are dealt to the 8 XCDs
// round-robin (block b to XCD b mod 8) and the items, in raster order, go to
// the blocks of one XCD after another, so neighbouring strips (which share halo
// rows) share an L2.
__device__ __forceinline__ int block_item(int b, int n)
{
    const int x = b & 7;
    int before = 0;
    for (int y = 0; y < x; ++y) before += (n - y + 7) >> 3;  // blocks of XCD y
    return before + (b >> 3);
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
// raw words are read, and u written, at 4- and 8-byte alignment (a bank of an
// even width starts at an even column), with an odd width at 2 and 4 bytes
// (structs: an alignment on a typedef is lost where the type is a template
// argument; 16-byte LDS stores at 8-byte alignment cost more than pairs of 8:
// 10,000 CSPAD frames 29.4 ms against 25.9, while at 16-byte alignment they are
// the better ones: three mixed detectors' 1,000 frames 2.60 ms against 2.70)
template <int A>
struct __attribute__((packed, aligned(A))) Raw4 {
    u32x4 v;
};
template <int A>
struct __attribute__((packed, aligned(A))) Val4 {
    f32x4 v;
};
typedef uint32_t u32_a2 __attribute__((aligned(2)));

// Values a lane holds in the finish of the medians (a group sorts S L).
template <int L>
constexpr int kV2Finish = L == 4 ? 4 : (L == 8 ? 3 : 2);

// Bank-rows a lane group takes one after another in a frame (PP).  256-column
// banks need 16 lanes for four waves per SIMD (128 registers), and two passes
// keep their strips as high as the others' (a strip loads two halo rows).  So do
// banks of 97 to 128 columns where a row holds many of them (v2_layout_of).
// (Banks of 257 to 512 columns: 32 columns a lane, one pass, half the waves.)
template <int L, int Q>
constexpr int kV2Passes = L == 16 && Q == 2 ? 2 : 1;

// The launch's arguments, read from the argument memory (scalar loads, cached).
// fresh() makes the fields read through it come from there at that place: read
// once ahead of the frame loop they would need more scalar registers than a
// wave has, and the compiler keeps the overflow in vector-register lanes, a
// VALU instruction a reload.
typedef const __attribute__((address_space(4))) V2Args *V2ArgsK;
__device__ __forceinline__ V2ArgsK fresh(V2ArgsK a)
{
    asm volatile("" : "+s"(a));
    return a;
}

// One workgroup's work: work item `item` of the launch over A's strips and
// frame groups (strip item % n_strips, frame group item / n_strips).  ODD: banks
// of an odd width, whose last column has no partner.
template <int L, int Q, int R, bool KEEP, int CMM, bool MG, bool ODD = false, int P = kV2Passes<L, Q>>
__device__ __forceinline__ void frame_body(const V2ArgsK A, const int item)
{
    constexpr int V = 8 * Q + R, G = 64 / L, S = kV2Finish<L>;
    constexpr int kCntRegs = (kV2Threads / L * P + 63) / 64;  // bank-rows of a workgroup, 64 a register
    constexpr int kBitWords = (8 * L * Q + L * R + 31) / 32;  // of the widest bank of this layout
    static_assert(V <= 32, "a lane's values are bits of one mask");
    using raw4 = Raw4<ODD ? 2 : 4>;
    // (without single slots a full bank is 8 L Q columns, so every bank starts
    // at a multiple of 4 floats: 16-byte LDS stores)
    using val4 = Val4<ODD ? 4 : (R == 0 ? 16 : 8)>;
    extern __shared__ __align__(16) float lds[];
#ifdef PDC_PHASE_TIMERS
    __shared__ unsigned long long s_tm[kV2Waves * 8];
    if (threadIdx.x < kV2Waves * 8) s_tm[threadIdx.x] = 0;
#endif
    __shared__ unsigned long long s_photons;
    __shared__ uint64_t s_base;
    __shared__ uint64_t s_chunk[2];  // staging chunk in use: next free entry, end

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int W = A->W, B = A->B, nb = A->nb, H = A->H;
    const V2Layout Ly = v2_layout(A->rmax, W, B, nb, A->seed_cap, A->hit_cap);
    const int RN = A->rmax * nb, cap = A->seed_cap, hcap = A->hit_cap, bw = (B + 31) / 32;
    float *s_v = lds + Ly.v;
    uint32_t *s_bits = reinterpret_cast<uint32_t *>(lds + Ly.bits);
    uint32_t *s_cnt = reinterpret_cast<uint32_t *>(lds + Ly.cnt);
    uint16_t *s_seed = reinterpret_cast<uint16_t *>(lds + Ly.seed);
    uint32_t *s_hcnt = reinterpret_cast<uint32_t *>(lds + Ly.hcnt);
    uint32_t *s_nseed = reinterpret_cast<uint32_t *>(lds + Ly.nseed);

    const int strip = item % A->n_strips;
    const int fg = item / A->n_strips;
    const V2Strip St = A->strips[strip];
    const int lr0 = St.lg0;  // global rows
    const int nrow = St.lg1 - lr0;
    const int own_lo = St.g0 - lr0, own_hi = St.g1 - lr0;
    const int bnd = St.gb == INT32_MAX ? nrow : St.gb - lr0;  // loaded row where a second tile starts
    const int BR = nrow * nb;
    const uint64_t npix = (uint64_t)A->T * H * W;
    // (n_frames <= 2^31)
    const uint32_t f_begin = (uint32_t)((A->n_frames * (uint64_t)fg) / A->n_fgroups);
    const uint32_t f_end = (uint32_t)((A->n_frames * (uint64_t)(fg + 1)) / A->n_fgroups);
    const uint32_t row_base = (uint32_t)lr0 * (uint32_t)W;  // pixel index of loaded row 0
    constexpr int kP3Wave = kV2Waves / 2;  // wave that runs phase 3 (few of phases 2 and 4's chunks fall to it)

    // Lane constants.  Bank-row i = (p kV2Waves + wave) G + lane / L belongs to
    // the lane's group in pass p of P; lane gl of the group holds, in slots
    // 8 c + s (c < Q), columns 8 (gl + L c) + s and, in slots 8 Q + r, columns
    // 8 L Q + L r + gl.  A group past the last bank-row repeats bank-row 0 and
    // stores nothing.  o4: strip position of slot 0; vmask: the slots inside
    // the bank.
    const SortSides<L> sides = sort_sides<L>();  // the bank-median finish's sort
    const int gl = lane & (L - 1);
    const bool full = B >= 8 * L * Q;  // (uniform) only the R single slots may lie past the bank
    uint32_t vmask = 0;
#pragma unroll
    for (int v = 0; v < V; ++v)
        if (8 * gl + slot_off<L, Q, R>(v, gl) < B) vmask |= 1u << v;
    int mi_[P], o4_[P], own_[P];
    bool wave_on[P];  // (uniform) the wave has a bank-row in this pass
#pragma unroll
    for (int p = 0; p < P; ++p) {
        mi_[p] = (p * kV2Waves + wave) * G + lane / L;
        wave_on[p] = (p * kV2Waves + wave) * G < BR;
        const bool act = mi_[p] < BR;
        const int row = act ? mi_[p] / nb : 0;
        o4_[p] = (act ? mi_[p] : 0) * B + 8 * gl;  // bank-rows follow one another
        own_[p] = act && row >= own_lo && row < own_hi ? 1 : 0;
        // opaque copies: kept in registers rather than recomputed per frame
        asm volatile("" : "+v"(mi_[p]), "+v"(o4_[p]), "+v"(own_[p]));
    }
    asm volatile("" : "+v"(vmask));

    // resident calibration of the lane's pixels
    float pd[P][V], kk[P][V];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const float *const pp = A->ped + row_base + (uint32_t)o4_[p], *const kp = A->k + row_base + (uint32_t)o4_[p];
        const bool quads = wave_on[p] && full;
#pragma unroll
        for (int v = 0; v < 8 * Q; v += 4) {
            const int o = slot_off<L, Q, R>(v, gl);
            f32x4 a = {0.0f, 0.0f, 0.0f, 0.0f}, b = a;
            if (quads) {
                a = reinterpret_cast<const val4 *>(pp + o)->v;
                b = reinterpret_cast<const val4 *>(kp + o)->v;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                pd[p][v + j] = a[j];
                kk[p][v + j] = b[j];
            }
        }
#pragma unroll
        for (int v = 0; v < V; ++v) {
            const int o = slot_off<L, Q, R>(v, gl);
            if (v >= 8 * Q) pd[p][v] = kk[p][v] = 0.0f;
            if (wave_on[p] && (v >= 8 * Q || !full) && ((vmask >> v) & 1u)) {
                pd[p][v] = pp[o];
                kk[p][v] = kp[o];
            }
        }
    }
    // the calibration loads complete here (vmcnt 0): left pending, their first
    // use inside the frame loop would make the compiler wait there for every
    // load in flight, the next frame's prefetch included
    __builtin_amdgcn_s_waitcnt(0x0F70);
    for (int x = tid; x < 2 * RN * bw; x += kV2Threads) s_bits[x] = 0;
    for (int x = tid; x < 2 * RN; x += kV2Threads) s_cnt[x] = 0;
    if (tid < 4) s_nseed[tid] = 0;
    if (tid < 2) s_hcnt[tid] = 0;
    if (tid == 0) s_photons = 0;
    if (tid == 0) s_chunk[0] = s_chunk[1] = 0;

    // Raw words of a frame: Q 16-byte groups and R single words a lane (a load
    // instruction's cost is the cache lines its lanes touch: with 8-byte groups
    // a CSPAD frame's loads cost half as much again).  Not
    // nontemporal: a line is shared by loads of neighbouring lane groups.  Where a
    // bank ends inside the Q groups they are read as column pairs, each pair
    // inside the bank or skipped.
    u32x4 raw_[P][Q];
    uint32_t rawt_[P][R > 0 ? R : 1];
#pragma unroll
    for (int p = 0; p < P; ++p) {
#pragma unroll
        for (int c = 0; c < Q; ++c) raw_[p][c] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
        for (int r = 0; r < (R > 0 ? R : 1); ++r) rawt_[p][r] = 0u;
    }
    const uint16_t *fr_next = A->frames + f_begin * npix + row_base;  // strip of the next frame to load
    auto chunk_in = [&](int c) { return ((vmask >> (8 * c)) & 0xFFu) == 0xFFu; };  // columns 8 c .. of the lane
    auto load_raw = [&](const uint16_t *fr, int o4, u32x4(&raw)[Q], uint32_t(&rawt)[R > 0 ? R : 1]) {
        if (full) {
#pragma unroll
            for (int c = 0; c < Q; ++c)
                raw[c] = reinterpret_cast<const raw4 *>(fr + (uint32_t)o4 + 8 * L * c)->v;
#pragma unroll
            for (int r = 0; r < R; ++r)
                if ((vmask >> (8 * Q + r)) & 1u)
                    rawt[r] = fr[(uint32_t)(o4 + slot_off<L, Q, R>(8 * Q + r, gl))];
        } else if constexpr (ODD) {
#pragma unroll
            for (int c = 0; c < Q; ++c) {
                const uint16_t *p = fr + (uint32_t)o4 + 8 * L * c;
                if (chunk_in(c)) {
                    raw[c] = reinterpret_cast<const raw4 *>(p)->v;
                } else {
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        if ((vmask >> (8 * c + 2 * j + 1)) & 1u) raw[c][j] = *reinterpret_cast<const u32_a2 *>(p + 2 * j);
                        else if ((vmask >> (8 * c + 2 * j)) & 1u) raw[c][j] = p[2 * j];
                    }
                }
            }
        } else {
#pragma unroll
            for (int c = 0; c < Q; ++c) {
                const uint32_t *p = reinterpret_cast<const uint32_t *>(fr + (uint32_t)o4 + 8 * L * c);
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    if ((vmask >> (8 * c + 2 * j)) & 1u) raw[c][j] = p[j];
            }
        }
    };
    // an odd bank's values to memory: whole groups of 8 slots, else one by one
    auto store_odd = [&](float *dst, const float(&x)[V]) {
#pragma unroll
        for (int c = 0; c < Q; ++c) {
            if (chunk_in(c)) {
#pragma unroll
                for (int h = 8 * c; h < 8 * c + 8; h += 4)
                    reinterpret_cast<val4 *>(dst + slot_off<L, Q, R>(h, gl))->v =
                        f32x4{x[h], x[h + 1], x[h + 2], x[h + 3]};
            } else {
#pragma unroll
                for (int v = 8 * c; v < 8 * c + 8; ++v)
                    if ((vmask >> v) & 1u) dst[slot_off<L, Q, R>(v, gl)] = x[v];
            }
        }
    };
    // the lane's values to and from LDS (an active group's, slots in the bank)
    auto store_v = [&](const float(&x)[V], int o4) {
        float *dst = s_v + o4;
        if (full) {
#pragma unroll
            for (int c = 0; c < 2 * Q; ++c)
                reinterpret_cast<val4 *>(dst + slot_off<L, Q, R>(4 * c, gl))->v =
                    f32x4{x[4 * c], x[4 * c + 1], x[4 * c + 2], x[4 * c + 3]};
#pragma unroll
            for (int r = 0; r < R; ++r)
                if ((vmask >> (8 * Q + r)) & 1u) dst[slot_off<L, Q, R>(8 * Q + r, gl)] = x[8 * Q + r];
        } else if constexpr (ODD) {
            store_odd(dst, x);
        } else {
#pragma unroll
            for (int v = 0; v < 8 * Q; v += 2)
                if ((vmask >> v) & 1u)
                    *reinterpret_cast<float2 *>(dst + slot_off<L, Q, R>(v, gl)) = make_float2(x[v], x[v + 1]);
        }
    };
    // Frames2 of the lane's pixels of frame f (own rows)
    auto store_corrected = [&](uint32_t f, const float(&y)[V], int o4) {
        float *dst = fresh(A)->corrected + f * npix + row_base + (uint32_t)o4;
        if (full) {
#pragma unroll
            for (int c = 0; c < 2 * Q; ++c)
                reinterpret_cast<val4 *>(dst + slot_off<L, Q, R>(4 * c, gl))->v =
                    f32x4{y[4 * c], y[4 * c + 1], y[4 * c + 2], y[4 * c + 3]};
#pragma unroll
            for (int r = 0; r < R; ++r)
                if ((vmask >> (8 * Q + r)) & 1u) dst[slot_off<L, Q, R>(8 * Q + r, gl)] = y[8 * Q + r];
        } else if constexpr (ODD) {
            store_odd(dst, y);
        } else {
#pragma unroll
            for (int v = 0; v < 8 * Q; v += 2)
                if ((vmask >> v) & 1u)
                    *reinterpret_cast<float2 *>(dst + slot_off<L, Q, R>(v, gl)) = make_float2(y[v], y[v + 1]);
        }
    };
    if (f_begin < f_end) {
#pragma unroll
        for (int p = 0; p < P; ++p)
            if (wave_on[p]) load_raw(fr_next, o4_[p], raw_[p], rawt_[p]);
    }
    __syncthreads();

    // Seeds of the lane's bank-row: the slots in vm (inside the bank, own rows)
    // with Frames2 above t, appended to the pooled list (order is free, phase 4
    // restores raster order) and counted in `slot`, with a DPP prefix of the
    // lanes' counts and one LDS atomic per wave.  The test is the sign of fl(t -
    // v) (a nonzero difference of finite values keeps its sign, equality gives
    // +0), one sign bit per value shifted in from the last value down.  All lanes
    // of the wave must call it.
    auto append_seeds = [&](const float(&xs)[V], float t, uint32_t vm, int slot, int o4) {
        uint32_t sb = 0;
#pragma unroll
        for (int v = V - 1; v >= 0; --v)
            sb = __builtin_amdgcn_alignbit(sb, __float_as_uint(__fsub_rn(t, xs[v])), 31);
        sb &= vm;
        const uint32_t ns = (uint32_t)__popc(sb);
        const uint32_t incl = wave_incl_scan(ns);
        const uint32_t wtot = (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
        if (wtot) {
            uint32_t base = 0;
            if (lane == 0) base = atomicAdd(&s_nseed[slot], wtot);
            uint32_t pos = (uint32_t)__builtin_amdgcn_readfirstlane((int)base) + incl - ns;
            while (sb) {
                const int v = __builtin_ctz(sb);
                sb &= sb - 1;
                if (pos < (uint32_t)cap) s_seed[pos] = (uint16_t)(o4 + slot_off<L, Q, R>(v, gl));
                ++pos;
            }
        }
    };

    // Frame loop, two barriers per frame.  Iteration f:
    //   A: the lanes correct frame f's words in registers (they were loaded a
    //      frame ahead) and issue frame f+1's loads;
    //   barrier 1: phase 2 of frame f-1 has read u for the last time;
    //   B: each wave writes its bank-rows' u to LDS, finds their medians and
    //      lists their seeds, with no other wave's data; one wave also runs
    //      frame f-1's phase 3;
    //   barrier 2: the seeds and u of frame f are complete;
    //   C: frame f's phase 2 over the pooled seeds and frame f-1's phase 4 over
    //      its hits, in chunks of 64, the first to the first waves and to the last
    //      ones; waves without a chunk go on to A of the next frame.
    // One more iteration drains it.
#ifdef PDC_PHASE_TIMERS
    unsigned long long tm_prev = __builtin_amdgcn_s_memtime();
#define PDC_PHASE(ph)                                                                     \
    {                                                                                     \
        const unsigned long long t_ = __builtin_amdgcn_s_memtime();                       \
        if ((threadIdx.x & 63) == 0) atomicAdd(&s_tm[(threadIdx.x >> 6) * 8 + (ph)], t_ - tm_prev); \
        tm_prev = t_;                                                                     \
    }
#else
#define PDC_PHASE(ph)
#endif
    for (uint32_t f = f_begin; f < f_end + 1; ++f) {
        // the slot tests are recomputed each frame from an opaque copy of the
        // mask: hoisted out of the loop they would be kept in scalar registers,
        // which this kernel does not have to spare
        asm volatile("" : "+v"(vmask));
#pragma unroll
        for (int p = 0; p < P; ++p) asm volatile("" : "+v"(o4_[p]));
        fr_next += npix;  // frame f + 1's strip
        const bool cur_ok = f < f_end;
        const bool p1_ok = f > f_begin;
        const int par = (int)(f & 1), pp = par ^ 1;
        const int sc0 = (int)(f & 3), sc1 = (int)((f + 3) & 3);  // seed counts of f, f-1

        // ================= A: correction of frame f in registers =================
        float x[V];
        uint32_t slow = 0;  // auto-ranging: slots not in range 0
        auto correct = [&](int p) {
            const u32x4(&raw)[Q] = raw_[p];
            const uint32_t(&rawt)[R > 0 ? R : 1] = rawt_[p];
            if constexpr (!MG) {
#pragma unroll
                for (int c = 0; c < Q; ++c)
#pragma unroll
                    for (int j = 0; j < 4; ++j) {
                        const int v = 8 * c + 2 * j;
                        const uint32_t w = raw[c][j] & 0x3FFF3FFFu;
                        x[v] = __fmul_rn(__fsub_rn(cvt_lo16(w), pd[p][v]), kk[p][v]);
                        x[v + 1] = __fmul_rn(__fsub_rn(cvt_hi16(w), pd[p][v + 1]), kk[p][v + 1]);
                    }
#pragma unroll
                for (int r = 0; r < R; ++r) x[8 * Q + r] = dark_gain(rawt[r], pd[p][8 * Q + r], kk[p][8 * Q + r]);
            } else {
                // range 0 from the resident planes; the other pixels (an invalid
                // code, or the rarer ranges 1 and 2) leave their raw word here as
                // bits and are finished in B
                slow = 0;
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    const uint32_t w = v < 8 * Q ? raw[v < 8 * Q ? v / 8 : 0][(v & 7) / 2] : rawt[v < 8 * Q ? 0 : v - 8 * Q];
                    const uint32_t h = v < 8 * Q && (v & 1) ? w >> 16 : w & 0xFFFFu;
                    const float u = dark_gain(h, pd[p][v], kk[p][v]);
                    const bool r0 = h < 0x4000u;
                    x[v] = r0 ? u : __uint_as_float(h);
                    slow |= (uint32_t)!r0 << v;
                }
                slow &= vmask;
            }
            if (f + 1 < f_end) load_raw(fr_next, o4_[p], raw_[p], rawt_[p]);
            if constexpr (!MG) {
                // columns past the bank
                if (!full) {
#pragma unroll
                    for (int v = 0; v < 8 * Q; ++v) x[v] = (vmask >> v) & 1u ? x[v] : INFINITY;
                }
#pragma unroll
                for (int r = 0; r < R; ++r) x[8 * Q + r] = (vmask >> (8 * Q + r)) & 1u ? x[8 * Q + r] : INFINITY;
            }
        };
        if (cur_ok && wave_on[0]) correct(0);
        PDC_PHASE(0);
        lds_barrier();  // 1
        PDC_PHASE(1);

        // ================= B: 1(f), one wave 3(f-1) ==============================
        const uint32_t nseed_1 = p1_ok ? s_nseed[sc1] : 0u;  // frame f-1's seeds and listed hits
        const uint32_t nhit_1 = p1_ok ? s_hcnt[pp] : 0u;
        // a seed list or a hit list that was full: the general kernel redoes the unit
        const bool ovf_1 = nseed_1 > (uint32_t)cap || nhit_1 > (uint32_t)hcap;
        // frame f's hit bitmaps and counts (parity par) are rebuilt by its local
        // maxima in C; their last reader was frame f-2's phase 4 in C of f-1
        if (cur_ok) {
            for (int j = tid; j < RN * bw; j += kV2Threads) s_bits[par * RN * bw + j] = 0;
            for (int j = tid; j < RN; j += kV2Threads) s_cnt[par * RN + j] = 0;
        }
        if (tid == 0) {
            s_nseed[(sc0 + 1) & 3] = 0;  // frame f+1's (last used by frame f-3)
            s_hcnt[par] = 0;
        }
        if (p1_ok && wave == kP3Wave) {
            // staging chunk claim for frame f-1's hits
            const uint32_t total = ovf_1 ? 0u : nhit_1;
            if (lane == 0) {
                const V2ArgsK K = fresh(A);
                // the chunk lives in LDS: in registers it would be spilled to
                // scratch, whose reload waits for the frame prefetch
                uint64_t chunk_cur = s_chunk[0], chunk_end = s_chunk[1];
                const uint64_t unit = (uint64_t)(f - 1) * K->n_strips + strip;
                uint64_t base = chunk_cur;
                if (ovf_1) {
                    // a list was full: the general kernel redoes this unit
                    atomicOr(&K->state->fallback, 1u);
                    if (K->fb_units) K->fb_units[atomicAdd(&K->state->n_fallback, 1ull)] = unit;
                    base = kNoBase;
                } else if (total > 0) {
                    if (chunk_cur + total > chunk_end) {
                        const uint64_t sz = total > K->chunk_hits ? total : K->chunk_hits;
                        chunk_cur = atomicAdd(&K->state->cursor, (unsigned long long)sz);
                        chunk_end = chunk_cur + sz;
                    }
                    if (chunk_cur + total <= K->pool_cap) {
                        base = chunk_cur;
                        chunk_cur += total;
                    } else {
                        base = kNoBase;
                        atomicOr(&K->state->overflow, 1u);
                    }
                }
                K->unit_base[unit] = base;
                K->unit_count[unit] = total;
                K->unit_photons[unit] = s_photons;  // frame f-1's, summed in its C
                s_photons = 0;
                s_base = base;
                s_chunk[0] = chunk_cur;
                s_chunk[1] = chunk_end;
            }
        }
#pragma unroll
        for (int p = 0; p < P; ++p) {
            if (!cur_ok || !wave_on[p]) continue;
            if (p > 0) correct(p);
            const int o4 = o4_[p], mi = mi_[p];
            const bool act = mi < BR, own = own_[p] != 0;
            uint32_t bad = 0;  // slots with an invalid code
            uint32_t vm = own ? vmask : 0u;  // slots that may be seeds
            if constexpr (MG) {
                // ranges 1 and 2: the raw word waits in the pixel's u slot
                if (act) store_v(x, o4);
                if (!act) slow = 0;
                uint32_t todo = slow;
                while (todo) {
                    const int v = __builtin_ctz(todo);
                    todo &= todo - 1u;
                    const int off = o4 + slot_off<L, Q, R>(v, gl);
                    const uint32_t w = __float_as_uint(s_v[off]);
                    const int rg = gain_range(w, A->gain_mode);
                    float u = INFINITY;
                    if (rg < 0) {
                        bad |= 1u << v;
                    } else {
                        const uint64_t o = row_base + (uint32_t)off + (uint64_t)rg * npix;
                        u = dark_gain(w, A->ped[o], A->k[o]);
                    }
                    s_v[off] = u;
                }
                const uint32_t ninv = own ? (uint32_t)__popc(bad) : 0u;
                const uint32_t tot = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan(ninv), 63);
                if (lane == 0 && tot) atomicAdd(fresh(A)->invalid + f, tot);
                // the lane wrote these words itself
#pragma unroll
                for (int v = 0; v < V; ++v) {
                    const float t = s_v[o4 + slot_off<L, Q, R>(v, gl)];
                    x[v] = (vmask >> v) & 1u ? t : INFINITY;
                }
                vm &= ~bad;
            }
            if constexpr (CMM != 0) {
                // thresholded mean (Fig. c)
                if constexpr (CMM == 1) {
                    // the bank-row's stacked stages: the sum of the noise values
                    // is exact, rounded once (the group's lanes add two binary64
                    // limbs).  A bank-row whose values span more than two limbs
                    // hold marks the frame's seed list full, so that the general
                    // kernel redoes the unit from the separately computed values.
                    SumWindow win = {A->sum_lo, A->sum_hi};
                    bool wide = false;
#pragma unroll
                    for (int s = 0; s < 3; ++s) {
                        if (s >= A->cm_stages) break;
                        int n;
                        bool fits;
                        const float sum = region_sum_grouped<L, V>(
                            x, A->t_cm, (uint32_t)B, win, n, fits,
                            [&](double &q0, double &q1, double sc, double sk, double pk) {
                                // a wide window (rare: a later stage's small
                                // value): the lane's values from its own LDS slots
                                if (act) store_v(x, o4);
#pragma unroll 1
                                for (int v = 0; v < V; ++v) {
                                    const float y = s_v[o4 + slot_off<L, Q, R>(v, gl)];
                                    const bool nz = y < A->t_cm && ((vmask >> v) & 1u);
                                    limbs2_add(q0, q1, (double)(nz ? y : 0.0f), sc, sk, pk);
                                }
                            });
                        wide |= !fits;
                        const int n0 = gsum_i<L>(n);
                        const float cm = __fdiv_rn(sum, fmaxf((float)n0, A->cm_guard));
                        win = next_window(win, cm);
#pragma unroll
                        for (int v = 0; v < V; ++v) x[v] = __fsub_rn(x[v], cm);
                    }
                    if (act && wide && gl == 0) atomicAdd(&s_nseed[sc0], (uint32_t)cap + 1u);
                } else {
                    // stage values computed ahead: v = ((u - c1) - c2) - c3
                    const uint32_t gi = (uint32_t)lr0 * nb + (uint32_t)(act ? mi : 0);  // bank-row of the frame
                    const uint32_t reg = A->cm_tile ? gi / ((uint32_t)nb * (uint32_t)H) : gi;
                    const float *cv = A->cm + ((uint64_t)f * A->cm_regions + reg) * 3;
                    const float c0 = cv[0], c1 = cv[1], c2 = cv[2];
#pragma unroll
                    for (int v = 0; v < V; ++v) x[v] = __fsub_rn(__fsub_rn(__fsub_rn(x[v], c0), c1), c2);
                }
            } else {
                if (!MG && act) store_v(x, o4);
                int nv = B, kq = (B - 1) / 2;
                bool actv = act;
                if constexpr (MG) {
                    // the median of the valid values only (invalid ones are +inf)
                    nv = B - gsum_i<L>(__popc(bad));
                    kq = nv > 0 ? (nv - 1) / 2 : 0;
                    actv = act && nv > 0;
                }
                // finish scratch: the frame's own hit list, unused until C
                float *gsc = lds + Ly.hl + par * Ly.hl_stride + (wave * G + lane / L) * (S * L);
                float m = group_median<L, Q, R, S, MG>(x, s_v + o4, nv, kq, A->rank_width, actv, gsc, full, sides);
                if (MG && !actv) m = 0.0f;
                // kept for patches: the own rows' medians (each row has one owner)
                if (float *const meds = fresh(A)->meds)
                    if (own && gl == 0)
                        meds[f * ((uint64_t)fresh(A)->T * H * nb) + (uint64_t)lr0 * nb + (uint32_t)mi] = m;
#pragma unroll
                for (int v = 0; v < V; ++v) x[v] = __fsub_rn(x[v], m);
            }
            // x holds Frames2 now; an invalid pixel's value is +0
            if constexpr (MG) {
#pragma unroll
                for (int v = 0; v < V; ++v) x[v] = x[v] < INFINITY ? x[v] : 0.0f;
            }
            if (act) store_v(x, o4);
            if (KEEP && own) store_corrected(f, x, o4);
            PDC_PHASE(2);
            append_seeds(x, A->t_seed, vm, sc0, o4);
        }
        PDC_PHASE(3);
        lds_barrier();  // 2
        PDC_PHASE(4);

        // ================= C: 2(f), 4(f-1) =======================================
        // few waves have work here and all the others wait for them at barrier 1
        __builtin_amdgcn_s_setprio(3);
        const uint32_t nseed_0 = cur_ok ? s_nseed[sc0] : 0u;
        if (nseed_0 <= (uint32_t)cap) {
            // frame f's seeds
            unsigned long long my_ph = 0;
            float *hq = lds + Ly.hl + par * Ly.hl_stride;
            uint16_t *hp = reinterpret_cast<uint16_t *>(hq + hcap);
            for (uint32_t c0 = 64u * (uint32_t)wave; c0 < nseed_0; c0 += 64u * kV2Waves) {
                const uint32_t j = c0 + lane;
                if (j < nseed_0) {
                    const uint32_t at = s_seed[j];
                    const int row = (int)(__umul24(at, A->row_mul) >> A->row_sh), col = (int)(at - __umul24(row, W));
                    // the 3x3 neighbourhood from the row above and the column
                    // left.  Neighbours outside the loaded rows, across a tile
                    // edge or outside the row are -inf: never above the seed nor
                    // above t_nb.
                    const float *up = s_v + (int)at - W - 1;
                    float nv[3][3];
#pragma unroll
                    for (int dr = 0; dr < 3; ++dr)
#pragma unroll
                        for (int dc = 0; dc < 3; ++dc) nv[dr][dc] = up[dr * W + dc];
                    const bool r0 = row >= 1 && row != bnd, r2 = row + 1 < nrow && row + 1 != bnd;
                    const bool c0ok = col >= 1, c2ok = col + 1 < W;
#pragma unroll
                    for (int dr = 0; dr < 3; ++dr) {
                        const bool rin = dr == 1 || (dr == 0 ? r0 : r2);
                        nv[dr][0] = rin && c0ok ? nv[dr][0] : -INFINITY;
                        nv[dr][1] = rin ? nv[dr][1] : -INFINITY;
                        nv[dr][2] = rin && c2ok ? nv[dr][2] : -INFINITY;
                    }
                    const float vp = nv[1][1];
                    // strictly above the neighbours before it in raster order,
                    // at least the ones after it (ties go to the first)
                    const float me = fmaxf(fmaxf(nv[0][0], nv[0][1]), fmaxf(nv[0][2], nv[1][0]));
                    const float ml2 = fmaxf(fmaxf(nv[1][2], nv[2][0]), fmaxf(nv[2][1], nv[2][2]));
                    const bool is_max = vp > me && vp >= ml2;
                    const uint64_t hm = __ballot(is_max);
                    if (is_max) {
                        const int bank = (int)(__umul24(col, A->bank_mul) >> kBankShift);
                        const int i = (int)__umul24(row, nb) + bank;
                        const int cb = col - (int)__umul24(bank, B);
                        const int first = __builtin_ctzll(hm);
                        uint32_t hbase = 0;
                        if (lane == first) hbase = atomicAdd(&s_hcnt[par], (uint32_t)__popcll(hm));
                        hbase = (uint32_t)__builtin_amdgcn_readfirstlane((int)hbase);
                        float qsum = 0.0f;
#pragma unroll
                        for (int dr = 0; dr < 3; ++dr)
#pragma unroll
                            for (int dc = 0; dc < 3; ++dc)
                                qsum = __fadd_rn(qsum, nv[dr][dc] > A->t_nb ? nv[dr][dc] : 0.0f);
                        atomicOr(&s_bits[__umul24(par * RN + i, bw) + (cb >> 5)], 1u << (cb & 31));
                        atomicAdd(&s_cnt[par * RN + i], 1u);
                        my_ph += photon_count(qsum, A->photon_adu);
                        // the hit list (any order; past its end the unit is redone)
                        const uint32_t h = hbase + (uint32_t)mbcnt(hm);
                        if (h < (uint32_t)hcap) {
                            hq[h] = qsum;
                            hp[h] = (uint16_t)at;
                        }
                    }
                }
            }
            // the wave's photons: 32-bit sums when every lane's is small (64 of
            // them then fit), else lane by lane
            if (__ballot(my_ph != 0)) {
                if (__ballot(my_ph >> 26) == 0) {
                    const uint32_t sum = (uint32_t)__builtin_amdgcn_readlane((int)wave_incl_scan((uint32_t)my_ph), 63);
                    if (lane == 0) atomicAdd(&s_photons, (unsigned long long)sum);
                } else if (my_ph) {
                    atomicAdd(&s_photons, my_ph);
                }
            }
        }
        PDC_PHASE(5);
        if (p1_ok && !ovf_1 && nhit_1) {
            // frame f-1's hits in raster position (bank-row prefix + hits left
            // of the hit in its bank-row)
            const uint64_t base = s_base;
            uint32_t c0 = 64u * (uint32_t)(kV2Waves - 1 - wave);
            if (base != kNoBase && c0 < nhit_1) {
                const float *hq = lds + Ly.hl + pp * Ly.hl_stride;
                const uint16_t *hp = reinterpret_cast<const uint16_t *>(hq + hcap);
                uint2 *const pool = fresh(A)->pool;
                // bank-row prefix of the hit counts: bank-row 64 k + lane in pref[k]
                uint32_t pref[kCntRegs], run = 0;
#pragma unroll
                for (int k = 0; k < kCntRegs; ++k) {
                    const int i = 64 * k + lane;
                    const uint32_t c = i < BR ? s_cnt[pp * RN + i] : 0u;
                    const uint32_t incl = wave_incl_scan(c);
                    pref[k] = run + incl - c;
                    run += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
                }
                for (; c0 < nhit_1; c0 += 64u * kV2Waves) {
                    // every lane takes part (a lane reads another's prefix); those
                    // past the list repeat its last hit and store nothing
                    const uint32_t j = c0 + lane;
                    const uint32_t jc = j < nhit_1 ? j : nhit_1 - 1u;
                    {
                        const uint32_t at = hp[jc];
                        const int row = (int)(__umul24(at, A->row_mul) >> A->row_sh), col = (int)(at - __umul24(row, W));
                        const int bank = (int)(__umul24(col, A->bank_mul) >> kBankShift);
                        const int i = (int)__umul24(row, nb) + bank;
                        const int cb = col - (int)__umul24(bank, B);
                        // (all words read at once: one LDS latency)
                        const uint32_t *bwp = s_bits + __umul24(pp * RN + i, bw);
                        uint32_t wd[kBitWords];
#pragma unroll
                        for (int w = 0; w < kBitWords; ++w) wd[w] = bwp[w];
                        uint32_t rank = 0;
#pragma unroll
                        for (int w = 0; w < kBitWords; ++w) {
                            const int k = cb - 32 * w;  // columns of word w left of the hit
                            rank += __popc(wd[w] & (k >= 32 ? ~0u : (k > 0 ? (1u << k) - 1u : 0u)));
                        }
                        uint32_t first = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * i, (int)pref[0]);
#pragma unroll
                        for (int k = 1; k < kCntRegs; ++k) {
                            const uint32_t t = (uint32_t)__builtin_amdgcn_ds_bpermute(4 * i, (int)pref[k]);
                            first = i >= 64 * k ? t : first;
                        }
                        const float q = hq[jc];
                        if (j < nhit_1) pool[base + first + rank] = make_uint2(row_base + at, __float_as_uint(q));
                    }
                }
            }
        }
        __builtin_amdgcn_s_setprio(0);
        PDC_PHASE(6);
    }
#ifdef PDC_PHASE_TIMERS
    __syncthreads();
    if (threadIdx.x < kV2Waves * 8) atomicAdd(&g_phase_cycles[threadIdx.x], s_tm[threadIdx.x]);
#endif
#undef PDC_PHASE
}

template <int L, int Q, int R, bool KEEP, int CMM, bool MG, bool ODD, int P>
__global__ void __launch_bounds__(kV2Threads) __attribute__((amdgpu_waves_per_eu(4, 4))) frame_kernel_v2(V2Args)
{
    frame_body<L, Q, R, KEEP, CMM, MG, ODD, P>((V2ArgsK)__builtin_amdgcn_kernarg_segment_ptr(), block_item((int)blockIdx.x, (int)gridDim.x));
}

// Banks of 257 to 512 columns: 32 values a lane, with dark and 1/gain and the next
// words 130 registers, so one workgroup (two waves per SIMD) a compute unit.
template <bool KEEP>
__global__ void __launch_bounds__(kV2Threads) __attribute__((amdgpu_waves_per_eu(2, 2))) frame_kernel_v2_wide(V2Args)
{
    frame_body<16, 4, 0, KEEP, 0, false>((V2ArgsK)__builtin_amdgcn_kernarg_segment_ptr(), block_item((int)blockIdx.x, (int)gridDim.x));
}

// Several detectors' batches in one launch: the work items of detector d are
// [first[d], first[d + 1]) of the launch (finer frame groups than a launch
// of its own, so that items of unequal cost even out as they are handed
// out), and each workgroup runs the body
// compiled for its detector's lane layout and gain mode (median common mode,
// Frames2 not kept: the variants v2_mix_variant lists).  TWO: with the bodies of
// the two-pass layout of up to 128 columns, which mixes without it leave out (they
// cost its other bodies registers: three mixed detectors' 1,000 frames 2.59 ms
// with them, 2.53 without).
template <bool TWO>
__global__ void __launch_bounds__(kV2Threads) __attribute__((amdgpu_waves_per_eu(4, 4))) frame_kernel_v2_mix(V2Mix)
{
    const auto M = (const __attribute__((address_space(4))) V2Mix *)__builtin_amdgcn_kernarg_segment_ptr();
    // work items in launch order: consecutive workgroups go to different
    // chiplets, so each chiplet takes a share of every detector's items
    const int item = (int)blockIdx.x;
    int d = 0;
    while (d + 1 < M->n && item >= M->first[d + 1]) ++d;
    const V2ArgsK A = &M->a[d];
    const int it = item - M->first[d];
    switch (M->variant[d]) {
    case 0: frame_body<4, 2, 0, false, 0, false>(A, it); break;
    case 1: frame_body<4, 3, 0, false, 0, false>(A, it); break;
    case 2: frame_body<8, 2, 0, false, 0, false>(A, it); break;
    case 3: frame_body<8, 3, 1, false, 0, false>(A, it); break;
    case 4: frame_body<16, 2, 0, false, 0, false>(A, it); break;
    case 5: frame_body<4, 2, 0, false, 0, true>(A, it); break;
    case 6: frame_body<4, 3, 0, false, 0, true>(A, it); break;
    case 7: frame_body<8, 2, 0, false, 0, true>(A, it); break;
    case 8: frame_body<8, 3, 1, false, 0, true>(A, it); break;
    case 9: frame_body<16, 2, 0, false, 0, true>(A, it); break;
    case 10:
        if constexpr (TWO) frame_body<8, 2, 0, false, 0, false, false, 2>(A, it);
        break;
    case 11:
        if constexpr (TWO) frame_body<8, 2, 0, false, 0, true, false, 2>(A, it);
        break;
    default: break;
    }
}

// Lane layouts (L lanes a bank-row, Q chunks of 8 columns and R single columns
// a lane) by bank width.  Few lanes a bank-row pay the search's reductions,
// control and sort once for more bank-rows (a wave holds 64 / L); the lane's
// values, dark and 1/gain (3 V registers, with V = 8 Q + R) and the next
// frame's words have to fit four waves per SIMD (128 registers).
//
// Layout 6 is layout 2 with two passes, for rows of more than 10 banks: one pass
// holds 64 bank-rows, so less than four own rows a strip beside two halo rows.
// 200 frames of 512 rows, one pass and two (us): 11 banks of 100 columns 428 and
// 318, 13 banks 575 and 395, 18 banks 1,094 and 563; 12 banks of 128 columns 338
// and 305.  With fewer banks a row the second pass costs more than the halo rows
// it saves (8 tiles of 185 rows of 2 banks of 128: 109 and 127) or about as much
// (8 of 128: 184 and 186), and two frames take longer (11 banks of 100: 20 and 25).
int v2_layout_of(int B, int nb)
{
    if (B > 96 && B <= 128) return nb > 10 ? 6 : 2;
    return B <= 64 ? 0 : (B <= 96 ? 1 : (B <= 200 ? 3 : (B <= 256 ? 4 : (B <= 512 ? 5 : -1))));
}
int v2_layout_bank_rows(int layout)
{
    constexpr int rows[] = {kV2Threads / 4, kV2Threads / 4, kV2Threads / 8, kV2Threads / 8,
                            kV2Threads / 16 * kV2Passes<16, 2>, kV2Threads / 16, kV2Threads / 8 * 2};
    return layout < 0 ? 0 : rows[layout];
}

size_t v2_layout_finish_bytes(int layout)
{
    return (size_t)kV2Threads * 4 * (layout < 2 ? kV2Finish<4> : (layout < 4 || layout == 6 ? kV2Finish<8> : kV2Finish<16>));
}

template <int L, int Q, int R, int P, bool KEEP, int CMM, bool MG, bool ODD = false>
static hipError_t launch_v2_k(const V2Args &a, uint32_t grid, size_t lds, hipStream_t s)
{
    auto k = frame_kernel_v2<L, Q, R, KEEP, CMM, MG, ODD, P>;
    hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(grid), dim3(kV2Threads), lds, s, a);
    return hipGetLastError();
}

template <int L, int Q, int R, int P = kV2Passes<L, Q>>
static hipError_t launch_v2_t(const V2Args &a, uint32_t grid, size_t lds, bool keep, hipStream_t s)
{
    if (a.cm_mode < 0 || a.cm_mode > 2) return hipErrorInvalidValue;
    if (a.B & 1) {  // (the plan keeps the other odd-bank modes on the general kernel)
        if (a.cm_mode || a.gain_mode) return hipErrorInvalidValue;
        return keep ? launch_v2_k<L, Q, R, P, true, 0, false, true>(a, grid, lds, s)
                    : launch_v2_k<L, Q, R, P, false, 0, false, true>(a, grid, lds, s);
    }
    switch (a.cm_mode * 4 + (keep ? 2 : 0) + (a.gain_mode ? 1 : 0)) {
    case 0: return launch_v2_k<L, Q, R, P, false, 0, false>(a, grid, lds, s);
    case 1: return launch_v2_k<L, Q, R, P, false, 0, true>(a, grid, lds, s);
    case 2: return launch_v2_k<L, Q, R, P, true, 0, false>(a, grid, lds, s);
    case 3: return launch_v2_k<L, Q, R, P, true, 0, true>(a, grid, lds, s);
    case 4: return launch_v2_k<L, Q, R, P, false, 1, false>(a, grid, lds, s);
    case 5: return launch_v2_k<L, Q, R, P, false, 1, true>(a, grid, lds, s);
    case 6: return launch_v2_k<L, Q, R, P, true, 1, false>(a, grid, lds, s);
    case 7: return launch_v2_k<L, Q, R, P, true, 1, true>(a, grid, lds, s);
    case 8: return launch_v2_k<L, Q, R, P, false, 2, false>(a, grid, lds, s);
    case 9: return launch_v2_k<L, Q, R, P, false, 2, true>(a, grid, lds, s);
    case 10: return launch_v2_k<L, Q, R, P, true, 2, false>(a, grid, lds, s);
    default: return launch_v2_k<L, Q, R, P, true, 2, true>(a, grid, lds, s);
    }
}

hipError_t launch_frame_kernel_v2(const V2Args &a, uint32_t grid, size_t lds, bool keep, hipStream_t s)
{
    const int lay = v2_layout_of(a.B, a.nb);
    if (a.B < 1 || lay < 0 || a.rmax * a.nb > v2_layout_bank_rows(lay)) return hipErrorInvalidValue;
    if (lay == 5) {
        if ((a.B & 1) || a.cm_mode || a.gain_mode) return hipErrorInvalidValue;
        auto k = keep ? frame_kernel_v2_wide<true> : frame_kernel_v2_wide<false>;
        hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
        if (e != hipSuccess) return e;
        hipLaunchKernelGGL(k, dim3(grid), dim3(kV2Threads), lds, s, a);
        return hipGetLastError();
    }
    switch (lay) {
    case 0: return launch_v2_t<4, 2, 0>(a, grid, lds, keep, s);
    case 1: return launch_v2_t<4, 3, 0>(a, grid, lds, keep, s);
    case 2: return launch_v2_t<8, 2, 0>(a, grid, lds, keep, s);
    case 3: return launch_v2_t<8, 3, 1>(a, grid, lds, keep, s);
    case 6: return launch_v2_t<8, 2, 0, 2>(a, grid, lds, keep, s);
    default: return launch_v2_t<16, 2, 0>(a, grid, lds, keep, s);
    }
}

int v2_mix_variant(const V2Args &a, bool keep)
{
    const int lay = v2_layout_of(a.B, a.nb);
    if (keep || a.cm_mode || a.meds || a.B < 1 || (a.B & 1) || lay == 5 || lay < 0 || a.rmax * a.nb > v2_layout_bank_rows(lay)) return -1;
    if (lay == 6) return a.gain_mode ? 11 : 10;
    return lay + (a.gain_mode ? 5 : 0);
}

size_t frame_kernel_v2_mix_static_lds()
{
    // (TWO's bodies are the other's and two more)
    hipFuncAttributes fa{};
    if (hipFuncGetAttributes(&fa, (const void *)frame_kernel_v2_mix<true>) != hipSuccess) return SIZE_MAX;
    return fa.sharedSizeBytes;
}

hipError_t launch_frame_kernel_v2_mix(const V2Mix &m, size_t lds, hipStream_t s)
{
    if (m.n < 1 || m.n > kMixMax) return hipErrorInvalidValue;
    bool two = false;
    for (int d = 0; d < m.n; ++d) {
        if (m.variant[d] < 0 || m.first[d + 1] < m.first[d]) return hipErrorInvalidValue;
        two |= m.variant[d] >= 10;
    }
    const uint32_t grid = (uint32_t)m.first[m.n];
    if (grid == 0) return hipSuccess;
    const auto k = two ? frame_kernel_v2_mix<true> : frame_kernel_v2_mix<false>;
    hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k, dim3(grid), dim3(kV2Threads), lds, s, m);
    return hipGetLastError();
}

}  // namespace pdc

#ifdef PDC_PHASE_TIMERS
// Tracing build only: copy the phase cycles of every launch since the last
// call to out[kV2Waves * 8] and clear them (synchronous).
extern "C" int pdc_debug_phase_cycles(unsigned long long *out)
{
    if (!out) return -1;
    if (hipDeviceSynchronize() != hipSuccess) return -3;
    if (hipMemcpyFromSymbol(out, HIP_SYMBOL(pdc::g_phase_cycles), sizeof(unsigned long long) * pdc::kV2Waves * 8) !=
        hipSuccess)
        return -3;
    static unsigned long long z[pdc::kV2Waves * 8];
    if (hipMemcpyToSymbol(HIP_SYMBOL(pdc::g_phase_cycles), z, sizeof z) != hipSuccess) return -3;
    return 0;
}
#endif
