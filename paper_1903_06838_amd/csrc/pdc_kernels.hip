// HIP kernels for gfx950: detector correction, bank-median common mode, photon
// finding and hit-list compaction.
//
// Arithmetic contract (identical to the public header): binary32, one rounding
// per operation, no contraction (this file is built with -ffp-contract=off and
// the pragma below), no fast-math, subnormals preserved.
#include <hip/hip_runtime.h>
#include <math.h>

#include "pdc_device.h"
#include "pdc_internal.h"

#pragma clang fp contract(off)

namespace pdc {

__global__ void init_state_kernel(BatchState *st)
{
    if (threadIdx.x == 0) {
        st->cursor = 0;
        st->overflow = 0;
        st->fallback = 0;
        st->total = 0;
        st->n_fallback = 0;
        st->t0 = st->t1 = wall_clock64();
    }
}

hipError_t launch_init_state(BatchState *state, hipStream_t s)
{
    hipLaunchKernelGGL(init_state_kernel, dim3(1), dim3(64), 0, s, state);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// v1 frame kernel: one workgroup per unit at a time (grid-stride over units).
//   load rows [r0-1, r1+1) of the tile (halo rows for the 3x3 window)
//   u = dark/gain corrected value -> LDS, row layout
//   per group of sort_rows rows: copy the banks into a sort buffer padded with
//   +inf, bitonic sort, subtract the lower median in place (LDS now holds v)
//   seeds, 3x3 local maximum, masked charge sum, photon count
//   ordered block compaction -> LDS hit list -> staging chunk
// ---------------------------------------------------------------------------
constexpr int kV1Threads = 256;

size_t frame_kernel_v1_lds_bytes(int strip_rows, int W, int nb, int sort_width, int sort_rows,
                                 uint32_t max_unit_hits)
{
    size_t rows = (size_t)strip_rows + 2;
    size_t floats = rows * W + (size_t)sort_rows * nb * sort_width;
    floats = (floats + 1) & ~(size_t)1;  // 8-byte align the hit list
    return floats * 4 + (size_t)max_unit_hits * 8;
}

template <bool KEEP>
__global__ void __launch_bounds__(kV1Threads) frame_kernel_v1(FrameKernelArgs A)
{
    extern __shared__ float lds[];
    __shared__ uint32_t s_wave[kV1Threads / 64];
    __shared__ unsigned long long s_photons;
    __shared__ uint64_t s_base;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int W = A.W, B = A.B, nb = A.nb, H = A.H, Pw = A.sort_width;
    const int rows_max = A.strip_rows + 2;
    float *s_v = lds;
    float *s_sort = s_v + (size_t)rows_max * W;
    size_t hit_off = (size_t)rows_max * W + (size_t)A.sort_rows * nb * Pw;
    hit_off = (hit_off + 1) & ~(size_t)1;
    uint2 *s_hits = reinterpret_cast<uint2 *>(lds + hit_off);
    const uint64_t npix = (uint64_t)A.T * H * W;
    const int kmed = (B - 1) / 2;

    uint64_t chunk_cur = 0, chunk_end = 0;  // staging chunk (used by thread 0)

    const uint64_t n_iter = A.unit_list ? A.n_list : A.n_units;
    for (uint64_t it = blockIdx.x; it < n_iter; it += gridDim.x) {
        const uint64_t unit = A.unit_list ? A.unit_list[it] : it;
        const uint64_t f = unit / (uint64_t)A.units_per_frame;
        const int su = (int)(unit - f * (uint64_t)A.units_per_frame);
        // rows r0..r1 (own) and lr0..lr1 (loaded) count from tile_base; rows
        // on either side of row gb belong to different tiles
        int t, r0, r1, lr0, lr1, gb = INT32_MAX;
        if (A.strips) {  // a persistent-kernel strip: global rows, may cross one tile edge
            const V2Strip S = A.strips[su];
            t = 0;
            r0 = S.g0;
            r1 = S.g1;
            lr0 = S.lg0;
            lr1 = S.lg1;
            gb = S.gb;
        } else {
            t = su / A.strips_per_tile;
            r0 = (su - t * A.strips_per_tile) * A.strip_rows;
            r1 = min(r0 + A.strip_rows, H);
            lr0 = max(r0 - 1, 0);
            lr1 = min(r1 + 1, H);
        }
        const int nrows = lr1 - lr0;
        const uint16_t *fr = A.frames + f * npix;
        const uint32_t tile_base = (uint32_t)t * (uint32_t)H * (uint32_t)W;

        // load + correct: u (auto-ranging: the reported range's planes, +inf
        // for an invalid code, counted on own rows)
        uint32_t ninv = 0;
        for (int i = tid; i < nrows * W; i += kV1Threads) {
            uint32_t p = tile_base + (uint32_t)lr0 * W + i;
            if (A.gain_mode) {
                bool bad;
                s_v[i] = dark_gain_ranged(fr[p], A.gain_mode, A.ped[p], A.k[p], A.ped, A.k, npix, p, bad);
                const int row = lr0 + i / W;
                if (bad && row >= r0 && row < r1) ++ninv;
            } else {
                s_v[i] = dark_gain(fr[p], A.ped[p], A.k[p]);
            }
        }
        if (ninv && !A.unit_list) atomicAdd(A.invalid + f, ninv);  // list mode: counted already
        __syncthreads();

        // thresholded-mean common mode, computed ahead: v = ((u - c1) - c2) - c3
        if (A.cm) {
            const float *cf = A.cm + f * (uint64_t)A.cm_regions * 3;
            for (int i = tid; i < nrows * W; i += kV1Threads) {
                const int row = i / W, c = i - row * W;
                const uint32_t grow = (uint32_t)t * H + lr0 + row;  // global row
                const uint32_t reg = A.cm_tile ? grow / (uint32_t)H : grow * (uint32_t)nb + c / B;
                const float *cv = cf + (uint64_t)reg * 3;
                const float u = s_v[i];
                s_v[i] = !(u < INFINITY) ? 0.0f : __fsub_rn(__fsub_rn(__fsub_rn(u, cv[0]), cv[1]), cv[2]);
            }
            __syncthreads();
        }
        // bank medians, a group of rows at a time; v = u - m in place
        for (int g0 = 0; g0 < (A.cm ? 0 : nrows); g0 += A.sort_rows) {
            const int gr = min(A.sort_rows, nrows - g0);
            const int total = gr * nb * Pw;
            for (int i = tid; i < total; i += kV1Threads) {
                int seg = i / Pw;
                int j = i - seg * Pw;
                int row = seg / nb;
                int b = seg - row * nb;
                s_sort[i] = j < B ? s_v[(g0 + row) * W + b * B + j] : INFINITY;
            }
            __syncthreads();
            for (int k = 2; k <= Pw; k <<= 1)
                for (int j = k >> 1; j > 0; j >>= 1) {
                    for (int q = tid; q < total / 2; q += kV1Threads) {
                        int i = (q / j) * 2 * j + (q % j);
                        int l = i + j;
                        bool asc = ((i & (Pw - 1)) & k) == 0;
                        float x = s_sort[i], y = s_sort[l];
                        if (asc ? (x > y) : (x < y)) {
                            s_sort[i] = y;
                            s_sort[l] = x;
                        }
                    }
                    __syncthreads();
                }
            for (int i = tid; i < gr * W; i += kV1Threads) {
                int row = i / W;
                int c = i - row * W;
                const float *seg = s_sort + (size_t)(row * nb + c / B) * Pw;
                float m;
                if (A.gain_mode) {
                    // the lower median of the valid values: invalid ones (+inf)
                    // sort last; an all-invalid bank has m = 0
                    int lo = 0, hi = B;
                    while (lo < hi) {
                        const int mid = (lo + hi) >> 1;
                        if (seg[mid] < INFINITY) lo = mid + 1;
                        else hi = mid;
                    }
                    m = lo > 0 ? seg[(lo - 1) / 2] : 0.0f;
                } else {
                    m = seg[kmed];
                }
                float u = s_v[(g0 + row) * W + c];
                if (!(u < INFINITY)) u = m;  // invalid: v = fl(m - m) = +0
                s_v[(g0 + row) * W + c] = __fsub_rn(u, m);
                // kept for patches: the own rows' medians, once per bank
                const int rl = lr0 + g0 + row;  // row in the tile
                if (A.meds && rl >= r0 && rl < r1 && c % B == 0)
                    A.meds[f * ((uint64_t)A.T * H * nb) + ((uint64_t)t * H + rl) * nb + c / B] = m;
            }
            __syncthreads();
        }
        if (tid == 0) s_photons = 0;

        if (KEEP) {
            const int off = (r0 - lr0) * W;
            float *dst = A.corrected + f * npix + tile_base + (uint64_t)r0 * W;
            for (int i = tid; i < (r1 - r0) * W; i += kV1Threads) dst[i] = s_v[off + i];
        }

        // photon finding with ordered (raster) compaction
        const int npx = (r1 - r0) * W;
        uint32_t count = 0;
        unsigned long long my_ph = 0;
        for (int base = 0; base < npx; base += kV1Threads) {
            int i = base + tid;
            bool hit = false;
            uint32_t pix = 0;
            float qsum = 0.0f;
            if (i < npx) {
                int r = r0 + i / W;
                int c = i - (i / W) * W;
                float vp = s_v[(r - lr0) * W + c];
                if (vp > A.t_seed) {
                    uint32_t p = tile_base + (uint32_t)r * W + c;
                    bool is_max = true;
                    for (int dr = -1; dr <= 1; ++dr)
                        for (int dc = -1; dc <= 1; ++dc) {
                            if (dr == 0 && dc == 0) continue;
                            int rr = r + dr, cc = c + dc;
                            if (rr < lr0 || rr >= lr1 || cc < 0 || cc >= W || ((rr >= gb) != (r >= gb))) continue;
                            float vq = s_v[(rr - lr0) * W + cc];
                            uint32_t q = tile_base + (uint32_t)rr * W + cc;
                            if (!(vp > vq || (vp == vq && p < q))) is_max = false;
                        }
                    if (is_max) {
                        for (int dr = -1; dr <= 1; ++dr)
                            for (int dc = -1; dc <= 1; ++dc) {
                                int rr = r + dr, cc = c + dc;
                                if (rr < lr0 || rr >= lr1 || cc < 0 || cc >= W || ((rr >= gb) != (r >= gb)))
                                    continue;
                                float vj = s_v[(rr - lr0) * W + cc];
                                qsum = __fadd_rn(qsum, vj > A.t_nb ? vj : 0.0f);
                            }
                        hit = true;
                        pix = p;
                        my_ph += photon_count(qsum, A.photon_adu);
                    }
                }
            }
            unsigned long long ballot = __ballot(hit);
            uint32_t pre = __popcll(ballot & ((1ull << lane) - 1ull));
            if (lane == 0) s_wave[wave] = __popcll(ballot);
            __syncthreads();
            uint32_t woff = 0, round_total = 0;
            for (int w = 0; w < kV1Threads / 64; ++w) {
                uint32_t cw = s_wave[w];
                if (w < wave) woff += cw;
                round_total += cw;
            }
            if (hit) s_hits[count + woff + pre] = make_uint2(pix, __float_as_uint(qsum));
            count += round_total;
            __syncthreads();
        }
        if (my_ph) atomicAdd(&s_photons, my_ph);
        __syncthreads();

        if (tid == 0) {
            uint64_t base = chunk_cur;
            if (count > 0) {
                if (chunk_cur + count > chunk_end) {
                    uint64_t sz = count > kChunkHits ? (uint64_t)count : kChunkHits;
                    chunk_cur = atomicAdd(&A.state->cursor, (unsigned long long)sz);
                    chunk_end = chunk_cur + sz;
                }
                if (chunk_cur + count <= A.pool_cap) {
                    base = chunk_cur;
                    chunk_cur += count;
                } else {
                    base = kNoBase;
                    atomicOr(&A.state->overflow, 1u);
                }
            }
            A.unit_base[unit] = base;
            A.unit_count[unit] = count;
            A.unit_photons[unit] = s_photons;
            s_base = base;
        }
        __syncthreads();
        const uint64_t base = s_base;
        if (base != kNoBase)
            for (uint32_t i = tid; i < count; i += kV1Threads) A.pool[base + i] = s_hits[i];
        __syncthreads();
    }
}

hipError_t launch_frame_kernel_v1(const FrameKernelArgs &a, uint32_t grid, size_t lds_bytes,
                                  bool keep_corrected, hipStream_t s)
{
    auto k = keep_corrected ? frame_kernel_v1<true> : frame_kernel_v1<false>;
    if (lds_bytes > 64 * 1024) {
        hipError_t e = hipFuncSetAttribute((const void *)k, hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds_bytes);
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(k, dim3(grid), dim3(kV1Threads), lds_bytes, s, a);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Block-wide exclusive scan helpers (256 threads = 4 waves of 64).
// ---------------------------------------------------------------------------
constexpr int kScanThreads = 256;

template <typename T>
__device__ __forceinline__ T wave_inclusive_scan(T x)
{
    const int lane = threadIdx.x & 63;
    for (int d = 1; d < 64; d <<= 1) {
        T y = __shfl_up(x, d, 64);
        if (lane >= d) x += y;
    }
    return x;
}

// Returns the exclusive prefix of x over the block; *block_total gets the sum.
template <typename T>
__device__ __forceinline__ T block_exclusive_scan(T x, T *s_tmp, T *block_total)
{
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    T inc = wave_inclusive_scan(x);
    if (lane == 63) s_tmp[wave] = inc;
    __syncthreads();
    T off = 0, tot = 0;
    for (int w = 0; w < kScanThreads / 64; ++w) {
        T v = s_tmp[w];
        if (w < wave) off += v;
        tot += v;
    }
    __syncthreads();
    *block_total = tot;
    return off + inc - x;
}

// The batch's state to its pinned copy (one thread, after the last change).
__device__ __forceinline__ void publish_state(const BatchState *st, const HostMirror &host)
{
    if (!host.state) return;
    *host.state = *st;
    __threadfence_system();
}

__global__ void __launch_bounds__(kScanThreads)
frame_sums_kernel(const uint32_t *unit_count, const unsigned long long *unit_photons,
                  uint64_t n_frames, int32_t upf, uint32_t *unit_local, uint32_t *frame_hits,
                  unsigned long long *frame_photons, BatchState *st, int stamp)
{
    __shared__ uint32_t s_tmp[kScanThreads / 64];
    __shared__ unsigned long long s_ph;
    const uint64_t f = blockIdx.x;
    if (f >= n_frames) return;
    if (stamp && f == 0 && threadIdx.x == 0) st->t1 = wall_clock64();
    if (threadIdx.x == 0) s_ph = 0;
    __syncthreads();
    const uint64_t u0 = f * (uint64_t)upf;
    uint32_t carry = 0;
    unsigned long long ph = 0;
    for (int base = 0; base < upf; base += kScanThreads) {
        int i = base + threadIdx.x;
        uint32_t c = i < upf ? unit_count[u0 + i] : 0u;
        if (i < upf) ph += unit_photons[u0 + i];
        uint32_t tot;
        uint32_t ex = block_exclusive_scan<uint32_t>(c, s_tmp, &tot);
        if (i < upf) unit_local[u0 + i] = carry + ex;
        carry += tot;
    }
    if (ph) atomicAdd(&s_ph, ph);
    __syncthreads();
    if (threadIdx.x == 0) {
        frame_hits[f] = carry;
        frame_photons[f] = s_ph;
    }
}

hipError_t launch_frame_sums(const uint32_t *unit_count, const unsigned long long *unit_photons,
                             uint64_t n_frames, int32_t units_per_frame, uint32_t *unit_local,
                             uint32_t *frame_hits, unsigned long long *frame_photons, BatchState *state,
                             bool stamp, hipStream_t s)
{
    if (n_frames == 0) return hipSuccess;
    hipLaunchKernelGGL(frame_sums_kernel, dim3((uint32_t)n_frames), dim3(kScanThreads), 0, s,
                       unit_count, unit_photons, n_frames, units_per_frame, unit_local,
                       frame_hits, frame_photons, state, stamp ? 1 : 0);
    return hipGetLastError();
}

__global__ void __launch_bounds__(kScanThreads)
frame_scan_kernel(const uint32_t *frame_hits, const unsigned long long *frame_photons, uint64_t n_frames,
                  unsigned long long *frame_offset, BatchState *st, HostMirror host)
{
    __shared__ unsigned long long s_tmp[kScanThreads / 64];
    unsigned long long carry = 0;
    for (uint64_t base = 0; base < n_frames; base += kScanThreads) {
        uint64_t i = base + threadIdx.x;
        unsigned long long c = i < n_frames ? frame_hits[i] : 0ull;
        unsigned long long tot;
        unsigned long long ex = block_exclusive_scan<unsigned long long>(c, s_tmp, &tot);
        if (i < n_frames) {
            frame_offset[i] = carry + ex;
            // (by one workgroup in whole lines: by each frame's workgroup of the
            // sums, 10,000 frames cost them 0.30 ms)
            if (host.frame_hits) {
                host.frame_hits[i] = (uint32_t)c;
                host.frame_photons[i] = frame_photons[i];
            }
        }
        carry += tot;
    }
    if (threadIdx.x == 0) {
        frame_offset[n_frames] = carry;
        st->total = carry;
        publish_state(st, host);
    }
    if (host.frame_hits) __threadfence_system();
}

hipError_t launch_frame_scan(const uint32_t *frame_hits, const unsigned long long *frame_photons, uint64_t n_frames,
                             unsigned long long *frame_offset, BatchState *state, HostMirror host, hipStream_t s)
{
    hipLaunchKernelGGL(frame_scan_kernel, dim3(1), dim3(kScanThreads), 0, s, frame_hits, frame_photons, n_frames,
                       frame_offset, state, host);
    return hipGetLastError();
}

// Each wave copies the staged runs of kScatterUnits consecutive units into
// the raster-order list.  A unit's run is short (about a hundred hits at
// occupancy 0.01), so one unit per wave left each wave two dependent memory
// round trips for little data; here lanes 0..kScatterUnits-1 read the units'
// counts, bases and destinations at once, and the first two 64-hit rows of
// every run are loaded before any is stored, so up to 2 kScatterUnits loads
// per lane are in flight.  Longer runs finish row by row.  Units whose run
// was not staged (kNoBase) or would end past hits_cap (only after a staging
// overflow; the batch is then recomputed) copy nothing.
constexpr int kScatterUnits = 4;

// The runs of U units held by lanes first .. first + U - 1 (count c, staging
// place b, destination dst).
__device__ __forceinline__ void copy_runs(uint32_t c, uint64_t b, uint64_t dst, int first, int lane, const uint2 *pool,
                                          uint2 *hits)
{
    constexpr int U = kScatterUnits;
    uint32_t cu[U];
    uint64_t bu[U], du[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
        cu[k] = (uint32_t)__builtin_amdgcn_readlane((int)c, first + k);
        bu[k] = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(b >> 32), first + k) << 32) |
                (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)b, first + k);
        du[k] = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(dst >> 32), first + k) << 32) |
                (uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)dst, first + k);
    }
    uint2 v[U][2];
#pragma unroll
    for (int k = 0; k < U; ++k)
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const uint32_t i = (uint32_t)lane + 64u * r;
            if (i < cu[k]) v[k][r] = pool[bu[k] + i];
        }
#pragma unroll
    for (int k = 0; k < U; ++k)
#pragma unroll
        for (int r = 0; r < 2; ++r) {
            const uint32_t i = (uint32_t)lane + 64u * r;
            if (i < cu[k]) hits[du[k] + i] = v[k][r];
        }
#pragma unroll
    for (int k = 0; k < U; ++k)
        for (uint32_t i = (uint32_t)lane + 128u; i < cu[k]; i += 64) hits[du[k] + i] = pool[bu[k] + i];
}


__global__ void __launch_bounds__(256)
scatter_kernel(const uint32_t *unit_count, const uint64_t *unit_base, const uint32_t *unit_local,
               const unsigned long long *frame_offset, const uint2 *pool, uint64_t n_units,
               int32_t upf, uint2 *hits, uint64_t hits_cap)
{
    constexpr int U = kScatterUnits;
    const uint64_t u0 = ((uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6)) * U;
    const int lane = threadIdx.x & 63;
    if (u0 >= n_units) return;
    uint32_t c = 0;
    uint64_t b = 0, dst = 0;
    if (lane < U && u0 + lane < n_units) {
        const uint64_t unit = u0 + lane;
        c = unit_count[unit];
        b = unit_base[unit];
        dst = frame_offset[unit / (uint64_t)upf] + unit_local[unit];
        if (b == kNoBase || dst + c > hits_cap) c = 0;
    }
    copy_runs(c, b, dst, 0, lane, pool, hits);
}

hipError_t launch_scatter(const uint32_t *unit_count, const uint64_t *unit_base,
                          const uint32_t *unit_local, const unsigned long long *frame_offset,
                          const uint2 *pool, uint64_t n_units, int32_t units_per_frame,
                          uint2 *hits, uint64_t hits_cap, hipStream_t s)
{
    if (n_units == 0) return hipSuccess;
    const uint64_t per_block = 4 * (uint64_t)kScatterUnits;  // 4 waves
    const uint64_t blocks = (n_units + per_block - 1) / per_block;
    hipLaunchKernelGGL(scatter_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, unit_count,
                       unit_base, unit_local, frame_offset, pool, n_units, units_per_frame, hits,
                       hits_cap);
    return hipGetLastError();
}

// frame_sums, frame_scan and scatter of a batch of few units in one launch: a
// workgroup of 16 units sums all unit counts before its own itself (a few
// loads a thread) instead of waiting for the scan of a launch before, forms the
// totals of the frames that start in its units, and copies its runs.  The last
// workgroup publishes the batch's state.  Launches and the gaps between them
// bound such batches: 16 CSPAD frames (3,168 units) took 13 us in the three
// kernels and 10 us more for a copy of the state, 6 us here.  The sums over the
// units before grow with their number: at 64 CSPAD frames (12,672 units) it is
// 10 us against 14, and larger batches keep the three kernels.
constexpr uint32_t kTailUnits = 16384, kTailUpf = 1024;

bool tail_fits(uint64_t n_units, int32_t upf)
{
    return n_units > 0 && n_units <= kTailUnits && upf <= (int32_t)kTailUpf;
}

__global__ void __launch_bounds__(256) tail_kernel(TailArgs a)
{
    constexpr uint32_t NU = 4 * kScatterUnits;  // units of a workgroup
    __shared__ uint32_t s_sum[4][2];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const uint32_t u0 = blockIdx.x * NU;
    const bool last = blockIdx.x == gridDim.x - 1;
    if (last && a.stamp && tid == 0) a.state->t1 = wall_clock64();
    const uint32_t f0 = u0 / a.upf, fs = f0 * a.upf;  // frame of unit u0, its first unit
    // hits before unit u0, and before unit fs (all of a tail_fits batch's fit 32 bits)
    uint32_t before = 0, before_f = 0;
    for (uint32_t i = 4u * tid; i < u0; i += 4u * 256u) {
        const uint4 c = *reinterpret_cast<const uint4 *>(a.unit_count + i);
        before += c.x + c.y + c.z + c.w;
        before_f += (i < fs ? c.x : 0u) + (i + 1u < fs ? c.y : 0u) + (i + 2u < fs ? c.z : 0u) + (i + 3u < fs ? c.w : 0u);
    }
    for (int d = 1; d < 64; d <<= 1) {
        before += (uint32_t)__shfl_xor((int)before, d, 64);
        before_f += (uint32_t)__shfl_xor((int)before_f, d, 64);
    }
    if (lane == 0) {
        s_sum[wave][0] = before;
        s_sum[wave][1] = before_f;
    }
    __syncthreads();
    before = before_f = 0;
    for (int w = 0; w < 4; ++w) {
        before += s_sum[w][0];
        before_f += s_sum[w][1];
    }
    // lane l < 16 of every wave: unit u0 + l
    const uint32_t unit = u0 + (uint32_t)lane;
    const bool in = (uint32_t)lane < NU && unit < a.n_units;
    uint32_t c = in ? a.unit_count[unit] : 0u;
    const uint64_t base = in ? a.unit_base[unit] : kNoBase;
    uint32_t incl = c;
    for (int d = 1; d < (int)NU; d <<= 1) {
        const uint32_t y = (uint32_t)__shfl_up((int)incl, d, 64);
        if (lane >= d) incl += y;
    }
    const uint32_t at = before + incl - c;  // hits before the lane's unit
    const uint32_t f = unit / a.upf, first = f * a.upf;
    const uint32_t at_first = (uint32_t)__shfl((int)at, first >= u0 ? (int)(first - u0) & 63 : 0, 64);
    if (wave == 0 && in) {
        a.unit_local[unit] = at - (first >= u0 ? at_first : before_f);
        if (unit == first) a.frame_offset[f] = at;
        if (unit == a.n_units - 1u) {
            a.frame_offset[a.n_frames] = at + c;
            a.state->total = at + c;
            publish_state(a.state, a.host);
        }
    }
    // frames whose first unit is one of these.  (No fence behind the writes to
    // pinned memory: the host reads them after an event behind the kernel.  One
    // fence a frame writes its chiplet's L2 back, and where a frame's units are a
    // multiple of 16 two chiplets hold them all: with fences 250 frames of 64 units
    // took 52 us from the frame kernel's end to the batch's, 12 so; of 51 units 22
    // and 12.)
    for (uint32_t g = (u0 + a.upf - 1u) / a.upf + (uint32_t)wave; g < a.n_frames && g * a.upf < u0 + NU; g += 4u) {
        uint32_t n = 0;
        unsigned long long ph = 0;
        for (uint32_t i = (uint32_t)lane; i < a.upf; i += 64) {
            n += a.unit_count[g * a.upf + i];
            ph += a.unit_photons[g * a.upf + i];
        }
        for (int d = 1; d < 64; d <<= 1) {
            n += (uint32_t)__shfl_xor((int)n, d, 64);
            ph += __shfl_xor(ph, d, 64);
        }
        if (lane == 0) {
            a.frame_hits[g] = n;
            a.frame_photons[g] = ph;
            if (a.host.frame_hits) {
                a.host.frame_hits[g] = n;
                a.host.frame_photons[g] = ph;
            }
        }
    }
    if (base == kNoBase || (uint64_t)at + c > a.hits_cap) c = 0;
    copy_runs(c, base, at, kScatterUnits * wave, lane, a.pool, a.hits);
}

hipError_t launch_tail(const TailArgs &a, hipStream_t s)
{
    if (!tail_fits(a.n_units, (int32_t)a.upf)) return hipErrorInvalidValue;
    const uint32_t blocks = (a.n_units + 4 * kScatterUnits - 1) / (4 * kScatterUnits);
    hipLaunchKernelGGL(tail_kernel, dim3(blocks), dim3(256), 0, s, a);
    return hipGetLastError();
}

// Like scatter_kernel, but each hit goes straight to its 16-byte record
// (frame, pixel, charge, photon count) at its raster position; records past
// out_cap are not written (the caller's destination keeps the first ones).
__global__ void __launch_bounds__(256)
scatter_records_kernel(const uint32_t *unit_count, const uint64_t *unit_base, const uint32_t *unit_local,
                       const unsigned long long *frame_offset, const uint2 *pool, uint64_t n_units, int32_t upf,
                       float photon_adu, HitRecord *out, uint64_t out_cap)
{
    const uint64_t unit = (uint64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (unit >= n_units) return;
    const uint32_t c = unit_count[unit];
    const uint64_t b = unit_base[unit];
    if (c == 0 || b == kNoBase) return;
    const uint64_t f = unit / (uint64_t)upf;
    const uint64_t dst = frame_offset[f] + unit_local[unit];
    for (uint32_t i = lane; i < c && dst + i < out_cap; i += 64) {
        const uint2 h = pool[b + i];
        const float q = __uint_as_float(h.y);
        HitRecord r;
        r.frame = (uint32_t)f;
        r.pixel = h.x;
        r.charge = q;
        r.nphot = photon_count(q, photon_adu);
        out[dst + i] = r;
    }
}

hipError_t launch_scatter_records(const uint32_t *unit_count, const uint64_t *unit_base,
                                  const uint32_t *unit_local, const unsigned long long *frame_offset,
                                  const uint2 *pool, uint64_t n_units, int32_t units_per_frame, float photon_adu,
                                  HitRecord *out, uint64_t out_cap, hipStream_t s)
{
    if (n_units == 0) return hipSuccess;
    uint64_t blocks = (n_units + 3) / 4;
    hipLaunchKernelGGL(scatter_records_kernel, dim3((uint32_t)blocks), dim3(256), 0, s, unit_count, unit_base,
                       unit_local, frame_offset, pool, n_units, units_per_frame, photon_adu, out, out_cap);
    return hipGetLastError();
}

// Largest f in [lo, hi) with frame_offset[f] <= g, by the wave together: 64
// probes a round, so three rounds for up to 2^18 frames.  Needs
// frame_offset[lo] <= g < frame_offset[hi]; all lanes active, uniform arguments.
__device__ __forceinline__ uint64_t wave_frame_of(const unsigned long long *frame_offset, uint64_t lo, uint64_t hi,
                                                  uint64_t g, int lane)
{
    while (hi - lo > 1) {
        const uint64_t step = (hi - lo + 63) / 64, i = lo + (uint64_t)lane * step;
        const unsigned long long m = __ballot(i < hi && frame_offset[i] <= g);
        lo += (uint64_t)(63 - __builtin_clzll(m)) * step;
        hi = lo + step < hi ? lo + step : hi;
    }
    return lo;
}

// Hits first .. first + n - 1 as 16-byte records.  24 bytes a hit bound it, so
// a wave takes 64 R consecutive hits, finds the frames of its first and last one
// once, and has a lane search between them only where they differ (a search over
// all frames per hit, one hit a thread, moved 1.65 TB/s: 10,000 CSPAD frames' 220
// million hits 3.21 ms, now 0.96 ms, 5.5 TB/s).
template <int R>
__global__ void __launch_bounds__(256)
format_hits_kernel(const uint2 *hits, const unsigned long long *frame_offset, uint64_t n_frames,
                   uint64_t first, uint64_t n, float photon_adu, HitRecord *out)
{
    constexpr uint64_t per_wave = 64 * R;
    const int lane = threadIdx.x & 63;
    const uint64_t wave = (uint64_t)blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const uint64_t i0 = wave * per_wave;
    if (i0 >= n) return;
    const uint64_t last = (n - i0 < per_wave ? n : i0 + per_wave) - 1;
    uint2 h[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint64_t i = i0 + 64u * r + lane;
        h[r] = hits[first + (i <= last ? i : last)];
    }
    // frame_offset[0] = 0 and frame_offset[n_frames] = total > first + n - 1
    const uint64_t f0 = wave_frame_of(frame_offset, 0, n_frames, first + i0, lane);
    const uint64_t f1 = frame_offset[f0 + 1] > first + last
                            ? f0
                            : wave_frame_of(frame_offset, f0 + 1, n_frames, first + last, lane);
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint64_t i = i0 + 64u * r + lane;
        if (i > last) return;
        uint64_t lo = f0, hi = f1 + 1;
        while (hi - lo > 1) {
            const uint64_t mid = (lo + hi) / 2;
            if (frame_offset[mid] <= first + i) lo = mid;
            else hi = mid;
        }
        const float q = __uint_as_float(h[r].y);
        HitRecord rec;
        rec.frame = (uint32_t)lo;
        rec.pixel = h[r].x;
        rec.charge = q;
        rec.nphot = photon_count(q, photon_adu);
        out[i] = rec;
    }
}

// One row a wave for short lists: their time is one wave's chain of searches,
// which the rows repeat (the call with a device destination, rows 1, 2 and 8, us:
// 968 hits of 100 small frames 14.0, 14.6, 19.5, by a search per hit 13.7; 100,000
// of 10 ePix100 frames 13.8, 14.0, 15.6, 13.9).  Long lists take two, which share
// the search: 300,000 hits of 64 CSPAD frames 14.5, 14.4, 15.9; 11 million 55.9,
// 50.9, 52.4, by a search per hit 88.8.
hipError_t launch_format_hits(const uint2 *hits, const unsigned long long *frame_offset,
                              uint64_t n_frames, uint64_t first, uint64_t n, float photon_adu,
                              HitRecord *out, hipStream_t s)
{
    if (n == 0) return hipSuccess;
    const int rows = n < (1u << 19) ? 1 : 2;
    const uint64_t blocks = (n + 256 * rows - 1) / (256 * rows);
    hipLaunchKernelGGL(rows == 1 ? format_hits_kernel<1> : format_hits_kernel<2>, dim3((uint32_t)blocks), dim3(256), 0,
                       s, hits, frame_offset, n_frames, first, n, photon_adu, out);
    return hipGetLastError();
}

}  // namespace pdc
