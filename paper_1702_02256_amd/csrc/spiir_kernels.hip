// gfx950 kernels of the SPIIR library.
//
//   k_stage   append a block to the band-0 input ring and run the /2 FIR
//             cascade (§2.2, resampling of Eq. 9 as a causal FIR) once per
//             stream, writing every band's new samples to its ring;
//   k_filter  the filter bank: Eq. 7 per filter with the state in VGPRs,
//             Eq. 8 as a deterministic two-level LDS reduction per piece;
//   k_filter_pipe  the same with the same bits for launches that leave the
//             compute units short of waves;
//   k_chain   chunk start states of a bank split in time;
//   k_upadd   per template: sum a band's pieces, add the x2 upsampled lower
//             band (§2.2, Fig. "multi"), lowest band first, write z;
//   k_prep    FP64 precompute of the carry corrections a1^C - fl32(a1)^C;
//   k_fill    zero fill (used instead of memset so the sequence stays a plain
//             chain of kernels).
#include <hip/hip_runtime.h>

#include <climits>
#include <mutex>
#include <type_traits>

#include "spiir_internal.h"

namespace spiir {

__device__ __forceinline__ float acc_fma(float a, float b, float c) { return fmaf(a, b, c); }
__device__ __forceinline__ double acc_fma(double a, double b, double c) { return fma(a, b, c); }

// Address-space views of device memory.  Pointers held in the bank
// descriptor are generic; through a generic pointer the compiler emits flat
// accesses, which count against the LDS wait counter too, so a wait for an
// LDS read would also wait for every outstanding flat store or load.  Memory
// that no thread writes during a kernel (the descriptor, coefficient tables,
// input rings, the clock) is read through the constant view, which also lets
// uniform reads become scalar loads; memory a kernel writes, or reads and
// writes, goes through the global view.
#if defined(__HIP_DEVICE_COMPILE__)
#define SPIIR_AS_GLOBAL __attribute__((address_space(1)))
#define SPIIR_AS_CONST __attribute__((address_space(4)))
#else  // the host pass over this file only parses the kernels
#define SPIIR_AS_GLOBAL
#define SPIIR_AS_CONST
#endif
template <class T>
__device__ __forceinline__ SPIIR_AS_GLOBAL T* gmem(T* p)
{
    return (SPIIR_AS_GLOBAL T*)p;
}
template <class T>
__device__ __forceinline__ const SPIIR_AS_CONST T* cmem(const T* p)
{
    return (const SPIIR_AS_CONST T*)p;
}
typedef const SPIIR_AS_CONST BankDev CBankDev;
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// Waits for the wave's global loads (vmcnt 0).  Before a loop that stores: a
// load whose wait the compiler cannot place on every path costs a wait in the
// loop, and there it would also wait for the stores, a microsecond each time.
__device__ __forceinline__ void wait_loads() { __builtin_amdgcn_s_waitcnt(0x0F70); }

// Requests that need no staging launch (single-rate banks of few workgroups):
// the filter kernel reads the block's new samples from x itself, its first
// workgroup appends them to the band-0 ring, and the workgroup that is the last
// to have read the device clock advances it.  The ring slots of the new samples
// are none of those the block's history is read from, so no workgroup reads
// what another writes.  A bank split in time is staged the same way by its
// end-state pass, and k_chain advances the clock.  With z written by the filter kernel too (piece_out), a
// call is one launch where it was three: 1024 templates of 512 filters, 2048
// samples, 282 -> 262 us; 2 templates, 74 samples 27 -> 20.
//
// First sample of the block; one thread reads it, before the ticket, so that
// every workgroup has it when the last ticket advances the clock.
__device__ __forceinline__ int64_t block_start(const ReqArg& q, CBankDev* bd, float* lds)
{
    int64_t* w = reinterpret_cast<int64_t*>(lds);
    if (threadIdx.x == 0) {
        volatile int64_t* clock = bd->clock;
        const int64_t s0 = clock[1];
        *w = s0;
        wait_loads();  // s0 has arrived before this workgroup is counted
        unsigned* ticket = reinterpret_cast<unsigned*>(bd->clock + 2);
        if (atomicAdd(ticket, 1u) == (unsigned)q.nblocks - 1u) {
            *ticket = 0u;
            clock[0] = s0;
            clock[1] = s0 + q.n;
        }
    }
    __syncthreads();
    const int64_t s0 = *w;
    __syncthreads();  // the words are reused
    return s0;
}

// ---------------------------------------------------------------------------
// Input staging and the downsample cascade (one workgroup per request).
//
// One workgroup walks the bands in turn, so its latency is what it costs: the
// block and every band's history are read before the first band (one wait each
// where each band had its own), and the common 32-tap decimator reads its
// window as 16 aligned pairs: 4096 samples, 7 bands, launch to end 17.5 ->
// 12.9 us before 4096 templates, 13.4 -> 10.2 before 512.
// LDS: cur [td-1 + max_block] | nxt [td-1 + max_block/2] | taps [td], each from an
// even word.
// ---------------------------------------------------------------------------
constexpr int kStageThreads = 1024;
constexpr int kStageFastTaps = 32;  // decimator length with an unrolled path
constexpr int kStageSamples = kInnerBlock / kStageThreads;  // block samples per thread

__global__ void __launch_bounds__(kStageThreads) k_stage(LaunchArgs args)
{
    extern __shared__ float sm[];
    const ReqArg& q = args.req[blockIdx.x];
    if (q.direct) return;
    CBankDev* bd = cmem(q.bd);
    SPIIR_AS_GLOBAL int64_t* clock = gmem(bd->clock);
    const SPIIR_AS_CONST float* x = cmem(q.x);
    const int n = q.n, tid = threadIdx.x;
    float xv[kStageSamples];
#pragma unroll
    for (int u = 0; u < kStageSamples; ++u) {
        const int i = tid + u * kStageThreads;
        xv[u] = i < n ? x[i] : 0.0f;
    }
    const int64_t s0 = clock[1];
    const int H = bd->H;
    SPIIR_AS_GLOBAL float* rings = gmem(bd->rings);
    SPIIR_AS_GLOBAL float* ring0 = rings + bd->ring_off[0];
    const int64_t m0 = bd->ring_mask[0];

    const int td = bd->td;
    const int hl = td - 1;  // at most kStageThreads: one history sample per thread and band
    const SPIIR_AS_CONST float* tap = cmem(bd->hd);
    float* cur = sm;
    float* nxt = sm + ((hl + bd->max_block + 1) & ~1);
    float* hd = nxt + ((hl + bd->max_block / 2 + 1) & ~1);
    float hist[kMaxBands] = {};
#pragma unroll
    for (int h = 0; h < kMaxBands - 1; ++h)
        if (h < H - 1 && tid < hl) hist[h] = rings[bd->ring_off[h] + (((s0 >> h) - hl + tid) & bd->ring_mask[h])];
    if (H > 1 && td != kStageFastTaps)
        for (int i = tid; i < td; i += kStageThreads) hd[i] = tap[i];
    // the block goes to the band-0 ring and to LDS (the ring slots of the
    // histories read above are not among the ones written here)
#pragma unroll
    for (int u = 0; u < kStageSamples; ++u) {
        const int i = tid + u * kStageThreads;
        if (i < n) {
            ring0[(s0 + i) & m0] = xv[u];
            if (H > 1) cur[hl + i] = xv[u];
        }
    }
    if (H > 1 && tid < hl) cur[tid] = hist[0];
    __syncthreads();
    if (tid == 0) {
        clock[0] = s0;  // read by the filter kernel that follows
        clock[1] = s0 + n;
    }

    for (int h = 1; h < kMaxBands; ++h) {
        if (h >= H) break;
        const int nh = n >> h;
        const int64_t s0h = s0 >> h;
        SPIIR_AS_GLOBAL float* ring = rings + bd->ring_off[h];
        const int64_t mk = bd->ring_mask[h];
        if (h < H - 1 && tid < hl) nxt[tid] = hist[h];
        for (int m = tid; m < nh; m += kStageThreads) {
            // x_h[m] = sum_j h_d[j] x_{h-1}[2m - j]; cur[hl + i] holds x_{h-1} at block offset i
            float s = 0.0f;
            if (td == kStageFastTaps) {
                // taps as scalar loads, the window (from the even word 2m) first, then
                // the multiply-adds in the same order as the loop below
                f32x2_t w[kStageFastTaps / 2];
                const f32x2_t* src = reinterpret_cast<const f32x2_t*>(cur + 2 * m);
#pragma unroll
                for (int j = 0; j < kStageFastTaps / 2; ++j) w[j] = src[j];
#pragma unroll
                for (int j = 0; j < kStageFastTaps; ++j) {
                    const int i = kStageFastTaps - 1 - j;
                    s = fmaf(tap[j], i & 1 ? w[i / 2].y : w[i / 2].x, s);
                }
            } else {
                const float* src = cur + hl + 2 * m;
                for (int j = 0; j < td; ++j) s = fmaf(hd[j], src[-j], s);
            }
            nxt[hl + m] = s;
            ring[(s0h + m) & mk] = s;
        }
        __syncthreads();
        float* t = cur;
        cur = nxt;
        nxt = t;
    }
}

// ---------------------------------------------------------------------------
// The filter bank.
// LDS: E0 [xcap] | E1 [xcap] (two copies only) | pbuf [L/2][kTile+1] c32 | l2 2 x [kTile][nrun_max] c32 |
//      pzoff [npiece_max] i64 | lmeta [L] i32 | prun [npiece_max] int2
// ---------------------------------------------------------------------------
// Address of a piece's output row: the workspace, or for a single-rate template that
// is one piece its row of z (no upsample-and-add pass over it then).
__device__ __forceinline__ long long piece_out(const ReqArg& q, const PieceDesc& pd)
{
    c32* row = q.z_direct && pd.whole ? q.z + (int64_t)pd.tmpl * q.ldz : q.zw + pd.zoff;
    return reinterpret_cast<long long>(row);
}
__device__ __forceinline__ SPIIR_AS_GLOBAL c32* piece_row(long long address)
{
    return gmem(reinterpret_cast<c32*>(address));
}

constexpr int kStageBatch = 4;  // window loads a thread keeps in flight

// Fills the input window: E0[i] = fetch(i) for i < wn and, with two copies,
// E1[i] = fetch(i + 1); kStageBatch loads in flight per thread before their
// LDS stores.  (fetch(wn) is called, its value not used by any filter.)
template <class Fetch>
__device__ __forceinline__ void stage_window(float* E0, float* E1, int wn, Fetch fetch)
{
    const int nt = blockDim.x;
    for (int i0 = threadIdx.x; i0 <= wn; i0 += kStageBatch * nt) {
        float v[kStageBatch];
#pragma unroll
        for (int u = 0; u < kStageBatch; ++u) {
            const int i = i0 + u * nt;
            v[u] = i <= wn ? fetch(i) : 0.0f;
        }
#pragma unroll
        for (int u = 0; u < kStageBatch; ++u) {
            const int i = i0 + u * nt;
            if (i < wn) E0[i] = v[u];
            if (E1 && i > 0 && i <= wn) E1[i - 1] = v[u];
        }
    }
}

// The ring append of such a request (see block_start), by its first workgroup.
__device__ __forceinline__ void append_block(const ReqArg& q, CBankDev* bd, int64_t s0)
{
    SPIIR_AS_GLOBAL float* ring = gmem(bd->rings + bd->ring_off[0]);
    const int64_t mk = bd->ring_mask[0];
    const SPIIR_AS_CONST float* x = cmem(q.x);
    for (int i0 = threadIdx.x; i0 < q.n; i0 += kStageBatch * blockDim.x) {
        float v[kStageBatch];
#pragma unroll
        for (int u = 0; u < kStageBatch; ++u) v[u] = x[min(i0 + u * (int)blockDim.x, q.n - 1)];
#pragma unroll
        for (int u = 0; u < kStageBatch; ++u)
            if (i0 + u * (int)blockDim.x < q.n) ring[(s0 + i0 + u * (int)blockDim.x) & mk] = v[u];
    }
    if (q.direct == kDirectSplit && threadIdx.x == 0) gmem(bd->clock)[0] = s0;  // k_chain advances [1]
}

// value of the other lane of the pair (lane ^ 1), via DPP quad_perm [1,0,3,2]
__device__ __forceinline__ float pair_swap(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0xB1, 0xF, 0xF, true));
}

template <int F>
__device__ __forceinline__ void lane_sum(float (&vr)[F], float (&vi)[F])
{
    // pairwise tree over the lane's filters; the result is left in element 0
#pragma unroll
    for (int s = 1; s < F; s *= 2)
#pragma unroll
        for (int i = 0; i + s < F; i += 2 * s) {
            vr[i] += vr[i + s];
            vi[i] += vi[i + s];
        }
}

// One sample of Eq. 7 for the lane's F filters, given their inputs xv[f]; the
// lane sum is combined with the other lane of the pair and stored, one
// component per lane (the even lane the real part, the odd lane the imaginary
// part) at pcol[2*j].
//
// Odd lanes hold their filters in swapped form, (Im y, Re y), with the tables
// transformed to match (a1 -> conj(a1), b0 -> (Im b0, Re b0), carry ->
// conj): the same arithmetic then advances the swapped state.  So every
// lane's first component sum is what it keeps (even: Re, odd: Im) and its
// second is what its partner needs, and the pair combine is one DPP add.
template <int F, bool SUM>
__device__ __forceinline__ void one_step(const float (&xv)[F], float* __restrict__ pcol, int j,
                                         const float (&ar)[F],
                                         const float (&ai)[F], const float (&br)[F],
                                         const float (&bi)[F], float (&yr)[F], float (&yi)[F])
{
    float tr[F], ti[F];
#pragma unroll
    for (int f = 0; f < F; ++f) {
        const float pr = br[f] * xv[f], pi = bi[f] * xv[f];
        const float nr = fmaf(ar[f], yr[f], fmaf(-ai[f], yi[f], pr));
        const float ni = fmaf(ar[f], yi[f], fmaf(ai[f], yr[f], pi));
        yr[f] = nr; yi[f] = ni;
        tr[f] = nr; ti[f] = ni;
    }
    if (!SUM) return;  // end-state pass of a time split: no output
    lane_sum<F>(tr, ti);
    // even lane: re_even + re_odd; odd lane: im_odd + im_even
    pcol[2 * j] = tr[0] + pair_swap(ti[0]);
}

// A full tile of kTile samples starting at an absolute multiple of kTile.
// x2[f] points at the 8-byte aligned pair (x[k - d], x[k + 1 - d]) of filter f
// in the window copy of its delay's parity, so one ds_read_b64 feeds two
// samples.  Each pair stays one ds_read_b64: the pair is a native vector (a
// struct would be split into two 32-bit loads), and the scheduling barrier
// after each step's loads keeps the compiler from fusing the reads of
// consecutive pairs into ds_read2_b64.  On gfx950 a wave's ds_read_b64 whose
// 32-lane halves touch distinct bank pairs takes 2 LDS cycles, while a
// ds_read2_b64 over the same addresses took 15 (measured with
// SQ_LDS_IDX_ACTIVE and SQ_LDS_BANK_CONFLICT), so the fused form made the
// window reads the largest LDS cost and undid the bank-aware placement.  The
// barrier still lets the next step's loads be issued during this step's
// arithmetic.  The restrict qualifiers tell the compiler that the
// partial-sum stores never alias the window.
template <int F, bool SUM>
__device__ __forceinline__ void tile_full(const f32x2_t* const (&xp)[F], float* __restrict__ pcol,
                                          const float (&ar)[F],
                                          const float (&ai)[F], const float (&br)[F],
                                          const float (&bi)[F], float (&yr)[F], float (&yi)[F])
{
    const f32x2_t* __restrict__ x2[F];
#pragma unroll
    for (int f = 0; f < F; ++f) x2[f] = xp[f];
#pragma unroll
    for (int jj = 0; jj < kTile / 2; ++jj) {
        float xa[F], xb[F];
#pragma unroll
        for (int f = 0; f < F; ++f) {
            const f32x2_t v = x2[f][jj];
            xa[f] = v.x;
            xb[f] = v.y;
        }
        __builtin_amdgcn_sched_barrier(0);
        one_step<F, SUM>(xa, pcol, 2 * jj, ar, ai, br, bi, yr, yi);
        one_step<F, SUM>(xb, pcol, 2 * jj + 1, ar, ai, br, bi, yr, yi);
    }
}

// A full tile from a single window copy: x1[f] points at x[k - d]; each
// sample is one 32-bit read (the compiler pairs them into two-word reads).
template <int F, bool SUM>
__device__ __forceinline__ void tile_full1(const float* const (&xp)[F], float* __restrict__ pcol,
                                           const float (&ar)[F], const float (&ai)[F],
                                           const float (&br)[F], const float (&bi)[F],
                                           float (&yr)[F], float (&yi)[F])
{
    const float* __restrict__ x1[F];
#pragma unroll
    for (int f = 0; f < F; ++f) x1[f] = xp[f];
#pragma unroll
    for (int j = 0; j < kTile; ++j) {
        float xv[F];
#pragma unroll
        for (int f = 0; f < F; ++f) xv[f] = x1[f][j];
        one_step<F, SUM>(xv, pcol, j, ar, ai, br, bi, yr, yi);
    }
}

// `cnt` samples from arbitrary starting points: x1[f] points at x[k - d] in the
// unshifted window copy.
template <int F, bool SUM>
__device__ __forceinline__ void tile_partial(const float* const (&xp)[F], int cnt,
                                             float* __restrict__ pcol, const float (&ar)[F], const float (&ai)[F],
                                             const float (&br)[F], const float (&bi)[F],
                                             float (&yr)[F], float (&yi)[F])
{
    for (int j = 0; j < cnt; ++j) {
        float xv[F];
#pragma unroll
        for (int f = 0; f < F; ++f) xv[f] = xp[f][j];
        one_step<F, SUM>(xv, pcol, j, ar, ai, br, bi, yr, yi);
    }
}

// Time chunk c of a band's block [s0h, s0h + nh) when the bank is split in
// time, at absolute multiples of lc: chunk 0 is the rest of the chunk in
// progress (from the block start to the first multiple; empty if the block
// starts on one), chunk c >= 1 covers [B + (c-1) lc, B + c lc) clipped to the
// block.
struct Chunk {
    int k0, k1;  // block-relative sample range (empty if k0 >= k1)
    bool last;   // last non-empty chunk of the block
};

__device__ __forceinline__ Chunk chunk_range(int c, int nchunk, int64_t s0h, int nh, int lc)
{
    Chunk r;
    if (nchunk == 1) {
        r.k0 = 0;
        r.k1 = nh;
        r.last = true;
        return r;
    }
    const int64_t B = (s0h + lc - 1) / lc * lc;
    const int last_c = s0h + nh - 1 < B ? 0 : 1 + (int)((s0h + nh - 1 - B) / lc);
    int64_t cs = c == 0 ? s0h : B + (int64_t)(c - 1) * lc;
    int64_t ce = c == 0 ? B : cs + lc;
    if (cs < s0h) cs = s0h;
    if (ce > s0h + nh) ce = s0h + nh;
    r.k0 = (int)(cs - s0h);
    r.k1 = ce > cs ? (int)(ce - s0h) : r.k0;
    r.last = c == last_c;
    return r;
}

// A time split cuts the recurrence at absolute multiples of a chunk length lc.
// Every chunk's samples run from its start state S, which k_chain forms from the
// zero-start run of the chunk before, S' = a1^lc S + E.  Both runs of a chunk
// in progress at a block's end are carried on, so where blocks begin changes no
// result.
//
// LOCAL: the end-state pass, every chunk from zero (the chunk in progress from
// its carried zero-start state); stores the end states, no output.  Otherwise
// the filter pass, every chunk from its start state (the chunk in progress from
// the carried state).
//
// Start state of a filter slot: y and the pending carry correction u = dC * (y
// at the start of the current carry chunk), added to y at that chunk's end.  A
// chunk starts on a carry-chunk boundary, so u = dC * y there.  The end-state
// pass copies the carried state (y0, ys0) for the filter pass, whose last chunk
// overwrites it.
//
// Which arrays a workgroup reads is decided once, and per slot the values are
// selected, without branches around arithmetic: with the product dC * y in a
// branch of its own, the compiler moved the negation of dC, which the sample
// loop uses too, into some of the branches and left the register undefined on
// another path.
struct Start {
    const c32 *y, *u;
    bool fresh;  // a chunk starts here: u = dC * y
};

// PAIR: neighbouring pointers by one scalar load from a selected address, which a
// workgroup of k_filter waits for less (4096 multi-rate templates 1237 -> 1229 us); in
// the pipelined kernel it costs 1% (86 single-rate templates 265 -> 267).
template <bool LOCAL, bool PAIR>
__device__ __forceinline__ Start start_from(CBankDev* bd, int nchunk, int tc)
{
    Start st;
    st.fresh = nchunk > 1 && tc > 0;
    if (PAIR) {
        typedef c32* Pointer;
        const SPIIR_AS_CONST Pointer* pair = LOCAL ? &bd->ey : nchunk > 1 ? &bd->y0 : &bd->y;
        st.y = pair[0];
        st.u = pair[1];
        if (st.fresh && !LOCAL) st.y = bd->schain + (int64_t)tc * bd->n_slots;
    } else if (LOCAL) {
        st.y = bd->ey;
        st.u = bd->eu;
    } else {
        st.y = st.fresh ? bd->schain + (int64_t)tc * bd->n_slots : nchunk > 1 ? bd->y0 : bd->y;
        st.u = nchunk > 1 ? bd->ys0 : bd->ys;
    }
    if (st.fresh) st.u = st.y;  // not used: the same words again
    return st;
}

// The carried state, kept for the filter pass.
__device__ __forceinline__ void save_state(CBankDev* bd, int64_t g)
{
    const c32 y = gmem(bd->y)[g], u = gmem(bd->ys)[g];
    gmem(bd->y0)[g] = y;
    gmem(bd->ys0)[g] = u;
}

template <bool LOCAL>
__device__ __forceinline__ void start_state(const Start& st, int64_t g, const c32& d, c32& y, c32& u)
{
    y = gmem(st.y)[g];
    u = gmem(st.u)[g];
    const c32 v{fmaf(d.x, y.x, -(d.y * y.y)), fmaf(d.x, y.y, d.y * y.x)};
    u.x = st.fresh ? (LOCAL ? 0.0f : v.x) : u.x;
    u.y = st.fresh ? (LOCAL ? 0.0f : v.y) : u.y;
    if (LOCAL) {
        y.x = st.fresh ? 0.0f : y.x;
        y.y = st.fresh ? 0.0f : y.y;
    }
}

template <int F, bool COMP, bool LOCAL>
__global__ void __launch_bounds__(filter_max_threads(F), filter_min_waves(F, COMP)) k_filter(LaunchArgs args)
{
    // Accumulator of the cross-lane sums: FP32 for the plain sum, FP64 for the
    // compensated one.
    using Acc = typename std::conditional<COMP, double, float>::type;
    extern __shared__ float sm[];
    const int bid = blockIdx.x;
    int lo = 0, hi = args.nseg;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (args.cum[mid] <= bid) lo = mid;
        else hi = mid;
    }
    const ReqArg& q = args.req[args.seg_req[lo]];
    const int h = args.seg_band[lo];
    CBankDev* bd = cmem(q.bd);
    const int nwg_h = bd->band_wg0[h + 1] - bd->band_wg0[h];
    const int li = bid - args.cum[lo];
    const int tc = li / nwg_h;  // time chunk (chunk-major order)
    const WgDesc wg = cmem(bd->wg)[bd->band_wg0[h] + (li - tc * nwg_h)];
    const int L = blockDim.x;
    const int tid = threadIdx.x;
    const int nh = q.n >> h;
    // who stages the block: the staging launch, this launch, or (single rate,
    // split in time) the end-state pass before it
    const bool stages = q.direct == (LOCAL ? kDirectSplit : kDirect);
    const int64_t s0 = q.direct == kDirect ? block_start(q, bd, sm)
                       : LOCAL && stages   ? cmem(bd->clock)[1]
                                           : cmem(bd->clock)[0];
    if (stages && li == 0) append_block(q, bd, s0);
    const int64_t s0h = s0 >> h;
    const Chunk ch = chunk_range(tc, q.nchunk, s0h, nh, bd->lc[h]);
    if (ch.k0 >= ch.k1) return;  // whole workgroup
    const int64_t cmask = bd->C - 1;
    const int nrun = bd->nrun_max;

    // The x window is held twice, E0[m] = x[origin + m] and E1[m] = x[origin + 1 + m]
    // (origin a multiple of 64 absolute samples, E1 32 banks after E0), or once (E0).
    const bool two_copies = bd->copies == 2;
    float* E0 = sm;
    float* E1 = sm + bd->xcap;
    c32* pbuf = reinterpret_cast<c32*>(sm + bd->copies * bd->xcap);
    c32* l2buf = pbuf + (L / 2) * (kTile + 1);  // two tile buffers of run sums
    long long* pzoff = reinterpret_cast<long long*>(l2buf + 2 * kTile * nrun);
    int* lmeta = reinterpret_cast<int*>(pzoff + bd->npiece_max);
    int2* prun = reinterpret_cast<int2*>(lmeta + L);

    lmeta[tid] = cmem(bd->lane_meta)[wg.meta_base + tid];
    for (int p = tid; p < wg.npiece; p += L) {
        const PieceDesc pd = cmem(bd->piece)[wg.piece_base + p];
        pzoff[p] = piece_out(q, pd);
        prun[p] = make_int2(pd.run0, pd.run1);
    }

    float ar[F], ai[F], br[F], bi[F], dr[F], di[F], yr[F], yi[F], ur[F], ui[F];
    int dl[F];
    const Start st = start_from<LOCAL, true>(bd, q.nchunk, tc);
#pragma unroll
    for (int f = 0; f < F; ++f) {
        const int64_t g = wg.slot_base + (int64_t)f * L + tid;
        // (not as constants, whose loads the compiler would move behind the barrier)
        const c32 a = gmem(bd->a)[g], b = gmem(bd->b)[g], d = gmem(bd->dc)[g];
        c32 y, u;
        start_state<LOCAL>(st, g, d, y, u);
        ar[f] = a.x; ai[f] = a.y;
        br[f] = b.x; bi[f] = b.y;
        dr[f] = d.x; di[f] = d.y;
        yr[f] = y.x; yi[f] = y.y;
        ur[f] = u.x; ui[f] = u.y;
        dl[f] = gmem(bd->off)[g];
    }
    if (LOCAL && !st.fresh)
#pragma unroll
        for (int f = 0; f < F; ++f) save_state(bd, wg.slot_base + (int64_t)f * L + tid);
    // without it a lone workgroup of 512 lanes waits in its tile loop: 15 templates, 7
    // bands, 3 streams of up to 14720 samples 2934 us, with it 2742
    wait_loads();
    __syncthreads();

    // level-1 role: sample row j1 of the 16-lane group q1; runs end where endmask
    // is set.  A wave reduces its own four groups; the first half-wave takes
    // groups 0 and 2 of them and the second 1 and 3, so that the two groups one
    // 32-lane half reads are 16 pair entries apart, 32 banks apart in the
    // [L/2][kTile+1] tile, and its 64-bit reads never share a bank pair.
    const int j1 = tid & (kTile - 1);
    const int q1 = (tid >> 6) * 4 + (((tid >> 4) & 1) << 1) + ((tid >> 5) & 1);
    unsigned endmask = 0;
    int slot0 = -1;
#pragma unroll
    for (int i = 0; i < kRunLanes / 2; ++i) {
        const int sl = lmeta[q1 * kRunLanes + 2 * i + 1] & 0xffff;
        if (sl != kSlotNone) {
            endmask |= 1u << i;
            if (slot0 < 0) slot0 = sl;
        }
    }
    // The single-run form applies when every 16-lane group the wave reduces is
    // one run; otherwise the whole wave takes the segmented form (which also
    // handles single-run groups), so no wave executes both.
    const bool wave_single_run = __all(endmask == (1u << (kRunLanes / 2 - 1)));

    const int S = bd->S[h];
    const SPIIR_AS_CONST float* ring = cmem(bd->rings) + bd->ring_off[h];
    const SPIIR_AS_CONST float* xblk = cmem(q.x);
    const int64_t mk = bd->ring_mask[h];
    // Lanes come in pairs of one run (segments span an even number of lanes).
    // The pair sum of sample j is entry e = lane/2 of row j: pbuf[e*(kTile+1) + j],
    // the even lane storing its real part and the odd lane its imaginary part.
    const int pe = tid >> 1;
    float* pcol = reinterpret_cast<float*>(pbuf + pe * (kTile + 1)) + (tid & 1);
    int parity = 0;

    for (int kb = ch.k0; kb < ch.k1; kb += S) {
        const int sub = min(S, ch.k1 - kb);
        // window start: a multiple of 64 at or below the oldest sample any filter
        // reads, minus one, so that an odd-delay pair never starts before E1[0]
        const int64_t origin = ((s0h + kb - wg.maxd - 1) >> 6) << 6;
        const int wn = (int)(s0h + kb + sub - origin);
        __syncthreads();
        if (stages)
            stage_window(E0, two_copies ? E1 : nullptr, wn, [&](int i) {
                const int64_t a = origin + i;  // (a past the block's end is not used)
                const SPIIR_AS_CONST float* p = a < s0 ? ring + (a & mk) : xblk + min((int)(a - s0), q.n - 1);
                return *p;
            });
        else
            stage_window(E0, two_copies ? E1 : nullptr, wn, [&](int i) { return ring[(origin + i) & mk]; });
        __syncthreads();

        int k = kb;
        while (k < kb + sub) {
            const int64_t kabs = s0h + k;
            int cnt = kTile - (int)(kabs & (kTile - 1));
            if (cnt > kb + sub - k) cnt = kb + sub - k;
            const int rel = (int)(kabs - origin);  // window position of sample k
            if (cnt == kTile && two_copies) {
                const f32x2_t* xp[F];
#pragma unroll
                for (int f = 0; f < F; ++f) {
                    const int par = dl[f] & 1;
                    xp[f] = reinterpret_cast<const f32x2_t*>((par ? E1 : E0) + (rel - dl[f] - par));
                }
                tile_full<F, !LOCAL>(xp, pcol, ar, ai, br, bi, yr, yi);
            } else if (cnt == kTile) {
                const float* xp[F];
#pragma unroll
                for (int f = 0; f < F; ++f) xp[f] = E0 + (rel - dl[f]);
                tile_full1<F, !LOCAL>(xp, pcol, ar, ai, br, bi, yr, yi);
            } else {
                const float* xp[F];
#pragma unroll
                for (int f = 0; f < F; ++f) xp[f] = E0 + (rel - dl[f]);
                tile_partial<F, !LOCAL>(xp, cnt, pcol, ar, ai, br, bi, yr, yi);
            }

            // carry correction after the last sample of an absolute chunk of C
            // samples: add the pending correction, then form the next chunk's
            // from the corrected state (each value keeps its own registers; the
            // product is negated, not di, whose negative would be kept in registers)
            if (((kabs + cnt) & cmask) == 0) {
#pragma unroll
                for (int f = 0; f < F; ++f) {
                    yr[f] += ur[f];
                    yi[f] += ui[f];
                    ur[f] = fmaf(dr[f], yr[f], -(di[f] * yi[f]));
                    ui[f] = fmaf(dr[f], yi[f], di[f] * yr[f]);
                }
            }

            if (!LOCAL) {
                // Level 1 reads only partials written by the thread's own wave (its
                // 16-lane group lies inside the wave), so a wave-local sync suffices.
                __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
                __builtin_amdgcn_wave_barrier();
                __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
                c32* l2 = l2buf + parity * (kTile * nrun);
                // level 1: each thread sums one sample row over the runs of a 16-lane group
                // (all 16 partials are loaded before any run result is stored); each run
                // sum is rounded to FP32 once
                if (j1 < cnt) {
                    constexpr int kPairs = kRunLanes / 2;
                    const int e0 = q1 * kPairs;
                    const c32* grp = pbuf + e0 * (kTile + 1) + j1;
                    // one ds_read_b64 each (the barriers keep the compiler from
                    // pairing them into ds_read2_b64, which takes twice as long)
                    c32 v[kPairs];
    #pragma unroll
                    for (int i = 0; i < kPairs; ++i) {
                        v[i] = grp[i * (kTile + 1)];
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    c32* out = l2 + j1 * nrun;
                    if (wave_single_run) {
                        // the whole group is one run: a pairwise tree (short dependency chains)
                        Acc tr[kPairs], ti[kPairs];
    #pragma unroll
                        for (int i = 0; i < kPairs; ++i) {
                            tr[i] = v[i].x;
                            ti[i] = v[i].y;
                        }
    #pragma unroll
                        for (int st = 1; st < kPairs; st *= 2)
    #pragma unroll
                            for (int i = 0; i + st < kPairs; i += 2 * st) {
                                tr[i] += tr[i + st];
                                ti[i] += ti[i + st];
                            }
                        out[slot0] = c32{(float)tr[0], (float)ti[0]};
                    } else {
                        // runs in order; the accumulator restarts after a run end by a
                        // multiplication with keep = 0 (exact, and no selects)
                        int slot = slot0;
                        Acc accr = v[0].x, acci = v[0].y;
    #pragma unroll
                        for (int i = 0; i < kPairs; ++i) {
                            if (i > 0) {
                                const Acc keep = (Acc)(((endmask >> (i - 1)) & 1u) ^ 1u);
                                accr = acc_fma(accr, keep, (Acc)v[i].x);
                                acci = acc_fma(acci, keep, (Acc)v[i].y);
                            }
                            if ((endmask >> i) & 1u) {
                                out[slot] = c32{(float)accr, (float)acci};
                                ++slot;
                            }
                        }
                    }
                }
                __syncthreads();
                // level 2: each (piece, sample) sums its runs in order and writes the output
                for (int task = tid; task < wg.npiece * kTile; task += L) {
                    const int p = task / kTile;
                    const int j = task & (kTile - 1);
                    if (j < cnt) {
                        const int2 rr = prun[p];
                        const c32* row = l2 + j * nrun;
                        Acc accr = 0, acci = 0;
                        for (int s = rr.x; s < rr.y; ++s) {
                            const c32 v = row[s];
                            accr += v.x;
                            acci += v.y;
                        }
                        piece_row(pzoff[p])[k + j] = c32{(float)accr, (float)acci};
                    }
                }
            }
            parity ^= 1;
            k += cnt;
        }
    }

    if (tid >= wg.lanes) return;  // the state of padding stays zero
    if (LOCAL) {
        SPIIR_AS_GLOBAL c32* ue = gmem(bd->uend) + (int64_t)tc * bd->n_slots;
#pragma unroll
        for (int f = 0; f < F; ++f) {
            const int64_t g = wg.slot_base + (int64_t)f * L + tid;
            ue[g] = c32{yr[f], yi[f]};
            if (ch.last) gmem(bd->euend)[g] = c32{ur[f], ui[f]};
        }
        return;
    }
    if (!ch.last) return;  // only the block's last chunk carries its state on
    bool bad = false;
#pragma unroll
    for (int f = 0; f < F; ++f) {
        const int64_t g = wg.slot_base + (int64_t)f * L + tid;
        gmem(bd->y)[g] = c32{yr[f], yi[f]};
        gmem(bd->ys)[g] = c32{ur[f], ui[f]};
        bad |= !(isfinite(yr[f]) && isfinite(yi[f]));
    }
    if (bad) {
        const int p = lmeta[tid] >> 16;
        atomicOr(&bd->flags[cmem(bd->piece)[wg.piece_base + p].tmpl], 1);
    }
}

// ---------------------------------------------------------------------------
// The filter bank for launches that do not fill the device: k_filter's layout,
// arithmetic and order of every sum (so its outputs and states bit for bit),
// with the wait for each cross-lane step hidden and, with X > 1, X threads per
// lane of the layout.
//
// What bounds k_filter there is latency: with one or two waves per SIMD a tile
// of 16 samples spends more time waiting for the LDS (64 clocks a read), the
// two reduction levels and the barrier between them than issuing.  Here one
// iteration runs three tiles at once: the recurrences of tile k, level 1 of
// tile k - 1 and level 2 of tile k - 2, with the reduction levels' reads
// issued before the recurrences and each x pair read one tile ahead into the
// registers its predecessor leaves, so no step waits and one barrier per tile
// is left.
//
// A lone wave issues at most one instruction per 4.4 clocks (measured), and
// more waves add to that.  So a launch with few waves splits every lane's F
// filters over X neighbouring threads: the in-lane pairwise tree becomes DPP
// additions in the same order.  Threads with odd p hold the swapped form of
// the state their slot stores (see one_step), so that each DPP addition
// serves both components.
//
// Measured, us per launch, k_filter -> this kernel: 1 template of 128 filters,
// 4096 samples 586 -> 143 (X = 4; 0.53 us per tile where k_filter takes 2.3);
// 512 multi-rate templates, 4096 samples 534 -> 375 (X = 2); 1024 of them
// 575 -> 427 (X = 1); 160 of them, 576 samples 88 -> 61 (X = 2).
//
// At most kPipeThreads threads, so that a lane may hold 256 registers: a register
// spilled in the tile loop would be read back behind the workspace stores, a
// microsecond.  X = 2 uses up to 182 of them (244 with the zero-start run), X = 4 133
// (172), X = 1 all and spills 26 (32 with the compensated sum), which are read back
// once per window, outside the tile loop.
// ---------------------------------------------------------------------------
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v)
{
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}

// The pair sum of one sample from the threads' F/X filters, one component in
// each thread: the real one where lane and part are both even or both odd.
template <int X, int NF>
__device__ __forceinline__ float split_sum(float (&tr)[NF], float (&ti)[NF])
{
    lane_sum<NF>(tr, ti);
    float s = tr[0] + dpp_mov<0xB1>(ti[0]);      // quad_perm [1,0,3,2]
    if (X == 2) s += dpp_mov<0x1B>(s);           // quad_perm [3,2,1,0]
    if (X == 4) {
        s += dpp_mov<0x4E>(s);                   // quad_perm [2,3,0,1]
        s += dpp_mov<0x141>(s);                  // row_half_mirror
    }
    return s;
}

// One sample of Eq. 7 (see one_step) with the pair sum returned; DUAL: the
// zero-start run (er, ei) too.
template <int X, int NF, bool SUM, bool DUAL>
__device__ __forceinline__ void split_step(const float (&xv)[NF], float& out, const float (&ar)[NF],
                                           const float (&ai)[NF], const float (&br)[NF],
                                           const float (&bi)[NF], float (&yr)[NF], float (&yi)[NF],
                                           float (&er)[NF], float (&ei)[NF])
{
    float tr[NF], ti[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const float pr = br[f] * xv[f], pi = bi[f] * xv[f];
        const float nr = fmaf(ar[f], yr[f], fmaf(-ai[f], yi[f], pr));
        const float ni = fmaf(ar[f], yi[f], fmaf(ai[f], yr[f], pi));
        yr[f] = nr; yi[f] = ni;
        tr[f] = nr; ti[f] = ni;
        if (DUAL) {
            const float mr = fmaf(ar[f], er[f], fmaf(-ai[f], ei[f], pr));
            const float mi = fmaf(ar[f], ei[f], fmaf(ai[f], er[f], pi));
            er[f] = mr; ei[f] = mi;
        }
    }
    if (SUM) out = split_sum<X, NF>(tr, ti);
}

// Waits for the wave's LDS reads (lgkmcnt 0).
__device__ __forceinline__ void wait_lds() { __builtin_amdgcn_s_waitcnt(0xC07F); }

// Keeps the LDS read before it from being fused with the next one (see
// tile_full), while arithmetic may still move across.
__device__ __forceinline__ void keep_single() { __builtin_amdgcn_sched_barrier(0x6); }

constexpr int kAhead = 4;  // x pairs read ahead

template <int F, int X, bool COMP, bool LOCAL, bool DUAL>
__global__ void __launch_bounds__(kPipeThreads) k_filter_pipe(LaunchArgs args)
{
    constexpr int NF = F / X;
    constexpr int kPairs = kRunLanes / 2;
    // run sums a level-2 task reads ahead, and those that pieces of more runs read
    // together after that.  With one thread per lane eight ahead add spills: 1024
    // multi-rate templates, 4096 samples 443 us, six ahead 434 (1400, compensated sum,
    // 569 and 535).  1012 single-rate templates of 508 filters, eight runs each, 4951
    // samples, compensated sum: 658, 683 with the last two one by one, 672 together.
    constexpr int kRunAhead = X == 1 ? 6 : 8;
    constexpr int kRunMore = X == 1 ? 2 : 0;
    using Acc = typename std::conditional<COMP, double, float>::type;
    extern __shared__ float sm[];
    const int bid = blockIdx.x;
    int lo = 0, hi = args.nseg;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (args.cum[mid] <= bid) lo = mid;
        else hi = mid;
    }
    const ReqArg& q = args.req[args.seg_req[lo]];
    const int h = args.seg_band[lo];
    CBankDev* bd = cmem(q.bd);
    const int nwg_h = bd->band_wg0[h + 1] - bd->band_wg0[h];
    const int li = bid - args.cum[lo];
    const int tc = li / nwg_h;
    const WgDesc wg = cmem(bd->wg)[bd->band_wg0[h] + (li - tc * nwg_h)];
    const int NT = blockDim.x, L = bd->L;  // lanes beyond NT / X are padding
    const int tid = threadIdx.x;
    const int ln = tid / X, part = tid % X;  // lane of the layout, thread of the lane
    const bool flip = part & 1;
    const int nh = q.n >> h;
    // who stages the block: the staging launch, this launch, or (single rate,
    // split in time) the end-state pass before it
    const bool stages = q.direct == (LOCAL ? kDirectSplit : kDirect);
    const int64_t s0 = q.direct == kDirect ? block_start(q, bd, sm)
                       : LOCAL && stages   ? cmem(bd->clock)[1]
                                           : cmem(bd->clock)[0];
    if (stages && li == 0) append_block(q, bd, s0);
    const int64_t s0h = s0 >> h;
    const Chunk ch = chunk_range(tc, q.nchunk, s0h, nh, bd->lc[h]);
    if (ch.k0 >= ch.k1) return;  // whole workgroup
    const int64_t cmask = bd->C - 1;
    const int nrun = bd->nrun_max;

    // the LDS layout of k_filter
    const bool two_copies = bd->copies == 2;
    float* E0 = sm;
    float* E1 = sm + bd->xcap;
    c32* pbuf = reinterpret_cast<c32*>(sm + bd->copies * bd->xcap);
    c32* l2buf = pbuf + (L / 2) * (kTile + 1);
    long long* pzoff = reinterpret_cast<long long*>(l2buf + 2 * kTile * nrun);
    int* lmeta = reinterpret_cast<int*>(pzoff + bd->npiece_max);
    int2* prun = reinterpret_cast<int2*>(lmeta + L);

    for (int i = tid; i < L; i += NT) lmeta[i] = cmem(bd->lane_meta)[wg.meta_base + i];
    for (int p = tid; p < wg.npiece; p += NT) {
        const PieceDesc pd = cmem(bd->piece)[wg.piece_base + p];
        pzoff[p] = piece_out(q, pd);
        prun[p] = make_int2(pd.run0, pd.run1);
    }

    float ar[NF], ai[NF], br[NF], bi[NF], dr[NF], di[NF], yr[NF], yi[NF], ur[NF], ui[NF];
    float er[NF], ei[NF], eur[NF], eui[NF];  // DUAL: the zero-start run of the chunk in progress
    int dl[NF];
    const bool dual = DUAL && q.dual;
    const int lc = bd->lc[h];
    const int to_boundary = dual ? lc - (int)(s0h % lc) : 0;  // samples to the end of the chunk in progress
    const int64_t slot0_ = wg.slot_base + (int64_t)part * NF * L + ln;
    Start st = start_from<LOCAL, false>(bd, q.nchunk, tc);
    if (dual && to_boundary == lc) {  // the block starts a chunk
        st.y = st.u = bd->s;
        st.fresh = true;
    }
    const c32* ey = dual ? bd->ey : st.y;
    const c32* eys = dual ? bd->eu : st.u;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int64_t g = slot0_ + (int64_t)f * L;
        c32 a = cmem(bd->a)[g], b = cmem(bd->b)[g], d = cmem(bd->dc)[g], y, u;
        start_state<LOCAL>(st, g, d, y, u);
        c32 e{0.0f, 0.0f}, eu{0.0f, 0.0f};
        if (DUAL) {
            e = gmem(ey)[g];
            eu = gmem(eys)[g];
            e.x = dual ? e.x : 0.0f;
            e.y = dual ? e.y : 0.0f;
            eu.x = dual ? eu.x : 0.0f;
            eu.y = dual ? eu.y : 0.0f;
        }
        if (flip) {
            e = c32{e.y, e.x};
            eu = c32{eu.y, eu.x};
            a.y = -a.y;
            d.y = -d.y;
            b = c32{b.y, b.x};
            y = c32{y.y, y.x};
            u = c32{u.y, u.x};
        }
        ar[f] = a.x; ai[f] = a.y;
        br[f] = b.x; bi[f] = b.y;
        dr[f] = d.x; di[f] = d.y;
        yr[f] = y.x; yi[f] = y.y;
        ur[f] = u.x; ui[f] = u.y;
        er[f] = e.x; ei[f] = e.y;
        eur[f] = eu.x; eui[f] = eu.y;
        dl[f] = cmem(bd->off)[g];
    }
    if (LOCAL && !st.fresh)
#pragma unroll
        for (int f = 0; f < NF; ++f) save_state(bd, slot0_ + (int64_t)f * L);
    __syncthreads();

    // Level-1 role: sample row j1 of the 16-lane group q1 (the wave's own
    // 4 / X groups); with X > 1 a thread sums one component, c1 (with X = 4 the
    // upper half-wave repeats the lower's sums).
    constexpr int kGroups = 4 / X;  // 16-lane groups per wave
    const int wl = tid & 63;
    const int j1 = wl & (kTile - 1);
    const int q1 = X == 1 ? (tid >> 6) * 4 + (((wl >> 4) & 1) << 1) + (wl >> 5)
                          : (tid >> 6) * kGroups + ((wl >> 4) & (kGroups - 1));
    const int c1 = X == 1 ? 0 : ((wl >> 4) / kGroups) & 1;
    unsigned endmask = 0;
    int slot0 = -1;
    // k_filter's vote: the tree only where all four groups of 64 lanes are single runs
    bool single = true;
#pragma unroll
    for (int i = 0; i < kPairs; ++i) {
        const int sl = lmeta[q1 * kRunLanes + 2 * i + 1] & 0xffff;
        if (sl != kSlotNone) {
            endmask |= 1u << i;
            if (slot0 < 0) slot0 = sl;
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int sg = lmeta[((q1 & ~3) + g) * kRunLanes + 2 * i + 1] & 0xffff;
            single &= (sg != kSlotNone) == (i == kPairs - 1);
        }
    }
    const bool wave_single_run = __all(single);
    const float* grp = reinterpret_cast<const float*>(pbuf + q1 * kPairs * (kTile + 1) + j1) + c1;

    // Level-2 role: row j2 of piece p2 (with X > 1, one component, c2), for the
    // waves that hold such tasks; tasks beyond NT are summed in a loop.
    constexpr int kComp = X == 1 ? 1 : 2;  // tasks per (piece, row)
    const int ntask2 = wg.npiece * kTile * kComp;
    // The last waves take them: they are the ones that may be idle.
    const int t2 = NT - 64 - (tid & ~63) + wl;
    const bool duty = __builtin_amdgcn_readfirstlane(t2 & ~63) < ntask2;
    const bool more_tasks = ntask2 > NT;
    const int j2 = (t2 / kComp) & (kTile - 1), c2 = X == 1 ? 0 : t2 & 1;
    const int p2 = min(t2 / (kComp * kTile), wg.npiece - 1);
    const int run0 = prun[p2].x, run1 = prun[p2].y;
    const bool long_run = __any(run1 - run0 > kRunAhead);
    SPIIR_AS_GLOBAL float* zrow = reinterpret_cast<SPIIR_AS_GLOBAL float*>(piece_row(pzoff[p2]) + j2) + c2;
    const int l2off = 2 * (j2 * nrun + run0) + c2;

    const int S = bd->S[h];
    const SPIIR_AS_CONST float* ring = cmem(bd->rings) + bd->ring_off[h];
    const SPIIR_AS_CONST float* xblk = cmem(q.x);
    const int64_t mk = bd->ring_mask[h];
    // Where the thread stores pair sums: of the X threads that hold the same
    // component of a pair, thread px stores every X-th sample.
    const int px = X == 1 ? 0 : X == 2 ? part : 2 * (ln & 1) + (part >> 1);
    float* pcol = reinterpret_cast<float*>(pbuf + (ln >> 1) * (kTile + 1)) + ((ln ^ part) & 1);
    float* const l2f = reinterpret_cast<float*>(l2buf);
    const int l2size = 2 * kTile * nrun;  // floats of one run-sum buffer

    // A wave of padding lanes takes no part in the tiles but their barriers and
    // its level-2 tasks (its run sums belong to no piece).
    const bool idle = __builtin_amdgcn_readfirstlane(ln) >= wg.lanes;

    // the tiles in flight: first sample and length of the tile whose partial
    // sums are in pbuf (1) and of the one whose run sums are in l2buf (2)
    int k1 = 0, cnt1 = 0, k2 = 0, cnt2 = 0, parity = 0;
    f32x2_t xv[NF][kAhead];  // the next kAhead x pairs of each filter

    // The reads of both levels, ahead of their use.  Reads past a piece's last
    // run stay inside the LDS (the piece tables follow the run sums) and are
    // not used.
    f32x2_t v1[kPairs], v2[kRunAhead];
    auto load1 = [&]() {
#pragma unroll
        for (int i = 0; i < kPairs; ++i) {
            const float* p = grp + 2 * i * (kTile + 1);
            if (X == 1) v1[i] = *reinterpret_cast<const f32x2_t*>(p);
            else v1[i].x = *p;
            keep_single();
        }
    };
    auto load2 = [&]() {
        const float* row = l2f + (parity ^ 1) * l2size + l2off;
#pragma unroll
        for (int i = 0; i < kRunAhead; ++i) {
            const float* p = row + 2 * i;
            if (X == 1) v2[i] = *reinterpret_cast<const f32x2_t*>(p);
            else v2[i].x = *p;
            keep_single();
        }
    };
    // level 1: the run sums of a 16-lane group, in k_filter's two orders.  In
    // the segmented one every pair stores its running sum in the slot of the
    // run it belongs to, so the run's last one stays.
    auto level1 = [&](auto single_run) {
        float* o = l2f + parity * l2size + 2 * j1 * nrun + c1;
        auto put = [&](int slot, Acc r, Acc i) {
            if (X == 1) *reinterpret_cast<f32x2_t*>(o + 2 * slot) = f32x2_t{(float)r, (float)i};
            else o[2 * slot] = (float)r;
        };
        if (single_run.value) {
            Acc tr[kPairs], ti[kPairs];
#pragma unroll
            for (int i = 0; i < kPairs; ++i) {
                tr[i] = v1[i].x;
                if (X == 1) ti[i] = v1[i].y;
            }
#pragma unroll
            for (int st = 1; st < kPairs; st *= 2)
#pragma unroll
                for (int i = 0; i + st < kPairs; i += 2 * st) {
                    tr[i] += tr[i + st];
                    if (X == 1) ti[i] += ti[i + st];
                }
            put(slot0, tr[0], ti[0]);
        } else {
            Acc accr = v1[0].x, acci = X == 1 ? v1[0].y : 0.0f;
#pragma unroll
            for (int i = 0; i < kPairs; ++i) {
                if (i > 0) {
                    const Acc keep = (Acc)(((endmask >> (i - 1)) & 1u) ^ 1u);
                    accr = acc_fma(accr, keep, (Acc)v1[i].x);
                    if (X == 1) acci = acc_fma(acci, keep, (Acc)v1[i].y);
                }
                put(slot0 + __popc(endmask & ((1u << i) - 1)), accr, acci);
            }
        }
    };
    // level 2: a piece's runs in order; the first kRunAhead were read ahead
    auto level2 = [&]() {
        Acc accr = 0, acci = 0;
#pragma unroll
        for (int i = 0; i < kRunAhead; ++i) {
            const bool in = run0 + i < run1;
            accr += in ? (Acc)v2[i].x : (Acc)0;
            if (X == 1) acci += in ? (Acc)v2[i].y : (Acc)0;
        }
        const float* l2r = l2f + (parity ^ 1) * l2size;
        if (long_run) {
            // (the reads of the first few together)
            f32x2_t w[kRunMore > 0 ? kRunMore : 1];
#pragma unroll
            for (int i = 0; i < kRunMore; ++i) {
                const float* p = l2r + l2off + 2 * (kRunAhead + i);
                if (X == 1) w[i] = *reinterpret_cast<const f32x2_t*>(p);
                else w[i].x = *p;
                keep_single();
            }
#pragma unroll
            for (int i = 0; i < kRunMore; ++i) {
                const bool in = run0 + kRunAhead + i < run1;
                accr += in ? (Acc)w[i].x : (Acc)0;
                if (X == 1) acci += in ? (Acc)w[i].y : (Acc)0;
            }
            for (int s = run0 + kRunAhead + kRunMore; s < run1; ++s) {
                const float* p = l2r + l2off + 2 * (s - run0);
                accr += p[0];
                if (X == 1) acci += p[1];
            }
        }
        if (t2 < ntask2 && j2 < cnt2) {
            SPIIR_AS_GLOBAL float* zp = zrow + 2 * k2;
            if (X == 1) *reinterpret_cast<SPIIR_AS_GLOBAL f32x2_t*>(zp) = f32x2_t{(float)accr, (float)acci};
            else *zp = (float)accr;
        }
        if (more_tasks)
            for (int task = t2 + NT; task < ntask2; task += NT) {
                const int p = task / (kComp * kTile), j = (task / kComp) & (kTile - 1), c = task & (kComp - 1);
                if (j >= cnt2) continue;
                const int2 rr = prun[p];
                Acc sr = 0, si = 0;
                for (int s = rr.x; s < rr.y; ++s) {
                    const float* v = l2r + 2 * (j * nrun + s) + c;
                    sr += v[0];
                    if (X == 1) si += v[1];
                }
                SPIIR_AS_GLOBAL float* zp = reinterpret_cast<SPIIR_AS_GLOBAL float*>(piece_row(pzoff[p]) + k2 + j) + c;
                zp[0] = (float)sr;
                if (X == 1) zp[1] = (float)si;
            }
    };
    auto unflip = [&](float r, float i) { return flip ? c32{i, r} : c32{r, i}; };
    int boundary = to_boundary;  // block sample where the chunk in progress ends (DUAL)
    // after block sample kend - 1: the carry correction, as in k_filter; DUAL,
    // at a chunk's end: the next one's start state (k_chain's arithmetic)
    auto correct = [&](int kend) {
        if (((s0h + kend) & cmask) != 0) return;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            yr[f] += ur[f];
            yi[f] += ui[f];
            ur[f] = fmaf(dr[f], yr[f], -(di[f] * yi[f]));
            ui[f] = fmaf(dr[f], yi[f], di[f] * yr[f]);
            if (DUAL) {
                er[f] += eur[f];
                ei[f] += eui[f];
                eur[f] = fmaf(dr[f], er[f], -(di[f] * ei[f]));
                eui[f] = fmaf(dr[f], ei[f], di[f] * er[f]);
            }
        }
        if (!dual || kend != boundary) return;
        boundary += lc;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            const int64_t g = slot0_ + (int64_t)f * L;
            c32 st = gmem(bd->s)[g], al = cmem(bd->al)[g], dl_ = cmem(bd->al)[bd->n_slots + g];
            if (flip) {
                st = c32{st.y, st.x};
                al.y = -al.y;
                dl_.y = -dl_.y;
            }
            const float ux = fmaf(dl_.x, st.x, fmaf(-dl_.y, st.y, er[f]));
            const float uy = fmaf(dl_.x, st.y, fmaf(dl_.y, st.x, ei[f]));
            st = c32{fmaf(al.x, st.x, fmaf(-al.y, st.y, ux)), fmaf(al.x, st.y, fmaf(al.y, st.x, uy))};
            if (ln < wg.lanes) gmem(bd->s)[g] = unflip(st.x, st.y);
            er[f] = ei[f] = eur[f] = eui[f] = 0.0f;
            if (kend < nh) {
                yr[f] = st.x;
                yi[f] = st.y;
                ur[f] = fmaf(dr[f], yr[f], -(di[f] * yi[f]));
                ui[f] = fmaf(dr[f], yi[f], di[f] * yr[f]);
            }
        }
    };
    // the pipeline one step on, after tile (k, cnt)
    auto advance = [&](int k, int cnt) {
        __syncthreads();
        k2 = k1; cnt2 = cnt1;
        k1 = k; cnt1 = cnt;
        parity ^= 1;
    };
    // levels 1 and 2 alone: idle waves, and the end of the block
    auto levels = [&]() {
        if (!idle) {
            load1();
            if (wave_single_run) level1(std::true_type{});
            else level1(std::false_type{});
        }
        if (duty) {
            load2();
            level2();
        }
    };

    for (int kb = ch.k0; kb < ch.k1; kb += S) {
        const int sub = min(S, ch.k1 - kb);
        const int64_t origin = ((s0h + kb - wg.maxd - 1) >> 6) << 6;
        const int wn = (int)(s0h + kb + sub - origin);
        __syncthreads();
        if (stages)
            stage_window(E0, two_copies ? E1 : nullptr, wn, [&](int i) {
                const int64_t a = origin + i;  // (a past the block's end is not used)
                const SPIIR_AS_CONST float* p = a < s0 ? ring + (a & mk) : xblk + min((int)(a - s0), q.n - 1);
                return *p;
            });
        else
            stage_window(E0, two_copies ? E1 : nullptr, wn, [&](int i) { return ring[(origin + i) & mk]; });
        wait_loads();
        __syncthreads();

        // the run of full tiles [ka, ke) of this window, between partial ones
        const int ka = min(kb + (int)(-(s0h + kb) & (kTile - 1)), kb + sub);
        const int ke = max(ka, kb + sub - (int)((s0h + kb + sub) & (kTile - 1)));
        const int rel0 = (int)(s0h - origin);  // window position of block sample 0

        auto partial = [&](int k, int cnt) {
            if (cnt <= 0) return;
            if (!LOCAL) levels();
            if (!idle) {
#pragma unroll 1
                for (int j = 0; j < cnt; ++j) {
                    float xs[NF], o = 0.0f;
#pragma unroll
                    for (int f = 0; f < NF; ++f) xs[f] = E0[rel0 + k + j - dl[f]];
                    split_step<X, NF, !LOCAL, DUAL>(xs, o, ar, ai, br, bi, yr, yi, er, ei);
                    if (!LOCAL && (j & (X - 1)) == px) pcol[2 * j] = o;
                }
                correct(k + cnt);
            }
            if (!LOCAL) advance(k, cnt);
        };
        auto full = [&](auto two, auto single_run) {
            const float* x1[NF];
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const int par = two.value ? dl[f] & 1 : 0;
                x1[f] = (par ? E1 : E0) + (rel0 + ka - dl[f] - par);
            }
            auto load_x = [&](int jj, int off) {  // pair jj, off samples on
#pragma unroll
                for (int f = 0; f < NF; ++f) {
                    const float* p = x1[f] + off;
                    if (two.value) xv[f][jj % kAhead] = reinterpret_cast<const f32x2_t*>(p)[jj];
                    else xv[f][jj % kAhead] = f32x2_t{p[2 * jj], p[2 * jj + 1]};
                }
                keep_single();
            };
#pragma unroll
            for (int jj = 0; jj < kAhead; ++jj) load_x(jj, 0);
            wait_lds();
#pragma unroll 1
            for (int k = ka; k < ke; k += kTile) {
                if (!LOCAL) {
                    load1();
                    if (duty) load2();
                }
                // the next tile's first pairs (after the last tile its own
                // again, which are in bounds)
                const int at = k + kTile < ke ? kTile : 0;
                float out[kTile];
#pragma unroll
                for (int jj = 0; jj < kTile / 2; ++jj) {
                    float xa[NF], xb[NF];
#pragma unroll
                    for (int f = 0; f < NF; ++f) {
                        xa[f] = xv[f][jj % kAhead].x;
                        xb[f] = xv[f][jj % kAhead].y;
                    }
                    split_step<X, NF, !LOCAL, DUAL>(xa, out[2 * jj], ar, ai, br, bi, yr, yi,
                                                           er, ei);
                    split_step<X, NF, !LOCAL, DUAL>(xb, out[2 * jj + 1], ar, ai, br, bi, yr, yi,
                                                           er, ei);
                    if (!LOCAL) {  // after load1
                        if (X == 1) {
                            pcol[4 * jj] = out[2 * jj];
                            pcol[4 * jj + 2] = out[2 * jj + 1];
                        } else if (X == 2) {
                            pcol[4 * jj + 2 * px] = px ? out[2 * jj + 1] : out[2 * jj];
                        } else if (jj & 1) {
                            const float lo2 = px & 1 ? out[2 * jj - 1] : out[2 * jj - 2];
                            const float hi2 = px & 1 ? out[2 * jj + 1] : out[2 * jj];
                            pcol[4 * jj - 4 + 2 * px] = px & 2 ? hi2 : lo2;
                        }
                    }
                    if (jj < kTile / 2 - kAhead) load_x(jj + kAhead, 0);
                    else load_x(jj - (kTile / 2 - kAhead), at);
                }
#pragma unroll
                for (int f = 0; f < NF; ++f) x1[f] += at;
                if (!LOCAL) {
                    level1(single_run);
                    if (duty) level2();
                }
                correct(k + kTile);
                if (!LOCAL) advance(k, kTile);
            }
        };

        partial(kb, ka - kb);
        if (idle) {
            if (!LOCAL)
                for (int k = ka; k < ke; k += kTile) {
                    levels();
                    advance(k, kTile);
                }
        } else if (two_copies) {
            if (LOCAL || wave_single_run) full(std::true_type{}, std::true_type{});
            else full(std::true_type{}, std::bool_constant<LOCAL>{});
        } else {
            if (LOCAL || wave_single_run) full(std::false_type{}, std::true_type{});
            else full(std::false_type{}, std::bool_constant<LOCAL>{});
        }
        partial(ke, kb + sub - ke);
    }
    if (!LOCAL) {
        // the two tiles still in flight
        for (int i = 0; i < 2; ++i) {
            levels();
            advance(0, 0);
        }
    }

    if (ln >= wg.lanes) return;  // the state of padding stays zero
    if (LOCAL) {
        SPIIR_AS_GLOBAL c32* ue = gmem(bd->uend) + (int64_t)tc * bd->n_slots;
#pragma unroll
        for (int f = 0; f < NF; ++f) {
            ue[slot0_ + (int64_t)f * L] = unflip(yr[f], yi[f]);
            if (ch.last) gmem(bd->euend)[slot0_ + (int64_t)f * L] = unflip(ur[f], ui[f]);
        }
        return;
    }
    if (!ch.last) return;  // only the block's last chunk carries its state on
    bool bad = false;
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        const int64_t g = slot0_ + (int64_t)f * L;
        gmem(bd->y)[g] = unflip(yr[f], yi[f]);
        gmem(bd->ys)[g] = unflip(ur[f], ui[f]);
        if (dual) {
            gmem(bd->ey)[g] = unflip(er[f], ei[f]);
            gmem(bd->eu)[g] = unflip(eur[f], eui[f]);
        }
        bad |= !(isfinite(yr[f]) && isfinite(yi[f]));
    }
    if (bad) {
        const int p = lmeta[ln] >> 16;
        atomicOr(&bd->flags[cmem(bd->piece)[wg.piece_base + p].tmpl], 1);
    }
}

// ---------------------------------------------------------------------------
// The filter bank on the matrix cores (single-rate banks; engine MFMA).
//
// Over a chunk of T = 8 samples starting at an absolute multiple of 8 (c is
// the chunk, Y_l[c] filter l's state before it), Eq. 6 applied to Eq. 7 gives
//   y_l[8c + t] = a_l^(t+1) Y_l[c] + sum_{s<=t} b_l a_l^(t-s) x[8c + s - d_l],
// so the sum over filters (Eq. 8) of one chunk is two matrix products with
// rows (t, re/im): a 16 x (2 per filter) block of powers a_l^(t+1) times the
// chunk states, and a 16 x (8 per filter) lower-triangular Toeplitz block of
// b_l a_l^(t-s) times the chunk's delayed inputs.  Both go through
// v_mfma_f32_16x16x32_f16 over 16 chunks at a time, each operand split into
// an fp16 high part and the fp16 rounding of the remainder (hi*hi + hi*lo +
// lo*hi, FP32 accumulation; the coefficients scaled by a power of two that
// keeps them in the fp16 range).  The vector units carry the states from
// chunk to chunk, Y[c+1] = a^8 Y[c] + sum_s b a^(7-s) x[8c + s - d], with the
// carry correction of the per-sample form applied every C/8 chunks.
//
// One workgroup of 256 threads per (template, up to 256 of its filters);
// thread i runs the chunk chain of filter i, wave w owns filters
// 64w .. 64w+63 in the products.  The input window is staged once per
// sub-block already split, as fp16 high and low parts, each held twice (the
// second copy one sample ahead) so that 8 samples from any position are four
// aligned 32-bit reads.  Per 128-sample tile: the chain stores the 16 chunk
// states (scaled, split) in LDS; each wave multiplies its filters' blocks;
// the four waves' partial sums are added in LDS and written as the piece's
// band output.
// LDS: Xh0 Xh1 Xl0 Xl1 [xcap] fp16 each | Yh [16][kMfmaYRow] half2 | Yl [same] | zp [4][16][kMfmaZRow] f32
// (rows padded so that the 16 chunks of a column read, and the 4 row groups
// of a partial-sum store, fall in different banks)
// ---------------------------------------------------------------------------
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
constexpr int kMfmaK2 = 16;    // Toeplitz K-blocks per wave (4 filters x 8 samples each)
constexpr int kMfmaK1 = 4;     // state K-blocks per wave (16 filters x re/im each)
constexpr int kMfmaSP = 14;    // log2 scale of the powers a1^(t+1)
constexpr int kMfmaSY = 8;     // log2 scale of the chunk states
constexpr int kMfmaYRow = kMfmaSlots + 4;  // words per chunk row of the state tile
constexpr int kMfmaZRow = 17;              // words per row of a wave's partial sums

__device__ __forceinline__ void split16(float v, _Float16& hi, _Float16& lo)
{
    hi = (_Float16)v;
    lo = (_Float16)(v - (float)hi);
}

__device__ __forceinline__ uint32_t pack_h2(_Float16 a, _Float16 b)
{
    return (uint32_t)__builtin_bit_cast(uint16_t, a) | ((uint32_t)__builtin_bit_cast(uint16_t, b) << 16);
}

// 8 fp16 values from position p of a window held twice (X1 one ahead of X0):
// four aligned 32-bit reads
__device__ __forceinline__ half8_t load8h(const _Float16* X0, const _Float16* X1, int p)
{
    const uint32_t* w = reinterpret_cast<const uint32_t*>((p & 1) ? X1 + p - 1 : X0 + p);
    const uint4 v = make_uint4(w[0], w[1], w[2], w[3]);
    return __builtin_bit_cast(half8_t, v);
}

__global__ void __launch_bounds__(kMfmaSlots, 2) k_filter_mfma(LaunchArgs args)
{
    extern __shared__ float sm[];
    const int bid = blockIdx.x;
    int lo = 0, hi = args.nseg;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (args.cum[mid] <= bid) lo = mid;
        else hi = mid;
    }
    const ReqArg& q = args.req[args.seg_req[lo]];
    CBankDev* bd = cmem(q.bd);
    const WgDesc wg = cmem(bd->wg)[bd->band_wg0[0] + (bid - args.cum[lo])];
    const PieceDesc pd = cmem(bd->piece)[wg.piece_base];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int n = q.n;
    const int64_t s0 = cmem(bd->clock)[0];
    const int xcap = bd->xcap;  // a multiple of 32 samples
    _Float16* Xh0 = reinterpret_cast<_Float16*>(sm);
    _Float16* Xh1 = Xh0 + xcap;
    _Float16* Xl0 = Xh1 + xcap;
    _Float16* Xl1 = Xl0 + xcap;
    uint32_t* Yh = reinterpret_cast<uint32_t*>(Xl1 + xcap);
    uint32_t* Yl = Yh + 16 * kMfmaYRow;
    float* zp = reinterpret_cast<float*>(Yl + 16 * kMfmaYRow);

    // chunk chain of filter slot tid
    const int64_t g = wg.slot_base + tid;
    const SPIIR_AS_CONST c32* kc = cmem(bd->kc);
    const SPIIR_AS_CONST c32* pw = cmem(bd->pw);
    c32 Y = gmem(bd->y)[g], u = gmem(bd->ys)[g];
    const c32 a8 = cmem(bd->a)[g], dc = cmem(bd->dc)[g];
    const int dA = cmem(bd->off)[g];
    float wr[kMfmaT], wi[kMfmaT];  // b a^(7-s): weight of sample s in the chunk's end state
#pragma unroll
    for (int s = 0; s < kMfmaT; ++s) {
        const c32 k = kc[g * kMfmaT + (kMfmaT - 1 - s)];
        wr[s] = k.x;
        wi[s] = k.y;
    }
    const int64_t cmask = bd->C - 1;

    // matrix operands of this wave: row r = (t, part), column group g4
    const int r = lane & 15, g4 = lane >> 4, t = r & 7, part = r >> 3, col = lane & 15;
    const float sA = ldexpf(1.0f, wg.scale);
    half8_t Ah[kMfmaK2], Al[kMfmaK2], Ph[kMfmaK1], Pl[kMfmaK1];
    int dB[kMfmaK2];
#pragma unroll
    for (int kb = 0; kb < kMfmaK2; ++kb) {
        const int64_t gf = wg.slot_base + wave * 64 + 4 * kb + g4;
#pragma unroll
        for (int s = 0; s < kMfmaT; ++s) {
            const c32 k = kc[gf * kMfmaT + ((t - s) & (kMfmaT - 1))];
            const float v = s <= t ? (part ? k.y : k.x) * sA : 0.0f;
            _Float16 h, l;
            split16(v, h, l);
            Ah[kb][s] = h;
            Al[kb][s] = l;
        }
        dB[kb] = cmem(bd->off)[gf];
    }
#pragma unroll
    for (int kb = 0; kb < kMfmaK1; ++kb) {
#pragma unroll
        for (int j = 0; j < 8; ++j) {
            const int64_t gf = wg.slot_base + wave * 64 + 16 * kb + 4 * g4 + (j >> 1);
            const c32 p = pw[gf * kMfmaT + t];
            // row (t, re): Re p Re Y - Im p Im Y;  row (t, im): Im p Re Y + Re p Im Y
            const float v = part == 0 ? ((j & 1) ? -p.y : p.x) : ((j & 1) ? p.x : p.y);
            _Float16 h, l;
            split16(ldexpf(v, kMfmaSP), h, l);
            Ph[kb][j] = h;
            Pl[kb][j] = l;
        }
    }
    const float unA = ldexpf(1.0f, -wg.scale), unP = ldexpf(1.0f, -(kMfmaSP + kMfmaSY));
    const float sY = ldexpf(1.0f, kMfmaSY);

    const int S = bd->S[0];
    const SPIIR_AS_CONST float* ring = cmem(bd->rings) + bd->ring_off[0];
    const int64_t mk = bd->ring_mask[0];
    SPIIR_AS_GLOBAL float* zout = reinterpret_cast<SPIIR_AS_GLOBAL float*>(gmem(q.zw) + pd.zoff);
    bool sat = false;
    for (int kb0 = 0; kb0 < n; kb0 += S) {
        const int sub = min(S, n - kb0);
        const int64_t origin = ((s0 + kb0 - wg.maxd - 1) >> 6) << 6;
        const int wn = (int)(s0 + kb0 + sub - origin);
        __syncthreads();
        // thread j writes word j of each copy: samples (2j, 2j+1) of X*0 and
        // (2j+1, 2j+2) of X*1, from x[origin + 2j .. origin + 2j + 2]
        uint32_t* Wh0 = reinterpret_cast<uint32_t*>(Xh0);
        uint32_t* Wh1 = reinterpret_cast<uint32_t*>(Xh1);
        uint32_t* Wl0 = reinterpret_cast<uint32_t*>(Xl0);
        uint32_t* Wl1 = reinterpret_cast<uint32_t*>(Xl1);
        for (int j = tid; 2 * j < wn; j += kMfmaSlots) {
            const int i = 2 * j;
            const float v0 = ring[(origin + i) & mk];
            const float v1 = i + 1 <= wn ? ring[(origin + i + 1) & mk] : 0.0f;
            const float v2 = i + 2 <= wn ? ring[(origin + i + 2) & mk] : 0.0f;
            _Float16 h0, l0, h1, l1, h2, l2;
            split16(v0, h0, l0);
            split16(v1, h1, l1);
            split16(v2, h2, l2);
            Wh0[j] = pack_h2(h0, h1);
            Wl0[j] = pack_h2(l0, l1);
            Wh1[j] = pack_h2(h1, h2);
            Wl1[j] = pack_h2(l1, l2);
        }
        __syncthreads();
        for (int k0 = kb0; k0 < kb0 + sub; k0 += kMfmaTile) {
            const int rel0 = (int)(s0 + k0 - origin);  // window position of the tile's first sample
            // chunk chain, four chunks at a time: their input sums first
            // (independent), then the states in order, each stored (scaled,
            // split) before its chunk
#pragma unroll 1
            for (int c4 = 0; c4 < 16; c4 += 4) {
            float er[4], ei[4];
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) {
                const int p = rel0 + kMfmaT * (c4 + cc) - dA;
                const half8_t xh = load8h(Xh0, Xh1, p);
                const half8_t xl = load8h(Xl0, Xl1, p);
                float ar = 0.0f, ai = 0.0f, br = 0.0f, bi = 0.0f;
#pragma unroll
                for (int s = 0; s < kMfmaT; ++s) {
                    const float x = (float)xh[s] + (float)xl[s];
                    if (s & 1) {
                        br = fmaf(wr[s], x, br);
                        bi = fmaf(wi[s], x, bi);
                    } else {
                        ar = fmaf(wr[s], x, ar);
                        ai = fmaf(wi[s], x, ai);
                    }
                }
                er[cc] = ar + br;
                ei[cc] = ai + bi;
            }
#pragma unroll
            for (int cc = 0; cc < 4; ++cc) {
                const int c = c4 + cc;
                _Float16 hr, lr, hi_, li;
                const float yr = Y.x * sY, yi = Y.y * sY;
                sat |= !(fabsf(yr) < 32768.0f && fabsf(yi) < 32768.0f);
                split16(yr, hr, lr);
                split16(yi, hi_, li);
                Yh[c * kMfmaYRow + tid] = pack_h2(hr, hi_);
                Yl[c * kMfmaYRow + tid] = pack_h2(lr, li);
                const float nr = fmaf(a8.x, Y.x, fmaf(-a8.y, Y.y, er[cc]));
                const float ni = fmaf(a8.x, Y.y, fmaf(a8.y, Y.x, ei[cc]));
                Y = c32{nr, ni};
                if (((s0 + k0 + kMfmaT * (c + 1)) & cmask) == 0) {
                    Y.x += u.x;
                    Y.y += u.y;
                    u = c32{fmaf(dc.x, Y.x, -dc.y * Y.y), fmaf(dc.x, Y.y, dc.y * Y.x)};
                }
            }
            }
            __syncthreads();
            // the wave's filters: Toeplitz input part and state part of 16 chunks,
            // in independent accumulators
            f32x4_t D2[4], D1[2];
#pragma unroll
            for (int i = 0; i < 4; ++i) D2[i] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int i = 0; i < 2; ++i) D1[i] = f32x4_t{0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
            for (int kb = 0; kb < kMfmaK2; ++kb) {
                const int p = rel0 + kMfmaT * col - dB[kb];
                const half8_t bh = load8h(Xh0, Xh1, p);
                const half8_t bl = load8h(Xl0, Xl1, p);
                f32x4_t& D = D2[kb & 3];
                D = __builtin_amdgcn_mfma_f32_16x16x32_f16(Ah[kb], bh, D, 0, 0, 0);
                D = __builtin_amdgcn_mfma_f32_16x16x32_f16(Ah[kb], bl, D, 0, 0, 0);
                D = __builtin_amdgcn_mfma_f32_16x16x32_f16(Al[kb], bh, D, 0, 0, 0);
            }
#pragma unroll
            for (int kb = 0; kb < kMfmaK1; ++kb) {
                const int f0 = wave * 64 + 16 * kb + 4 * g4;
                const uint4 hv = *reinterpret_cast<const uint4*>(Yh + col * kMfmaYRow + f0);
                const uint4 lv = *reinterpret_cast<const uint4*>(Yl + col * kMfmaYRow + f0);
                const half8_t bh = __builtin_bit_cast(half8_t, hv);
                const half8_t bl = __builtin_bit_cast(half8_t, lv);
                f32x4_t& D = D1[kb & 1];
                D = __builtin_amdgcn_mfma_f32_16x16x32_f16(Ph[kb], bh, D, 0, 0, 0);
                D = __builtin_amdgcn_mfma_f32_16x16x32_f16(Ph[kb], bl, D, 0, 0, 0);
                D = __builtin_amdgcn_mfma_f32_16x16x32_f16(Pl[kb], bh, D, 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const float v2 = (D2[0][i] + D2[1][i]) + (D2[2][i] + D2[3][i]);
                zp[(wave * 16 + 4 * g4 + i) * kMfmaZRow + col] = fmaf(v2, unA, (D1[0][i] + D1[1][i]) * unP);
            }
            __syncthreads();
            // sum of the four waves' partials: element (row, chunk) = (tid >> 4, tid & 15)
            {
                const int row = tid >> 4, ch = tid & 15;
                const float* zr = zp + row * kMfmaZRow + ch;
                const float v = (zr[0] + zr[16 * kMfmaZRow]) + (zr[32 * kMfmaZRow] + zr[48 * kMfmaZRow]);
                zout[2 * (int64_t)(k0 + kMfmaT * ch + (row & 7)) + (row >> 3)] = v;
            }
        }
    }
    gmem(bd->y)[g] = Y;
    gmem(bd->ys)[g] = u;
    if (sat || !(isfinite(Y.x) && isfinite(Y.y))) atomicOr(&bd->flags[pd.tmpl], 1);
}

// ---------------------------------------------------------------------------
// Upsample-and-add chain, one workgroup of kUpThreads per (request, template).
// The piece sums of bands 1.. are fetched into registers first (one burst of
// independent loads), band 0's once the lowest band is in LDS, so they arrive
// while the chain runs from LDS, lowest band first.  A thread owns low-rate
// samples m = tid + kUpThreads*i of acc_{h+1} and writes both polyphase
// outputs acc_h[2m] and acc_h[2m+1] from the same window.
// LDS: cur [hu_len + max_block/2] c32 | nxt [same] | histories of bands
// 1..H-2 [(H-2) hu_len] c32 | taps [tu]
// ---------------------------------------------------------------------------
constexpr int kUpThreads = 256;
constexpr int kUpFastTaps = 32;  // interpolator length with an unrolled path

// low-rate samples per thread for the boundary between band h and h+1
__host__ __device__ constexpr int up_slots(int h)
{
    return (kInnerBlock >> (h + 1)) / kUpThreads > 1 ? (kInnerBlock >> (h + 1)) / kUpThreads : 1;
}
__host__ __device__ constexpr int up_slot_base(int h)
{
    return h == 0 ? 0 : up_slot_base(h - 1) + up_slots(h - 1);
}
constexpr int kUpSlotsTotal = up_slot_base(kMaxBands);
// sample pairs (2m, 2m+1) of band h in a block of n base-rate samples
__device__ __forceinline__ int up_pairs(int n, int h) { return ((n >> h) + 1) >> 1; }

// Adds piece p of band h's segment to the thread's slots of pv (piece 0 is
// loaded into the zeroed slots, the others are added in piece order).
__device__ __forceinline__ void up_load(float4 (&pv)[kUpSlotsTotal], int h, const SPIIR_AS_CONST c32* zw,
                                        const SegDesc& sg, int64_t zstride, int n, int tid, int p)
{
    if (sg.npiece <= p) return;
    const SPIIR_AS_CONST float4* row =
        reinterpret_cast<const SPIIR_AS_CONST float4*>(zw + sg.zoff + p * zstride);
#pragma unroll
    for (int i = 0; i < up_slots(h); ++i) {
        const int m = tid + kUpThreads * i;
        if (m < up_pairs(n, h)) {
            const float4 u = row[m];
            float4& v = pv[up_slot_base(h) + i];
            if (p == 0) {
                v = u;
            } else {
                v.x += u.x;
                v.y += u.y;
                v.z += u.z;
                v.w += u.w;
            }
        }
    }
}

__device__ __forceinline__ c32 piece_sum(const SPIIR_AS_CONST c32* zw, const SegDesc& sg, int64_t stride, int k)
{
    float vr = 0.0f, vi = 0.0f;
    for (int p = 0; p < sg.npiece; ++p) {
        const c32 u = zw[sg.zoff + p * stride + k];
        vr += u.x;
        vi += u.y;
    }
    return c32{vr, vi};
}

// Trigger reduction of one template's block (the step after the filter in the
// search pipeline, §5): the largest |z|^2, the first sample attaining it and
// the number of samples at or above a threshold.  |z|^2 is re*re + im*im with
// each product and the sum rounded to FP32 (no contraction), so a caller can
// repeat the decision exactly from the FP32 output.
struct PeakAcc {
    float v = -1.0f;
    int i = INT_MAX;
    int cnt = 0;
    __device__ __forceinline__ void add(float re, float im, int k, float thr2)
    {
#pragma clang fp contract(off)
        const float m = re * re + im * im;  // two rounded products, one rounded sum
        if (m > v) {  // a thread visits its samples in increasing order
            v = m;
            i = k;
        }
        cnt += m >= thr2 ? 1 : 0;
    }
    __device__ __forceinline__ void merge(float ov, int oi, int oc)
    {
        if (ov > v || (ov == v && oi < i)) {
            v = ov;
            i = oi;
        }
        cnt += oc;
    }
};

// `lds`: 12 words of the kernel's dynamic LDS that no thread reads any more
// (the kernel keeps no static LDS, so its dynamic limit can be raised to the
// full 160 KB).
__device__ void peak_store(PeakAcc a, const ReqArg& q, int t, int tid, float* lds)
{
    float* sv = lds;
    int* si = reinterpret_cast<int*>(lds + kUpThreads / 64);
    int* sc = si + kUpThreads / 64;
    for (int off = 32; off >= 1; off >>= 1)
        a.merge(__shfl_xor(a.v, off), __shfl_xor(a.i, off), __shfl_xor(a.cnt, off));
    if ((tid & 63) == 0) {
        sv[tid >> 6] = a.v;
        si[tid >> 6] = a.i;
        sc[tid >> 6] = a.cnt;
    }
    __syncthreads();
    if (tid != 0) return;
    for (int w = 1; w < kUpThreads / 64; ++w) a.merge(sv[w], si[w], sc[w]);
    SPIIR_AS_GLOBAL spiir_peak* pk = gmem(q.peaks) + t;
    float v = a.v;
    int idx = a.i == INT_MAX ? -1 : q.c0 + a.i;
    int cnt = a.cnt;
    if (q.c0 > 0) {  // later chunk of the caller's block: combine with the earlier ones
        const spiir_peak old = *pk;
        if (!(idx >= 0 && (old.index < 0 || v > old.peak2))) {
            v = old.peak2;
            idx = old.index;
        }
        cnt += old.n_above;
    }
    *pk = spiir_peak{v, idx, cnt, 0};
}

__global__ void __launch_bounds__(kUpThreads, 4) k_upadd(LaunchArgs args)
{
    extern __shared__ float sm[];
    const int bid = blockIdx.x;
    int r = 0;
    while (r + 1 < args.nreq && args.tcum[r + 1] <= bid) ++r;
    const ReqArg& q = args.req[r];
    CBankDev* bd = cmem(q.bd);
    const int t = bid - args.tcum[r];
    const int tid = threadIdx.x;
    const int H = bd->H, n = q.n, HU = bd->hu_len, tu = bd->tu, MB = bd->max_block;
    const SPIIR_AS_CONST SegDesc* seg = cmem(bd->seg) + (int64_t)t * H;
    const SPIIR_AS_CONST c32* zw = cmem(q.zw);
    SPIIR_AS_GLOBAL c32* zrow = q.z ? gmem(q.z) + (int64_t)t * q.ldz : nullptr;
    const bool peaks = q.peaks != nullptr;
    PeakAcc acc;
    // The common 32-tap interpolator reads its taps as uniform scalar loads
    // and runs the tap loop unrolled; other lengths read the taps from LDS.
    // Both add the terms in the same order, so they give the same bits.
    const bool taps32 = tu == kUpFastTaps;
    const SPIIR_AS_CONST float* tap = cmem(bd->hu);

    if (H == 1) {
        const SegDesc sg = seg[0];
        if (q.z_direct && sg.npiece == 1) return;  // written by the filter kernel
        for (int k = tid; k < n; k += kUpThreads) {
            const c32 v = piece_sum(zw, sg, bd->zstride[0], k);
            if (zrow) zrow[k] = v;
            if (peaks) acc.add(v.x, v.y, k, q.thr2);
        }
        if (peaks) peak_store(acc, q, t, tid, sm);  // this path uses no other LDS
        return;
    }

    const int ext = HU + MB / 2;
    c32* cur = reinterpret_cast<c32*>(sm);
    c32* nxt = cur + ext;
    c32* hl = nxt + ext;  // histories of bands 1..H-2, loaded once up front
    float* hu = reinterpret_cast<float*>(hl + (H - 2) * HU);
    for (int i = tid; i < tu; i += kUpThreads) hu[i] = tap[i];
    const SPIIR_AS_GLOBAL c32* hist_in = gmem(bd->uphist) + ((int64_t)t * H + 1) * HU;
    for (int i = tid; i < (H - 2) * HU; i += kUpThreads) hl[i] = hist_in[i];

    // Every band's own output, as sample pairs (2m, 2m+1) (the lowest band may
    // end on an unpaired sample; its partner is a workspace word that is read
    // but not used).  Bands 1.. are loaded for all slots at once (independent
    // loads, one wait), then the other pieces of split segments are added.
    // Band 0, the largest, is loaded once the lowest band is in place, so its
    // loads are in flight while the chain runs through the lower bands.
    float4 pv[kUpSlotsTotal];
#pragma unroll
    for (int h = 0; h < kMaxBands; ++h)
#pragma unroll
        for (int i = 0; i < up_slots(h); ++i) pv[up_slot_base(h) + i] = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
#pragma unroll
    for (int h = 1; h < kMaxBands; ++h)
        if (h < H) up_load(pv, h, zw, seg[h], bd->zstride[h], n, tid, 0);
#pragma unroll
    for (int h = 1; h < kMaxBands; ++h) {
        if (h >= H) continue;
        const SegDesc sg = seg[h];
        for (int p = 1; p < sg.npiece; ++p) up_load(pv, h, zw, sg, bd->zstride[h], n, tid, p);
    }

    // lowest band: acc_{H-1} = z_{H-1}, placed after its history
    {
        const int nh = n >> (H - 1);
        SPIIR_AS_GLOBAL c32* hist = gmem(bd->uphist) + ((int64_t)t * H + H - 1) * HU;
        for (int i = tid; i < HU; i += kUpThreads) cur[i] = hist[i];
#pragma unroll
        for (int h = 1; h < kMaxBands; ++h) {
            if (h == H - 1) {
#pragma unroll
                for (int i = 0; i < up_slots(h); ++i) {
                    const int m = tid + kUpThreads * i;
                    if (m < up_pairs(n, h)) {
                        const float4 v = pv[up_slot_base(h) + i];
                        cur[HU + 2 * m] = c32{v.x, v.y};
                        if (2 * m + 1 < nh) cur[HU + 2 * m + 1] = c32{v.z, v.w};
                    }
                }
            }
        }
        __syncthreads();
        for (int i = tid; i < HU; i += kUpThreads) hist[i] = cur[nh + i];
    }
    up_load(pv, 0, zw, seg[0], bd->zstride[0], n, tid, 0);

    const int ne = HU, no = tu / 2;  // even and odd polyphase tap counts
#pragma unroll
    for (int h = kMaxBands - 2; h >= 0; --h) {
        if (h <= H - 2) {
            const int nh = n >> h, nlo = n >> (h + 1);
            SPIIR_AS_GLOBAL c32* hist = gmem(bd->uphist) + ((int64_t)t * H + h) * HU;
            if (h > 0)
                for (int i = tid; i < HU; i += kUpThreads) nxt[i] = hl[(h - 1) * HU + i];
            if (h == 0)
                for (int p = 1; p < seg[0].npiece; ++p) up_load(pv, 0, zw, seg[0], bd->zstride[0], n, tid, p);
            // all of the thread's slots hold samples of this block
            const bool full = nlo >= kUpThreads * up_slots(h);
#pragma unroll
            for (int i = 0; i < up_slots(h); ++i) {
                const int m = tid + kUpThreads * i;
                if (full || m < nlo) {
                    const float4 v = pv[up_slot_base(h) + i];
                    float er = v.x, ei = v.y, orr = v.z, oi = v.w;
                    const c32* a = cur + HU + m;
                    if (taps32) {
                        // the whole window first (independent LDS reads), then the taps
                        c32 u[kUpFastTaps / 2];
#pragma unroll
                        for (int j = 0; j < kUpFastTaps / 2; ++j) u[j] = a[-j];
#pragma unroll
                        for (int j = 0; j < kUpFastTaps / 2; ++j) {
                            er = fmaf(tap[2 * j], u[j].x, er);
                            ei = fmaf(tap[2 * j], u[j].y, ei);
                            orr = fmaf(tap[2 * j + 1], u[j].x, orr);
                            oi = fmaf(tap[2 * j + 1], u[j].y, oi);
                        }
                    } else {
                        for (int j = 0; j < ne; ++j) {
                            const c32 u = a[-j];
                            const float ce = hu[2 * j];
                            er = fmaf(ce, u.x, er);
                            ei = fmaf(ce, u.y, ei);
                            if (j < no) {
                                const float co = hu[2 * j + 1];
                                orr = fmaf(co, u.x, orr);
                                oi = fmaf(co, u.y, oi);
                            }
                        }
                    }
                    if (h == 0) {
                        if (zrow) {
                            zrow[2 * m] = c32{er, ei};
                            zrow[2 * m + 1] = c32{orr, oi};
                        }
                        if (peaks) {
                            acc.add(er, ei, 2 * m, q.thr2);
                            acc.add(orr, oi, 2 * m + 1, q.thr2);
                        }
                    } else {
                        nxt[HU + 2 * m] = c32{er, ei};
                        nxt[HU + 2 * m + 1] = c32{orr, oi};
                    }
                }
            }
            __syncthreads();
            if (h > 0) {
                for (int i = tid; i < HU; i += kUpThreads) hist[i] = nxt[nh + i];
                c32* tmp = cur;
                cur = nxt;
                nxt = tmp;
            }
        }
    }
    if (peaks) peak_store(acc, q, t, tid, sm);  // after the last phase's barrier
}

// ---------------------------------------------------------------------------
// Time split, middle pass: per filter slot, the start state of every chunk of
// the block, S[c+1] = a1^lc S[c] + uend[c] from the carried start of the first
// one, and what is carried on: the start state of the chunk in progress at the
// block's end and its zero-start state so far.  a1^lc is taken as fl32 plus
// the rest, so that its rounding does not add up over a slow filter's many
// chunks.  The product uses the same component formula as the recurrence, so it
// also holds for the swapped form of odd lanes.  One thread per slot; request r
// owns blocks [cum[r], cum[r+1]).
// ---------------------------------------------------------------------------
constexpr int kChainThreads = 256;
constexpr int kChainAhead = 8;

__global__ void __launch_bounds__(kChainThreads) k_chain(LaunchArgs args)
{
    const int bid = blockIdx.x;
    int r = 0;
    while (r + 1 < args.nreq && args.cum[r + 1] <= bid) ++r;
    const ReqArg& q = args.req[r];
    CBankDev* bd = cmem(q.bd);
    const int64_t s0 = cmem(bd->clock)[0];
    const int64_t g = (int64_t)(bid - args.cum[r]) * kChainThreads + threadIdx.x;
    if (q.direct == kDirectSplit && g == 0) gmem(bd->clock)[1] = s0 + q.n;
    if (g >= bd->n_slots) return;
    const int h = cmem(bd->wg)[g / ((int64_t)bd->F * bd->L)].band;
    const int nh = q.n >> h, lc = bd->lc[h];
    const int64_t s0h = s0 >> h, end = s0h + nh;
    const int64_t B = (s0h + lc - 1) / lc * lc;
    const int first_c = B == s0h ? 1 : 0;
    const int last_c = end - 1 < B ? 0 : 1 + (int)((end - 1 - B) / lc);
    const int64_t ns = bd->n_slots;
    const SPIIR_AS_CONST c32* uend = cmem(bd->uend);
    SPIIR_AS_GLOBAL c32* schain = gmem(bd->schain);
    c32 st = gmem(bd->s)[g];
    const c32 al = cmem(bd->al)[g], dl = cmem(bd->al)[ns + g];
    const bool whole = end % lc == 0;  // the last chunk ends with the block
    c32 u{0.0f, 0.0f};
    // the end states are read kChainAhead at a time: one wait for as many chunks
    for (int c0 = first_c; c0 <= last_c; c0 += kChainAhead) {
        c32 ue[kChainAhead];
#pragma unroll
        for (int i = 0; i < kChainAhead; ++i) ue[i] = uend[min(c0 + i, last_c) * ns + g];
#pragma unroll
        for (int i = 0; i < kChainAhead; ++i) {
            const int c = c0 + i;
            if (c > last_c) break;
            schain[c * ns + g] = st;
            u = ue[i];
            if (c == last_c && !whole) break;
            u.x = fmaf(dl.x, st.x, fmaf(-dl.y, st.y, u.x));
            u.y = fmaf(dl.x, st.y, fmaf(dl.y, st.x, u.y));
            st = c32{fmaf(al.x, st.x, fmaf(-al.y, st.y, u.x)), fmaf(al.x, st.y, fmaf(al.y, st.x, u.y))};
        }
    }
    gmem(bd->s)[g] = st;
    gmem(bd->ey)[g] = whole ? c32{0.0f, 0.0f} : u;
    gmem(bd->eu)[g] = whole ? c32{0.0f, 0.0f} : gmem(bd->euend)[g];
}

int launch_chain(const LaunchArgs& a, int64_t nblocks, void* stream)
{
    hipLaunchKernelGGL(k_chain, dim3((unsigned)nblocks), dim3(kChainThreads), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

// ---------------------------------------------------------------------------
// FP64 carry precompute and FP32 conversion of the tables (once, at create).
// ---------------------------------------------------------------------------
__device__ __forceinline__ c64 cmul(c64 u, c64 v)
{
    return c64{u.x * v.x - u.y * v.y, u.x * v.y + u.y * v.x};
}

__global__ void k_prep(const c64* __restrict__ a, const c64* __restrict__ b, int64_t n, int C,
                       c32* fa, c32* fb, c32* fdc, const int32_t* __restrict__ slot_lc, c32* fal)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const c64 av = a[i], bv = b[i];
    const float ar = (float)av.x, ai = (float)av.y;
    const double tr = ar, ti = ai;  // fl32(a1) carried in FP64
    double pr = 1.0, pi = 0.0, qr = 1.0, qi = 0.0;
    for (int c = 0; c < C; ++c) {
        const double npr = pr * av.x - pi * av.y, npi = pr * av.y + pi * av.x;
        const double nqr = qr * tr - qi * ti, nqi = qr * ti + qi * tr;
        pr = npr; pi = npi;
        qr = nqr; qi = nqi;
    }
    const float dcr = (float)(pr - qr), dci = (float)(pi - qi);
    // a1^lc for the time split, by repeated squaring in FP64
    c64 al{1.0, 0.0};
    if (slot_lc) {
        c64 base = av;
        for (int e = slot_lc[i]; e > 0; e >>= 1) {
            if (e & 1) al = cmul(al, base);
            base = cmul(base, base);
        }
    }
    const float alr = (float)al.x, ali = (float)al.y;
    const float rlr = (float)(al.x - (double)alr), rli = (float)(al.y - (double)ali);
    if (i & 1) {
        // odd lane (slots of a workgroup are lane-contiguous and L is even):
        // tables for the swapped state (Im y, Re y)
        fa[i] = c32{ar, -ai};
        fb[i] = c32{(float)bv.y, (float)bv.x};
        fdc[i] = c32{dcr, -dci};
        if (fal) fal[i] = c32{alr, -ali}, fal[n + i] = c32{rlr, -rli};
    } else {
        fa[i] = c32{ar, ai};
        fb[i] = c32{(float)bv.x, (float)bv.y};
        fdc[i] = c32{dcr, dci};
        if (fal) fal[i] = c32{alr, ali}, fal[n + i] = c32{rlr, rli};
    }
}

__global__ void k_fill(uint32_t* p, int64_t words)
{
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < words;
         i += (int64_t)gridDim.x * blockDim.x)
        p[i] = 0u;
}

// ---------------------------------------------------------------------------
// Launchers
// ---------------------------------------------------------------------------
int launch_stage(const LaunchArgs& a, int lds_bytes, void* stream)
{
    hipLaunchKernelGGL(k_stage, dim3(a.nreq), dim3(kStageThreads), lds_bytes, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

template <int F, bool COMP, bool LOCAL>
static int launch_filter_t(const LaunchArgs& a, int nblocks, int L, int lds_bytes,
                           hipStream_t s)
{
    hipLaunchKernelGGL((k_filter<F, COMP, LOCAL>), dim3(nblocks), dim3(L), lds_bytes, s, a);
    return (int)hipGetLastError();
}

template <int F, bool COMP>
static int allow_lds_t()
{
    int e = (int)hipFuncSetAttribute((const void*)k_filter<F, COMP, false>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, filter_max_lds());
    if (!e)
        e = (int)hipFuncSetAttribute((const void*)k_filter<F, COMP, true>,
                                     hipFuncAttributeMaxDynamicSharedMemorySize, filter_max_lds());
    return e;
}

template <int X>
static int allow_pipe_lds_t()
{
    int e = 0;
    constexpr bool kDual = X > 1;
    for (const void* k :
         {(const void*)k_filter_pipe<4, X, false, false, false>, (const void*)k_filter_pipe<4, X, true, false, false>,
          (const void*)k_filter_pipe<4, X, false, true, false>, (const void*)k_filter_pipe<4, X, false, false, kDual>,
          (const void*)k_filter_pipe<4, X, true, false, kDual>})
        if (!e) e = (int)hipFuncSetAttribute(k, hipFuncAttributeMaxDynamicSharedMemorySize, filter_max_lds());
    return e;
}

// Raises the dynamic LDS limit of the filter-kernel variants and the
// upsample-and-add kernel on the current device (done outside any launch
// sequence, so recorded sequences hold launches only).
int allow_filter_lds()
{
    int e = (int)hipFuncSetAttribute((const void*)k_upadd, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     filter_max_lds());
    if (!e)
        e = (int)hipFuncSetAttribute((const void*)k_filter_mfma, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     filter_max_lds());
    if (!e) e = allow_pipe_lds_t<1>();
    if (!e) e = allow_pipe_lds_t<2>();
    if (!e) e = allow_pipe_lds_t<4>();
    if (!e) e = allow_lds_t<1, false>();
    if (!e) e = allow_lds_t<1, true>();
    if (!e) e = allow_lds_t<2, false>();
    if (!e) e = allow_lds_t<2, true>();
    if (!e) e = allow_lds_t<4, false>();
    if (!e) e = allow_lds_t<4, true>();
    if (!e) e = allow_lds_t<6, false>();
    if (!e) e = allow_lds_t<6, true>();
    if (!e) e = allow_lds_t<8, false>();
    if (!e) e = allow_lds_t<8, true>();
    return e;
}

template <bool LOCAL>
static int launch_filter_any(int F, int precision, const LaunchArgs& a, int nblocks, int L,
                             int lds_bytes, hipStream_t s)
{
    const bool comp = precision == SPIIR_FP32_COMPENSATED;
    switch (F) {
    case 1: return comp ? launch_filter_t<1, true, LOCAL>(a, nblocks, L, lds_bytes, s)
                        : launch_filter_t<1, false, LOCAL>(a, nblocks, L, lds_bytes, s);
    case 2: return comp ? launch_filter_t<2, true, LOCAL>(a, nblocks, L, lds_bytes, s)
                        : launch_filter_t<2, false, LOCAL>(a, nblocks, L, lds_bytes, s);
    case 4: return comp ? launch_filter_t<4, true, LOCAL>(a, nblocks, L, lds_bytes, s)
                        : launch_filter_t<4, false, LOCAL>(a, nblocks, L, lds_bytes, s);
    case 6: return comp ? launch_filter_t<6, true, LOCAL>(a, nblocks, L, lds_bytes, s)
                        : launch_filter_t<6, false, LOCAL>(a, nblocks, L, lds_bytes, s);
    case 8: return comp ? launch_filter_t<8, true, LOCAL>(a, nblocks, L, lds_bytes, s)
                        : launch_filter_t<8, false, LOCAL>(a, nblocks, L, lds_bytes, s);
    default: return (int)hipErrorInvalidValue;
    }
}

int launch_filter(int F, int precision, const LaunchArgs& a, int nblocks, int L, int lds_bytes,
                  void* stream)
{
    return launch_filter_any<false>(F, precision, a, nblocks, L, lds_bytes, (hipStream_t)stream);
}

// the end-state pass of a time split (the compensated sum plays no part in it)
int launch_filter_local(int F, int precision, const LaunchArgs& a, int nblocks, int L, int lds_bytes,
                        void* stream)
{
    (void)precision;
    return launch_filter_any<true>(F, SPIIR_FP32, a, nblocks, L, lds_bytes, (hipStream_t)stream);
}

template <int X, bool COMP, bool LOCAL, bool DUAL>
static int launch_pipe_t(const LaunchArgs& a, int nblocks, int lanes, int lds_bytes, hipStream_t s)
{
    hipLaunchKernelGGL((k_filter_pipe<4, X, COMP, LOCAL, DUAL>), dim3(nblocks), dim3(lanes * X), lds_bytes, s, a);
    return (int)hipGetLastError();
}

template <int X>
static int launch_pipe_x(PipeMode mode, bool comp, const LaunchArgs& a, int nblocks, int lanes, int lds_bytes,
                         hipStream_t s)
{
    constexpr bool kDual = X > 1;  // one thread per lane has no registers left for it
    if (mode == PipeMode::kLocal) return launch_pipe_t<X, false, true, false>(a, nblocks, lanes, lds_bytes, s);
    if (mode == PipeMode::kDual)
        return !kDual ? (int)hipErrorInvalidValue
               : comp ? launch_pipe_t<X, true, false, kDual>(a, nblocks, lanes, lds_bytes, s)
                      : launch_pipe_t<X, false, false, kDual>(a, nblocks, lanes, lds_bytes, s);
    return comp ? launch_pipe_t<X, true, false, false>(a, nblocks, lanes, lds_bytes, s)
                : launch_pipe_t<X, false, false, false>(a, nblocks, lanes, lds_bytes, s);
}

int launch_filter_pipe(int X, PipeMode mode, int precision, const LaunchArgs& a, int nblocks, int lanes, int lds_bytes,
                       void* stream)
{
    const bool comp = precision == SPIIR_FP32_COMPENSATED;
    hipStream_t s = (hipStream_t)stream;
    return X == 1   ? launch_pipe_x<1>(mode, comp, a, nblocks, lanes, lds_bytes, s)
           : X == 2 ? launch_pipe_x<2>(mode, comp, a, nblocks, lanes, lds_bytes, s)
                    : launch_pipe_x<4>(mode, comp, a, nblocks, lanes, lds_bytes, s);
}

int launch_filter_mfma(const LaunchArgs& a, int nblocks, int lds_bytes, void* stream)
{
    hipLaunchKernelGGL(k_filter_mfma, dim3(nblocks), dim3(kMfmaSlots), lds_bytes, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

int launch_upadd(const LaunchArgs& a, int nblocks, int lds_bytes, void* stream)
{
    hipLaunchKernelGGL(k_upadd, dim3(nblocks), dim3(kUpThreads), lds_bytes, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

int launch_prep(const c64* a, const c64* b, int64_t n, int C, c32* fa, c32* fb, c32* fdc,
                const int32_t* slot_lc, c32* fal, void* stream)
{
    if (n <= 0) return 0;
    const int bs = 256;
    const int64_t nb = (n + bs - 1) / bs;
    hipLaunchKernelGGL(k_prep, dim3((unsigned)nb), dim3(bs), 0, (hipStream_t)stream, a, b, n, C,
                       fa, fb, fdc, slot_lc, fal);
    return (int)hipGetLastError();
}

int launch_fill(void* p, int64_t bytes, void* stream)
{
    if (bytes <= 0) return 0;
    const int64_t words = bytes / 4;
    int64_t nb = (words + 255) / 256;
    if (nb > 4096) nb = 4096;
    hipLaunchKernelGGL(k_fill, dim3((unsigned)nb), dim3(256), 0, (hipStream_t)stream,
                       (uint32_t*)p, words);
    return (int)hipGetLastError();
}

int filter_max_lds() { return 160 * 1024; }

// ---------------------------------------------------------------------------
// Static workspace of spiir_process_block_noalloc: one array per device,
// loaded with the code object and held until the process ends.  Host code
// never passes the array's name to a kernel (on the host it is a stand-in,
// not a device address); it passes the address hipGetSymbolAddress returns
// for the current device, taken once per device and kept.
// ---------------------------------------------------------------------------
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

constexpr int kMaxDevices = 64;

int scratch_ptr(int device, void** out)
{
    static std::mutex mu;
    static void* ptrs[kMaxDevices] = {};
    *out = nullptr;
    int cur = -1;
    if (device < 0 || device >= kMaxDevices) return (int)hipErrorInvalidDevice;
    hipError_t e = hipGetDevice(&cur);
    if (e != hipSuccess) return (int)e;
    if (cur != device) return (int)hipErrorInvalidDevice;  // the device must be current
    std::lock_guard<std::mutex> lk(mu);
    if (!ptrs[device]) {
        void* p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return (int)e;
        if (!p) return (int)hipErrorInvalidSymbol;
        ptrs[device] = p;
    }
    *out = ptrs[device];
    return 0;
}

}  // namespace spiir
