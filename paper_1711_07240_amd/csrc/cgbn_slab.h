// Column-slab kernels: the whole forward or backward of a group of neighbouring channels in one launch, every
// activation value read once and kept in registers while the statistics complete.
//
// The tensor is seen as a matrix: channels-last, a row is a pixel and a column a channel; NCHW with small planes, a
// row is an image and a column one value of one plane (`cpc` columns per channel).  A *slab* is `cols` neighbouring
// 16-byte vectors of every row, i.e. a few whole channels.  A workgroup of 512 threads takes one slab (SOLO) or a run
// of its rows (a *unit*; U units per slab) into registers: thread t holds vector column t % cols of rows t / cols,
// t / cols + rpp, ...
//
// SOLO, U == 1: the workgroup holds all values of its channels, so the devices' sums of Algorithm 1 and its reduce
// step are one sum inside the workgroup: no row is published, nothing is waited for, one launch and no prepared
// workspace.
//
// U > 1: a unit publishes, per channel, s = sum(x - p) and q = sum(x - a)^2 about its own centre (backward: sum dy and
// sum dy * xhat) as one 8-byte store, and counts itself in on the slab's counter; the unit that completes the count
// raises the slab's flag; every unit then fetches the slab's rows and reduces them itself in double precision and in
// a fixed order (the same in every unit), as the NCHW single-launch kernels do.  Unlike those, no wait here needs its
// siblings to be resident: a unit whose wait runs out marks itself in the slab's bitmap (unless the count completed
// meanwhile) and its workgroup moves on; the unit that completes the count finds the marks in the value its own
// arrival returned and, once it has the statistics, reads the marked units' values again and writes their results.
// So every launch drains and is right whatever else the device runs; sharing it only costs the re-reads.
#pragma once

#include "cgbn_fused.h"

namespace cgbn {

constexpr int kSlabThreads = 512;
constexpr int kSlabWaves = kSlabThreads / kWave;
constexpr int kSlabMaxRows = 12288;        // forward: (channel, unit) pairs of one slab kept in LDS while they are reduced
constexpr int kSlabMaxChannels = 128;      // channels of one slab
constexpr unsigned kSlabWaitTicks = 30000; // 100 MHz ticks (300 us) a unit waits for its siblings before it moves on ...
constexpr unsigned kSlabWaitTicksLater = 3000;   // ... once some unit of the launch has done so
constexpr unsigned long long kSlabBackstopTicks = 100000000ull;     // a second: waits that end within microseconds in a sound launch
// words of the sync area: [2] "some unit has moved on"; then per slab the counter (low half: units counted in, high
// half: units that moved on), the bitmap of units that moved on, and the flag
constexpr int kSlabMovedOn = 2;

struct SlabArgs {
    const void* x;
    const void* dy;       // backward: dy; forward: the shortcut
    const void* aux;      // backward: the stored output y (ReLU)
    void* out;
    void* out2;           // dz, the shortcut's gradient (may be null)
    const float* gamma;
    const float* beta;
    float* mean;          // forward: out; backward: in
    float* mean_lo;       // forward: the caller's optional output; backward: in, may be null
    float* invstd;
    float* dgamma;
    float* dbeta;
    unsigned* rows;       // [slab][unit][channel] pairs of floats
    unsigned* sync;
    long long R;          // rows of the matrix
    long long row_bytes;
    double M, inv_M_f64, eps;
    float inv_M;
    int vecs;             // 16-byte vectors per row
    int cols, ncols;      // vector columns of a slab, its element columns
    int pow2;             // cols is a power of two <= 64: row lanes are folded inside the wavefronts first
    int rpp;              // rows per pass
    int rch;                  // channels per slab
    int cpc, nch, nsh, tpc;   // columns per channel, rch rounded up to a power of two 2^nsh, threads that add one channel's partial sums
    int C, slabs, U, rpu; // rpu: rows per unit
    int total_units;
    int inflight;         // slabs whose units the grid holds at once
    long long pivot_stride;   // elements between the first values of consecutive channels
    int nt;
    unsigned spin_limit;
    unsigned bitmap_words;    // per slab
    unsigned cpc_magic;       // 2^32 / cpc, rounded up: i / cpc is the high word of i * cpc_magic for the small i here
};

// LDS of a workgroup; SOLO needs no staging for other units' rows
template <bool SOLO, bool STAGE> struct SlabLds {
    float part[2][kSlabThreads * 8];                     // [row lane or wavefront][column]
    float rows[2][STAGE ? kSlabMaxRows : 1];             // forward: the thread's own pairs between the two passes over them
    double dsum[SOLO ? 1 : 2][SOLO ? 1 : kSlabThreads];
    double mean[SOLO ? 1 : kSlabMaxChannels];
    float piv[kSlabMaxChannels], ctr[kSlabMaxChannels];  // forward: pivot and the unit's centre
    float k0[kSlabMaxChannels], k1[kSlabMaxChannels], k2[kSlabMaxChannels], k3[kSlabMaxChannels];   // write-out constants
    int skip, last, fix, redo;        // this unit moves on (2: rows are missing for good); it completed the count; there are units for it to finish
};

// Sums a thread's column values over the slab: the row lanes of a wavefront by shuffles (power-of-two column counts),
// then through LDS; the first of a channel's `tpc` threads (t % tpc == 0, channel t / tpc) gets the channel's sums.
template <int VEC, int Q, class LDS>
__device__ __forceinline__ void slab_sum(const SlabArgs& A, LDS& L, float (&v)[Q][VEC], int col, int r, double (&out)[Q])
{
    const int t = threadIdx.x, lane = t & (kWave - 1), w = t >> 6;
    if (A.pow2) {
        for (int off = A.cols; off < kWave; off <<= 1)
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int e = 0; e < VEC; ++e) v[q][e] += __shfl_xor(v[q][e], off);
        if (lane < A.cols)
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int e = 0; e < VEC; ++e) L.part[q][w * A.ncols + col * VEC + e] = v[q][e];
    } else if (r < A.rpp) {
#pragma unroll
        for (int q = 0; q < Q; ++q)
#pragma unroll
            for (int e = 0; e < VEC; ++e) L.part[q][r * A.ncols + col * VEC + e] = v[q][e];
    }
    __syncthreads();
    const int lanes = A.pow2 ? kSlabWaves : A.rpp;
    const int ch = t / A.tpc, sub = t & (A.tpc - 1);
#pragma unroll
    for (int q = 0; q < Q; ++q) {
        double acc = 0.0;
        if (ch * A.cpc < A.ncols) {               // (channels beyond the slab's columns hold zeros)
            if (A.cpc == 1) {
                for (int i = sub; i < lanes; i += A.tpc) acc += (double)L.part[q][i * A.ncols + ch];
            } else {
                // the channel's cpc columns of every row lane, dealt to its threads
                for (int k = sub; k < lanes * A.cpc; k += A.tpc) {
                    const int i = (int)__umulhi((unsigned)k, A.cpc_magic), j = k - i * A.cpc;
                    acc += (double)L.part[q][i * A.ncols + ch * A.cpc + j];
                }
            }
        }
        for (int off = 1; off < A.tpc; off <<= 1) acc += __shfl_xor(acc, off);
        out[q] = acc;
    }
}

__device__ __forceinline__ unsigned slab_bits(float v)      // NaN in canonical form: never the sentinel
{
    return v != v ? 0x7fc00000u : __float_as_uint(v);
}

// After a unit's rows are on their way: counts it in and waits for the slab.  Returns false if the unit moves on
// (its bitmap bit is set).  L.fix: units that moved on before this one completed the count.
template <class LDS>
__device__ __forceinline__ bool slab_hand_over(const SlabArgs& A, LDS& L, int slab, int u)
{
    unsigned* cnt = A.sync + kSyncHeader + slab;
    unsigned* bitmap = A.sync + kSyncHeader + A.C + (size_t)slab * A.bitmap_words;
    __syncthreads();                  // every wavefront has issued its row stores
    if (threadIdx.x < kWave) {
        const int lane = threadIdx.x;
        unsigned old = 0;
        if (lane == 0) old = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        const unsigned long long t0 = wall_clock64();
        unsigned long long limit = kSlabWaitTicks;
        bool up = false;
        const unsigned* rep = A.rows + (size_t)slab * A.U * A.nch * 2;
        for (unsigned polls = 0; polls < A.spin_limit; ++polls) {
            bool miss = false;
            for (int k = lane; k < A.U; k += kWave) miss |= ld_agent(rep + (size_t)k * A.nch * 2) == kRowSentinel;
            if (__ballot(miss) == 0ull) { up = true; break; }
            if ((polls & 31u) == 31u) {
                if (ld_agent(A.sync + kSlabMovedOn) != 0u) limit = kSlabWaitTicksLater;
                if (wall_clock64() - t0 > limit) break;
            }
            __builtin_amdgcn_s_sleep(2);
        }
        if (lane == 0) {
            L.skip = L.last = L.fix = 0;
            if ((old & 0xffffu) == (unsigned)(A.U - 1)) {
                L.last = 1;
                const int moved = (int)(old >> 16);
                if (moved > 0) {
                    // (their workgroups are about to set their bits: they have seen the count)
                    for (;;) {
                        int have = 0;
                        for (unsigned i = 0; i < A.bitmap_words; ++i) have += __popc(ld_agent(bitmap + i));
                        if (have >= moved) { L.fix = 1; break; }
                        if (wall_clock64() - t0 > kSlabBackstopTicks) { atomicExch(A.sync + 1, 1u); break; }
                        __builtin_amdgcn_s_sleep(1);
                    }
                }
            } else if (!up) {
                // Moving on is settled on the counter: if the count is not complete yet, whoever completes it learns of
                // this unit from the high half, and waits for its bit above.
                const unsigned seen = __hip_atomic_fetch_add(cnt, 0x10000u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                if ((seen & 0xffffu) != (unsigned)A.U) {
                    L.skip = 1;
                    atomicOr(bitmap + (u >> 5), 1u << (u & 31));
                    __hip_atomic_store(A.sync + kSlabMovedOn, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
        }
    }
    __syncthreads();
    return L.skip == 0;
}

// Adds up the slab's rows, double precision, fixed order.  Thread t fetches the pairs t, t + 512, ...: all of channel
// t % nch (nch divides 512), units t / nch, t / nch + 512 / nch, ...; `f(k, unit, first, second)` takes each in (k: the thread's k-th
// pair).  Rows still in flight are fetched again: all of them have been issued.  The bound is a backstop; when it is
// hit, L.skip = 2 makes the caller poison the statistics.
template <class LDS, class F>
__device__ __forceinline__ void slab_gather(const SlabArgs& A, LDS& L, int slab, F f)
{
    const int t = threadIdx.x, pairs = A.U * A.nch;
    const unsigned long long* src = reinterpret_cast<const unsigned long long*>(A.rows) + (size_t)slab * pairs;
    const unsigned long long t0 = wall_clock64();
    constexpr int B = 8;                                  // fetches in flight per lane
    for (int i = t; i < pairs; i += B * kSlabThreads) {
        unsigned long long v[B];
        for (;;) {
            bool missing = false;
#pragma unroll
            for (int b = 0; b < B; ++b) {
                const int j = i + b * kSlabThreads;
                v[b] = __hip_atomic_load(src + (j < pairs ? j : i), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (int b = 0; b < B; ++b) missing |= ((unsigned)v[b] == kRowSentinel) | ((unsigned)(v[b] >> 32) == kRowSentinel);
            if (!missing) break;
            if (wall_clock64() - t0 > kSlabBackstopTicks) {
                atomicExch(A.sync + 1, 1u);
                L.skip = 2;
                break;
            }
        }
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int j = i + b * kSlabThreads;
            if (j < pairs) f(j / kSlabThreads, j >> A.nsh, __uint_as_float((unsigned)v[b]), __uint_as_float((unsigned)(v[b] >> 32)));
        }
    }
}

// The threads' values of a channel added in a fixed order (lane by lane through LDS, then a tree); all of the channel's
// `tpc` threads (channel t / tpc) get the sum.
template <class LDS> __device__ __forceinline__ double slab_channel_total(const SlabArgs& A, LDS& L, double v, int slot)
{
    const int t = threadIdx.x;
    L.dsum[slot][t] = v;
    __syncthreads();
    const int ch = t / A.tpc, sub = t & (A.tpc - 1);
    double acc = 0.0;
    if (ch < A.nch)
        for (int i = sub; i < kSlabThreads / A.nch; i += A.tpc) acc += L.dsum[slot][i * A.nch + ch];
    for (int off = 1; off < A.tpc; off <<= 1) acc += __shfl_xor(acc, off);
    return acc;
}

// the next unit after `u` that moved on, -1 if there is none (the completing unit is never marked)
__device__ __forceinline__ int slab_next_moved(const SlabArgs& A, int slab, int u)
{
    const unsigned* bitmap = A.sync + kSyncHeader + A.C + (size_t)slab * A.bitmap_words;
    for (int k = u + 1; k < A.U; ++k)
        if ((ld_agent(bitmap + (k >> 5)) >> (k & 31)) & 1u) return k;
    return -1;
}

// where a workgroup's unit lies
struct SlabGeom {
    int n;                    // rows of the unit
    long long base;           // byte offset of the unit's first row, first column
};
__device__ __forceinline__ SlabGeom slab_geometry(const SlabArgs& A, int slab, int u)
{
    SlabGeom g;
    const long long row0 = (long long)u * A.rpu, left = A.R - row0;
    g.n = (int)(left < A.rpu ? left : A.rpu);
    g.base = row0 * A.row_bytes + (long long)slab * A.cols * 16;
    return g;
}

// SOLO: consecutive slabs share lines and go to one XCD (workgroups are dealt to the 8 XCDs in turn; measured, slabs of
// 64 bytes x 2100 rows, 8 MB copied through registers: 8.3 us in plain order, 5.8 so).  Bijective for any grid size.
__device__ __forceinline__ int slab_of_block(int b, int G)
{
    const int q = G >> 3, rem = G & 7, xcd = b & 7, i = b >> 3;
    return xcd * q + min(xcd, rem) + i;
}

__device__ __forceinline__ void slab_forget(u32x4& v) { asm volatile("" : "+v"(v)); }    // (see forget)

// Several units: the order in which the slabs are taken.  Those in flight together are spread evenly over the row, and a
// round moves on by one slab: neighbouring columns at a long row stride would crowd the memory channels (measured,
// the loads and stores alone, 67200 rows of 4096 bytes: eight neighbouring slabs in flight 154 us, eight spread 114; rows
// of 1024 bytes 115 either way).  Bijective for any number of slabs.
__device__ __forceinline__ int slab_of_turn(const SlabArgs& A, int turn)
{
    const int q = A.slabs / A.inflight, rem = A.slabs - q * A.inflight;
    const int k = turn / A.inflight, j = turn - k * A.inflight;
    return j * q + min(j, rem) + k;
}

template <bool NT> __device__ __forceinline__ void slab_load(const char* p, u32x4& d)
{
    d = NT ? __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(p)) : *reinterpret_cast<const u32x4*>(p);
}
__device__ __forceinline__ void slab_store(char* p, const u32x4& d, int nt)
{
    if (nt) __builtin_nontemporal_store(d, reinterpret_cast<u32x4*>(p));
    else *reinterpret_cast<u32x4*>(p) = d;
}
template <typename T> __device__ __forceinline__ void slab_unpack(const u32x4& d, float (&f)[16 / sizeof(T)])
{
    constexpr int EPW = Packed<T>::EPW;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float g[EPW];
        Packed<T>::unpack(d[q], g);
#pragma unroll
        for (int e = 0; e < EPW; ++e) f[q * EPW + e] = g[e];
    }
}
template <typename T> __device__ __forceinline__ u32x4 slab_pack(const float (&f)[16 / sizeof(T)])
{
    constexpr int EPW = Packed<T>::EPW;
    u32x4 d;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        float g[EPW];
#pragma unroll
        for (int e = 0; e < EPW; ++e) g[e] = f[q * EPW + e];
        d[q] = Packed<T>::pack(g);
    }
    return d;
}

// the slab's channel of each of a thread's columns (0 for threads beyond the slab's columns)
template <int VEC> struct SlabChannels {
    int c[VEC];
    __device__ __forceinline__ SlabChannels(const SlabArgs& A, int col)
    {
        const int c0 = col * VEC < A.ncols ? col * VEC : 0;
        if (A.cpc == 1) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) c[e] = c0 + e;
        } else {
            int q = (int)__umulhi((unsigned)c0, A.cpc_magic), rem = c0 - q * A.cpc;
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                while (rem >= A.cpc) { rem -= A.cpc; ++q; }
                c[e] = q;
                ++rem;
            }
        }
    }
    __device__ __forceinline__ int operator[](int e) const { return c[e]; }
};

// The P loads of a unit, as straight-line code: the compiler then waits for each vector where it is used, and the sums of
// the first ones run while the later ones are still in flight.  (Were a load skipped when the unit has fewer rows, the
// first use would have to wait for all loads.)  So passes beyond the unit re-read the first row of its last pass, as do
// lanes without a row: the same few lines, whose values nothing uses.
struct SlabPass {
    unsigned loff;            // uniform base + 32-bit lane offset (the host checks that it fits)
    int nr, passes;           // rows of this thread, passes of the unit
    long long step;
    __device__ __forceinline__ unsigned lane(int i) const { return i < nr ? loff : 0u; }
    __device__ __forceinline__ long long advance(int i) const { return i + 1 < passes ? step : 0; }
};
__device__ __forceinline__ SlabPass slab_pass(const SlabArgs& A, int n, bool live, int r, int col)
{
    SlabPass p;
    p.loff = fresh(live ? (unsigned)r * (unsigned)A.row_bytes + (unsigned)col * 16u : 0u);
    p.nr = live ? (n - r + A.rpp - 1) / A.rpp : 0;
    p.passes = (n + A.rpp - 1) / A.rpp;
    p.step = (long long)A.rpp * A.row_bytes;
    return p;
}

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------
// P: vectors per thread.  ACT as in the NCHW kernels; the shortcut (ACT == 2) is fetched with x where the
// registers allow (P <= 20), else while the unit is written out.
//
// Statistics.  One pass, under the loads: per column sum(x - p) and D = sum (x - p)^2 about the channel's pivot p, its
// first stored value.  With a the unit's own centre, q = sum (x - a)^2 = D - 2 (a - p) sum(x - p) + n (a - p)^2 in double
// precision.  That loses (a - p)^2 / variance times the accuracy of D, so a unit in which some channel's pivot lies more
// than 8 standard deviations from its mean makes a second pass over its registers, about a, for q.
template <typename T, int ACT, int P, bool SOLO>
__global__ __launch_bounds__(kSlabThreads, P * (ACT == 2 ? 2 : 1) <= 4 ? 4 : 2) void slab_forward(SlabArgs A)
{
    constexpr int VEC = 16 / (int)sizeof(T);
    constexpr bool EARLY = ACT == 2 && P <= 20;
    __shared__ SlabLds<SOLO, !SOLO> L;
    const int t = threadIdx.x;
    const int col = t % A.cols, r = t / A.cols;
    const int ch = t / A.tpc, sub = t & (A.tpc - 1);      // the channel this thread helps to add up
    const char* xb = static_cast<const char*>(A.x);
    const char* rb = static_cast<const char*>(A.dy);
    char* yb = static_cast<char*>(A.out);
    if (SOLO && blockIdx.x == 0 && t == 0) A.sync[1] = 0u;

    for (int unit = SOLO ? slab_of_block(blockIdx.x, gridDim.x) : (int)blockIdx.x; unit < A.total_units; unit += gridDim.x) {
        const int turn = SOLO ? unit : unit / A.U, u = SOLO ? 0 : unit - turn * A.U;
        const int slab = SOLO ? unit : slab_of_turn(A, turn);
        const int c0 = slab * A.rch;
        const bool live = r < A.rpp && slab * A.cols + col < A.vecs;
        const SlabGeom g = slab_geometry(A, slab, u);
        const SlabPass ps = slab_pass(A, g.n, live, r, col);
        u32x4 d[P], s[EARLY ? P : 1];
        // ---- pivots, then the unit's vectors
        const SlabChannels<VEC> cl(A, col);
        float piv[VEC];
        if (A.cpc == 1) {
            u32x4 pw;
            slab_load<false>(xb + (long long)slab * A.cols * 16 + (live ? (unsigned)col * 16u : 0u), pw);
            slab_unpack<T>(pw, piv);
        } else {
#pragma unroll
            for (int e = 0; e < VEC; ++e)
                piv[e] = Elem<T>::load1(static_cast<const T*>(A.x) + (long long)min(c0 + cl[e], A.C - 1) * A.pivot_stride);
        }
        float pv = 0.f, gm = 0.f, bt = 0.f;               // of the channel whose first thread this is
        if (ch < A.rch && sub == 0 && c0 + ch < A.C) {
            pv = Elem<T>::load1(static_cast<const T*>(A.x) + (long long)(c0 + ch) * A.pivot_stride);
            gm = A.gamma[c0 + ch];
            bt = A.beta[c0 + ch];
        }
        {
            const char* xu = xb + g.base;
            const char* ru = rb + g.base;
            unroll_planes<P>([&](auto i_) __attribute__((always_inline)) {
                constexpr int i = decltype(i_)::value;
                slab_load<!SOLO>(xu + ps.lane(i), d[i]);
                xu += ps.advance(i);
            });
            if constexpr (EARLY) {
                unroll_planes<P>([&](auto i_) __attribute__((always_inline)) {
                    constexpr int i = decltype(i_)::value;
                    slab_load<!SOLO>(ru + ps.lane(i), s[i]);
                    ru += ps.advance(i);
                });
            }
        }
        // ---- sums about the pivots
        float a[2][VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) a[0][e] = a[1][e] = 0.f;
        unroll_planes<P>([&](auto i_) __attribute__((always_inline)) {
            constexpr int i = decltype(i_)::value;
            if (i < ps.nr) {
                float f[VEC];
                slab_unpack<T>(d[i], f);
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const float dv = f[e] - piv[e];
                    a[0][e] += dv;
                    a[1][e] += dv * dv;
                }
            }
        });
        if (t == 0) L.redo = 0;
        double tot[2];
        slab_sum<VEC, 2>(A, L, a, col, r, tot);
        const double n_row = (double)g.n * (double)A.cpc;
        const float sf = (float)tot[0];
        const float ctr = row_centre(pv, sf, (float)n_row);
        double q;
        {
            const double off = (double)ctr - (double)pv, mm = tot[0] * tot[0] / n_row;
            q = tot[1] - off * (2.0 * tot[0] - n_row * off);
            if (ch < A.nch && sub == 0) {
                L.piv[ch] = pv;
                L.ctr[ch] = ctr;
                if (mm > 64.0 * (tot[1] - mm)) L.redo = 1;
            }
        }
        __syncthreads();
        if (L.redo) {
            float b[1][VEC];
            const SlabChannels<VEC> c2(A, (int)fresh((unsigned)col));
#pragma unroll
            for (int e = 0; e < VEC; ++e) { piv[e] = L.ctr[c2[e]]; b[0][e] = 0.f; }
            unroll_planes<P>([&](auto i_) __attribute__((always_inline)) {
                constexpr int i = decltype(i_)::value;
                if (i < ps.nr) {
                    float f[VEC];
                    slab_unpack<T>(d[i], f);
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        const float dv = f[e] - piv[e];
                        b[0][e] += dv * dv;
                    }
                }
            });
            double sq[1];
            slab_sum<VEC, 1>(A, L, b, col, r, sq);
            q = sq[0];
        }
        // ---- steps 4-5 and 9-10
        double mean, dev;
        bool ok = true, mine = true;
        if (SOLO) {
            mean = (double)pv + tot[0] * A.inv_M_f64;
            const double dd = (double)ctr - mean;
            dev = q + dd * (2.0 * (tot[0] - n_row * ((double)ctr - (double)pv)) + n_row * dd);
        } else {
            if (ch < A.nch && sub == 0)
                __hip_atomic_store(reinterpret_cast<unsigned long long*>(A.rows) + ((size_t)slab * A.U + u) * A.nch + ch,
                                   ((unsigned long long)slab_bits((float)q) << 32) | slab_bits(sf),
                                   __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            mine = slab_hand_over(A, L, slab, u);
            if (mine) {
                double acc = 0.0;
                slab_gather(A, L, slab, [&](int k, int, float sk, float qk) {
                    acc += (double)sk;
                    L.rows[0][k * kSlabThreads + t] = sk;
                    L.rows[1][k * kSlabThreads + t] = qk;
                });
                acc = slab_channel_total(A, L, acc, 0);
                mean = (double)pv + acc * A.inv_M_f64;
                if (ch < A.nch && sub == 0) L.mean[ch] = mean;
                __syncthreads();
                ok = L.skip != 2;
                const int gc = t & (A.nch - 1);           // the channel of the pairs this thread fetched
                const float p = L.piv[gc];
                const double m = L.mean[gc];
                acc = 0.0;
                for (int j = t; j < A.U * A.nch; j += kSlabThreads) {
                    const int k = j >> A.nsh;
                    const double n = (double)(k + 1 < A.U ? A.rpu : (int)(A.R - (long long)k * A.rpu)) * (double)A.cpc;
                    acc += row_sqdev(L.rows[0][j], L.rows[1][j], n, p, m);
                }
                dev = slab_channel_total(A, L, acc, 1);
            }
        }
        if (mine) {
            if (ch < A.nch && sub == 0) {
                float hi = (float)mean, lo = (float)(mean - (double)hi);
                float is = (float)rsqrt_f64(dev * A.inv_M_f64 + A.eps);
                if (!ok) hi = is = __uint_as_float(0x7fc00000u);
                const float gs = gm * is;
                L.k0[ch] = hi;
                L.k1[ch] = gs;
                L.k2[ch] = bt - gs * lo;
                if ((SOLO || L.last) && ch < A.rch && c0 + ch < A.C) {
                    A.mean[c0 + ch] = hi;
                    if (A.mean_lo) A.mean_lo[c0 + ch] = lo;
                    A.invstd[c0 + ch] = is;
                }
            }
            __syncthreads();
            // ---- step 11
            float mu[VEC], gsc[VEC], bsh[VEC];
            const SlabChannels<VEC> c3(A, (int)fresh((unsigned)col));
#pragma unroll
            for (int e = 0; e < VEC; ++e) { mu[e] = L.k0[c3[e]]; gsc[e] = L.k1[c3[e]]; bsh[e] = L.k2[c3[e]]; }
            auto value = [&](const u32x4& v, const u32x4& w) __attribute__((always_inline)) {
                float f[VEC], h[VEC];
                slab_unpack<T>(v, f);
                if constexpr (ACT == 2) slab_unpack<T>(w, h);
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    float z = (f[e] - mu[e]) * gsc[e] + bsh[e];
                    if constexpr (ACT == 2) z += h[e];
                    if (ACT != 0) z = z < 0.f ? 0.f : z;
                    f[e] = z;
                }
                return slab_pack<T>(f);
            };
            // (every load has landed, and the compiler knows it: see wait_vector_memory)
            wait_vector_memory();
            char* yu = yb + g.base;
            if constexpr (ACT == 2 && !EARLY) {
                constexpr int B = 4;
                static_assert(P % B == 0, "whole batches");
                const char* ru = rb + g.base;
                unroll_planes<P / B>([&](auto i_) __attribute__((always_inline)) {
                    constexpr int i0 = decltype(i_)::value * B;
                    if (i0 < ps.passes) {
                        u32x4 b[B];
#pragma unroll
                        for (int j = 0; j < B; ++j)
                            if (i0 + j < ps.nr) slab_load<!SOLO>(ru + j * ps.step + ps.loff, b[j]);
#pragma unroll
                        for (int j = 0; j < B; ++j)
                            if (i0 + j < ps.nr) slab_store(yu + j * ps.step + ps.loff, value(d[i0 + j], b[j]), A.nt);
                        ru += B * ps.step;
                        yu += B * ps.step;
                    }
                });
            } else {
                unroll_planes<P>([&](auto i_) __attribute__((always_inline)) {
                    constexpr int i = decltype(i_)::value;
                    if (i < ps.nr) {
                        slab_forget(d[i]);
                        slab_store(yu + ps.loff, value(d[i], s[EARLY ? i : 0]), A.nt);
                    }
                    yu += ps.step;
                });
            }
            // ---- units that moved on and are this one's to finish
            if constexpr (!SOLO) {
                for (int k = L.fix ? slab_next_moved(A, slab, -1) : -1; k >= 0; k = slab_next_moved(A, slab, k)) {
                    const SlabGeom m = slab_geometry(A, slab, k);
                    for (int i = r; live && i < m.n; i += A.rpp) {
                        const long long o = m.base + (long long)i * A.row_bytes + (long long)col * 16;
                        u32x4 v, w = {0u, 0u, 0u, 0u};
                        slab_load<false>(xb + o, v);
                        if constexpr (ACT == 2) slab_load<false>(rb + o, w);
                        slab_store(yb + o, value(v, w), 0);
                    }
                }
            }
        }
        if (!SOLO) __syncthreads();       // the hand-over's verdicts have been read by everyone
    }
}

// ---------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------
// P: vectors per thread and tensor.  ACT != 0: dy is first masked by the stored output (A.aux) being positive; the
// output's vectors are loaded beside the other two where the registers allow (P <= 10), else through the storage x takes
// afterwards.
template <typename T, int ACT, int P, bool SOLO>
__global__ __launch_bounds__(kSlabThreads, P * (ACT != 0 ? 3 : 2) <= 8 ? 4 : 2) void slab_backward(SlabArgs A)
{
    constexpr int VEC = 16 / (int)sizeof(T);
    constexpr bool THREE = ACT != 0 && P <= 10;
    __shared__ SlabLds<SOLO, false> L;
    const int t = threadIdx.x;
    const int col = t % A.cols, r = t / A.cols;
    const int ch = t / A.tpc, sub = t & (A.tpc - 1);
    const char* xb = static_cast<const char*>(A.x);
    const char* gb = static_cast<const char*>(A.dy);
    const char* ab = static_cast<const char*>(A.aux);
    char* ob = static_cast<char*>(A.out);
    char* zb = static_cast<char*>(A.out2);
    if (SOLO && blockIdx.x == 0 && t == 0) A.sync[1] = 0u;

    for (int unit = SOLO ? slab_of_block(blockIdx.x, gridDim.x) : (int)blockIdx.x; unit < A.total_units; unit += gridDim.x) {
        const int turn = SOLO ? unit : unit / A.U, u = SOLO ? 0 : unit - turn * A.U;
        const int slab = SOLO ? unit : slab_of_turn(A, turn);
        const int c0 = slab * A.rch;
        const bool live = r < A.rpp && slab * A.cols + col < A.vecs;
        const SlabGeom g = slab_geometry(A, slab, u);
        const SlabPass ps = slab_pass(A, g.n, live, r, col);
        u32x4 xd[P], gd[P], yd[THREE ? P : 1];
        auto mask = [&](u32x4& v, const u32x4& y) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 4; ++q) v[q] = mask_by_positive<T>(v[q], y[q]);
        };
        const SlabChannels<VEC> cl(A, col);
        float mu[VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) mu[e] = A.mean[min(c0 + cl[e], A.C - 1)];
        float lv = 0.f, is = 0.f, gm = 0.f;               // of the channel whose first thread this is
        if (ch < A.rch && sub == 0 && c0 + ch < A.C) {
            lv = A.mean_lo ? A.mean_lo[c0 + ch] : 0.f;
            is = A.invstd[c0 + ch];
            gm = A.gamma[c0 + ch];
        }
        {
            const char* gu = gb + g.base;
            const char* xu = xb + g.base;
            const char* yu = ab + g.base;
            unroll_planes<P>([&](auto i_) __attribute__((always_inline)) {
                constexpr int i = decltype(i_)::value;
                slab_load<!SOLO>(gu + ps.lane(i), gd[i]);
                gu += ps.advance(i);
                if constexpr (ACT == 0 || THREE) {
                    slab_load<!SOLO>(xu + ps.lane(i), xd[i]);
                    xu += ps.advance(i);
                }
                if constexpr (ACT != 0) {
                    if constexpr (THREE) slab_load<!SOLO>(yu + ps.lane(i), yd[i]);
                    else slab_load<!SOLO>(yu + ps.lane(i), xd[i]);
                    yu += ps.advance(i);
                }
            });
            if constexpr (ACT != 0 && !THREE) {           // mask; x over the stored output's storage
                SlabPass again = ps;                      // (lane offsets formed anew: kept, they would cost a register each)
                again.loff = fresh(ps.loff);
                again.nr = (int)fresh((unsigned)ps.nr);
                unroll_planes<P>([&](auto i_) __attribute__((always_inline)) {
                    constexpr int i = decltype(i_)::value;
                    mask(gd[i], xd[i]);
                    slab_forget(gd[i]);       // (or the masking moves to the sums, and y and x are both held until there)
                    slab_load<!SOLO>(xu + again.lane(i), xd[i]);
                    xu += again.advance(i);
                });
            }
        }
        float a[2][VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) a[0][e] = a[1][e] = 0.f;
        unroll_planes<P>([&](auto i_) __attribute__((always_inline)) {
            constexpr int i = decltype(i_)::value;
            if (i < ps.nr) {
                if constexpr (THREE) mask(gd[i], yd[i]);
                float fx[VEC], fg[VEC];
                slab_unpack<T>(xd[i], fx);
                slab_unpack<T>(gd[i], fg);
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    a[0][e] += fg[e];
                    a[1][e] += fg[e] * (fx[e] - mu[e]);
                }
            }
        });
        double tot[2];
        slab_sum<VEC, 2>(A, L, a, col, r, tot);
        double db, dg;
        bool ok = true, mine = true;
        if (SOLO) {
            db = tot[0];
            dg = (tot[1] - (double)lv * tot[0]) * (double)is;
        } else {
            if (ch < A.nch && sub == 0) {
                const float ta = (float)tot[0], tb = (float)((tot[1] - (double)lv * tot[0]) * (double)is);
                __hip_atomic_store(reinterpret_cast<unsigned long long*>(A.rows) + ((size_t)slab * A.U + u) * A.nch + ch,
                                   ((unsigned long long)slab_bits(tb) << 32) | slab_bits(ta), __ATOMIC_RELAXED,
                                   __HIP_MEMORY_SCOPE_AGENT);
            }
            mine = slab_hand_over(A, L, slab, u);
            if (mine) {
                double s0 = 0.0, s1 = 0.0;
                slab_gather(A, L, slab, [&](int, int, float ak, float bk) {
                    s0 += (double)ak;
                    s1 += (double)bk;
                });
                db = slab_channel_total(A, L, s0, 0);
                dg = slab_channel_total(A, L, s1, 1);
                ok = L.skip != 2;
            }
        }
        if (mine) {
            if (ch < A.nch && sub == 0) {
                float dbf = (float)db, dgf = (float)dg;
                if (!ok) dbf = dgf = __uint_as_float(0x7fc00000u);
                // dx = gsc * dy + k0 - k2 * (x - mu), see nchw_fused_backward.  SOLO, where a channel may have a handful of
                // values: gsc * (dy - c1) + (k0 - k2 * (x - mu)), so that what cancels is dy and its mean, as stored
                const float gs = gm * is, c1 = dbf * A.inv_M, c2 = dgf * A.inv_M, kk = gs * is * c2;
                L.k0[ch] = SOLO ? kk * lv : kk * lv - gs * c1;
                if (SOLO) L.k3[ch] = c1;
                L.k1[ch] = gs;
                L.k2[ch] = -kk;
                if ((SOLO || L.last) && ch < A.rch && c0 + ch < A.C) {
                    A.dbeta[c0 + ch] = dbf;
                    A.dgamma[c0 + ch] = dgf;
                }
            }
            __syncthreads();
            float nk2[VEC], gsc[VEC], k0[VEC], c1[SOLO ? VEC : 1];
            const SlabChannels<VEC> c3(A, (int)fresh((unsigned)col));
#pragma unroll
            for (int e = 0; e < VEC; ++e) {
                k0[e] = L.k0[c3[e]]; gsc[e] = L.k1[c3[e]]; nk2[e] = L.k2[c3[e]];
                if constexpr (SOLO) c1[e] = L.k3[c3[e]];
            }
            auto value = [&](const u32x4& vx, const u32x4& vg) __attribute__((always_inline)) {
                float fx[VEC], fg[VEC];
                slab_unpack<T>(vx, fx);
                slab_unpack<T>(vg, fg);
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    if constexpr (SOLO) fg[e] = gsc[e] * (fg[e] - c1[e]) + (nk2[e] * (fx[e] - mu[e]) + k0[e]);
                    else fg[e] = nk2[e] * (fx[e] - mu[e]) + (gsc[e] * fg[e] + k0[e]);
                }
                return slab_pack<T>(fg);
            };
            wait_vector_memory();
            char* ou = ob + g.base;
            char* zu = zb + g.base;      // (used if zb is not null)
            unroll_planes<P>([&](auto i_) __attribute__((always_inline)) {
                constexpr int i = decltype(i_)::value;
                if (i < ps.nr) {
                    slab_forget(xd[i]);
                    slab_forget(gd[i]);
                    slab_store(ou + ps.loff, value(xd[i], gd[i]), A.nt);
                    if (ACT != 0 && zb != nullptr) slab_store(zu + ps.loff, gd[i], A.nt);
                }
                ou += ps.step;
                if (ACT != 0) zu += ps.step;
            });
            if constexpr (!SOLO) {
                for (int k = L.fix ? slab_next_moved(A, slab, -1) : -1; k >= 0; k = slab_next_moved(A, slab, k)) {
                    const SlabGeom m = slab_geometry(A, slab, k);
                    for (int i = r; live && i < m.n; i += A.rpp) {
                        const long long o = m.base + (long long)i * A.row_bytes + (long long)col * 16;
                        u32x4 vx, vg, vy;
                        slab_load<false>(xb + o, vx);
                        slab_load<false>(gb + o, vg);
                        if constexpr (ACT != 0) {
                            slab_load<false>(ab + o, vy);
                            mask(vg, vy);
                        }
                        slab_store(ob + o, value(vx, vg), 0);
                        if (ACT != 0 && zb != nullptr) slab_store(zb + o, vg, 0);
                    }
                }
            }
        }
        if (!SOLO) __syncthreads();
    }
}

// X(vectors per thread (and tensor), one unit per slab)
#define CGBN_SLAB_FORWARD_P(X) X(4, true) X(8, true) X(12, true) X(20, true) X(6, false) X(12, false) X(20, false) X(28, false) X(36, false)
#define CGBN_SLAB_BACKWARD_P(X) X(4, true) X(8, true) X(12, true) X(20, true) X(6, false) X(10, false) X(14, false) X(18, false)

}  // namespace cgbn
