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
// U > 1: a unit publishes, per channel, s = sum(x - p) and q, the squared deviations from its own mean (backward: sum dy and
// sum dy * xhat) as two doubles (with a handful of units there are few roundings to average: as floats, two units of 6272 values
// each left the mean 1e-7 standard deviations off, now 3e-10), and counts itself in on the slab's counter; the unit that completes the count
// learns so from it; the units share out the slab's channels, add up their rows in double precision and in a fixed order
// and publish the results, which every unit then fetches.  Unlike in the NCHW single-launch kernels, no wait here needs its
// siblings to be resident: a unit whose wait runs out marks itself in the slab's bitmap (unless the count completed
// meanwhile) and its workgroup moves on; the unit that completes the count finds the marks in the value its own
// arrival returned and, once it has the statistics, reads the marked units' values again and writes their results.
// So every launch drains and is right whatever else the device runs; sharing it only costs the re-reads.
#pragma once

#include "cgbn_fused.h"

namespace cgbn {

constexpr int kSlabThreads = 512;
constexpr int kSlabWaves = kSlabThreads / kWave;
constexpr int kSlabRowsPerLane = 4;        // rows of a channel that one lane adds up: at most 4 x 64 units per slab
constexpr int kSlabMaxChannels = 128;      // channels of one slab
constexpr int kSlabMaxPixelCols = 16;      // vector columns of a slab whose channels are one column each
constexpr int kSlabPartWords = 8 * (kSlabThreads + 8 * kSlabMaxPixelCols + 8);
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
    unsigned long long* rows; // per slab: [channel][unit][2] doubles, then [channel][2] pairs of floats, the results
    unsigned* sync;
    long long R;          // rows of the matrix
    long long row_bytes;
    double inv_M_f64, eps;
    float inv_M;
    int vecs;             // 16-byte vectors per row
    int cols, ncols;      // vector columns of a slab, its element columns
    int rpp;              // rows per pass
    int rch;                  // channels per slab
    int cpc, nch, tpc;    // columns per channel, rch rounded up to a power of two, threads that add one channel's partial sums
    int C, slabs, U, rpu; // rpu: rows per unit
    int total_units;
    int G;                // lanes that add up one channel's rows
    int inflight;         // slabs whose units the grid holds at once
    long long pivot_stride;   // elements between the first values of consecutive channels
    int nt;
    unsigned spin_limit;
    unsigned stagger;     // start-up stagger: 100 MHz ticks per slab in flight
    int prefetch;         // several rounds: the wavefronts from this one on fetch the next unit's first passes into LDS during the hand-over
    int ahead;            // ... 2: all passes the LDS has room for; 1: the first kSlabAheadFew (backward)
    unsigned bitmap_words;    // per slab
    int neighbours;           // the slabs in flight together lie side by side
    unsigned cpc_magic;       // 2^32 / cpc, rounded up: i / cpc is the high word of i * cpc_magic for the small i here
};

// LDS of a workgroup
struct SlabLds {
    float part[2][kSlabPartWords];                       // see slab_sum
    float piv[kSlabMaxChannels];                         // forward: pivots
    float res[3][kSlabMaxChannels];                      // several units: the channels' results (forward mean, its rest, 1/sqrt; backward dbeta, dgamma)
    float k0[kSlabMaxChannels], k1[kSlabMaxChannels], k2[kSlabMaxChannels], k3[kSlabMaxChannels];   // write-out constants
    int skip, last, fix, wait;  // this unit moves on (2: results are missing for good); it completed the count; there are units for it to finish; the count is complete, the results are not there yet
};

// Sums over groups of `lanes` lanes (a power of two up to 64, uniform): f(off) adds the lanes that differ in one bit.
template <class F> __device__ __forceinline__ void lanes_add(int lanes, F f)
{
    asm volatile("" : "+s"(lanes));                   // (or the compiler keeps every comparison of every call in registers)
    if (lanes > 1) f(std::integral_constant<int, 1>{});
    if (lanes > 2) f(std::integral_constant<int, 2>{});
    if (lanes > 4) f(std::integral_constant<int, 4>{});
    if (lanes > 8) f(std::integral_constant<int, 8>{});
    if (lanes > 16) f(std::integral_constant<int, 16>{});
    if (lanes > 32) f(std::integral_constant<int, 32>{});
}

// Sums a thread's column values over the slab, in double precision: every thread leaves its values in LDS, and each channel's
// `tpc` threads add them up; the first of them (t % tpc == 0, channel t / tpc) gets the channel's sums.  One column a channel:
// the values of a column lie side by side, columns 8 words further on than they need be, so that neither the stores (lanes that
// differ in column and row) nor the loads (in channel and row) meet in a bank.  (Folding the row lanes of a wavefront first, in
// float, left the mean of 2100 x 2048 bf16 1.1e-7 standard deviations off, now 7e-10, and took longer:
// backward of 2100 x 512 9.6 us, now 8.9; forward 9.4, now 8.7.)
// `add(i, x, out)`: adds the Q values x that row lane i left for a column.
template <int VEC, int Q, class LDS, class F>
__device__ __forceinline__ void slab_sum(const SlabArgs& A, LDS& L, float (&v)[Q][VEC], int col, int r, double (&out)[2], F add)
{
    constexpr int qs = VEC * (kSlabPartWords / 8);        // words between a thread's quantities
    static_assert(Q * qs <= 2 * kSlabPartWords, "they fit");
    float* part = L.part[0];
    const int t = (int)fresh(threadIdx.x);
    const int rs = A.rpp + 8, es = A.cols * rs + 8;       // one column a channel: words between columns, between a thread's values
    if (r < A.rpp) {
        if (A.cpc == 1) {
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int e = 0; e < VEC; ++e) part[q * qs + e * es + col * rs + r] = v[q][e];
        } else {
#pragma unroll
            for (int q = 0; q < Q; ++q)
#pragma unroll
                for (int e = 0; e < VEC; ++e) part[q * qs + r * A.ncols + col * VEC + e] = v[q][e];
        }
    }
    __syncthreads();
    const int ch = t / A.tpc, sub = t & (A.tpc - 1);
    out[0] = out[1] = 0.0;
    auto take = [&](int i, int w) __attribute__((always_inline)) {
        float x[Q];
#pragma unroll
        for (int q = 0; q < Q; ++q) x[q] = part[q * qs + w];
        add(i, x, out);
    };
    if (ch * A.cpc < A.ncols) {                   // (channels beyond the slab's columns hold zeros)
        if (A.cpc == 1) {
            const int w0 = (ch % VEC) * es + (ch / VEC) * rs;
            for (int i = sub; i < A.rpp; i += A.tpc) take(i, w0 + i);
        } else {
            // the channel's cpc columns of every row lane, dealt to its threads
            for (int k = sub; k < A.rpp * A.cpc; k += A.tpc) {
                const int i = (int)__umulhi((unsigned)k, A.cpc_magic), j = k - i * A.cpc;
                take(i, i * A.ncols + ch * A.cpc + j);
            }
        }
    }
    lanes_add(A.tpc, [&](auto off) __attribute__((always_inline)) {
        out[0] = lane_add<decltype(off)::value>(out[0]);
        out[1] = lane_add<decltype(off)::value>(out[1]);
    });
}

__device__ __forceinline__ unsigned slab_bits(float v)      // NaN in canonical form: never the sentinel
{
    return v != v ? 0x7fc00000u : __float_as_uint(v);
}

// A slab's memory: [channel][unit][2] rows of doubles (a channel's lie side by side: they are fetched again and again until they are all
// there, and by lines that hold nothing else), then the channels' results (two pairs of floats each), all 8-byte words that
// hold the sentinel until they are written.
__device__ __forceinline__ unsigned long long* slab_rows(const SlabArgs& A, int slab)
{
    return A.rows + (size_t)slab * (A.U + 1) * A.nch * 2;
}
__device__ __forceinline__ void slab_put_row(const SlabArgs& A, int slab, int u, int c, double a, double b)
{
    unsigned long long* p = slab_rows(A, slab) + ((size_t)c * A.U + u) * 2;
    // (NaN in canonical form, as in slab_bits)
    __hip_atomic_store(p, a != a ? 0x7ff8000000000000ull : (unsigned long long)__double_as_longlong(a), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    __hip_atomic_store(p + 1, b != b ? 0x7ff8000000000000ull : (unsigned long long)__double_as_longlong(b), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void slab_put(unsigned long long* p, float lo, float hi)
{
    __hip_atomic_store(p, ((unsigned long long)slab_bits(hi) << 32) | slab_bits(lo), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ bool slab_missing(unsigned long long v)
{
    return (unsigned)v == kRowSentinel || (unsigned)(v >> 32) == kRowSentinel;
}

// Polls with `fetch` (false: something is missing) until a wavefront has everything, `polls` or the time runs out.
template <class F> __device__ __forceinline__ bool slab_poll(const SlabArgs& A, bool patient, F fetch)
{
    const unsigned long long t0 = wall_clock64();
    unsigned long long limit = patient ? kSlabBackstopTicks : kSlabWaitTicks;
    for (unsigned polls = 0; patient || polls < A.spin_limit; ++polls) {
        if (__ballot(!fetch()) == 0ull) return true;
        if ((polls & 31u) == 31u) {
            if (!patient && ld_agent(A.sync + kSlabMovedOn) != 0u) limit = kSlabWaitTicksLater;
            if (wall_clock64() - t0 > limit) return false;
        }
        __builtin_amdgcn_s_sleep(1);
    }
    return false;
}

// 1 / n to about 1e-14 (a Newton step from the hardware's float reciprocal); with two steps, to the last bit or two
template <int STEPS = 1> __device__ __forceinline__ double slab_reciprocal(double n)
{
    double r = (double)__builtin_amdgcn_rcpf((float)n);
#pragma unroll
    for (int i = 0; i < STEPS; ++i) r = r * (2.0 - n * r);
    return r;
}

// One channel's rows added up by the `G` lanes of a group (lane `gl`), double precision, fixed order; the group's first
// lane writes the results.  False: rows are missing.  (Lanes without a channel take part in the polls.)
template <bool FWD> __device__ __forceinline__ bool slab_reduce(const SlabArgs& A, SlabLds& L, int slab, int c, bool patient)
{
    const int gl = (int)fresh(threadIdx.x) & (A.G - 1);
    const bool duty = c < A.rch;
    const unsigned long long* row = slab_rows(A, slab) + ((size_t)(duty ? c : 0) * A.U + gl) * 2;
    unsigned long long v[kSlabRowsPerLane], w[kSlabRowsPerLane];
#pragma unroll
    for (int j = 0; j < kSlabRowsPerLane; ++j) v[j] = w[j] = duty && gl + j * A.G < A.U ? ~0ull : 0ull;       // (two words of kRowSentinel: not there yet)
    if (!slab_poll(A, patient, [&] {
            bool there = true;
#pragma unroll
            for (int j = 0; j < kSlabRowsPerLane; ++j) {
                if (v[j] == ~0ull || w[j] == ~0ull) {         // (what has come is not fetched again)
                    const unsigned long long* p = row + (size_t)(j * A.G) * 2;
                    v[j] = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    w[j] = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
#pragma unroll
            for (int j = 0; j < kSlabRowsPerLane; ++j) there &= v[j] != ~0ull && w[j] != ~0ull;
            return there;
        }))
        return false;
    double s0 = 0.0, s1 = 0.0;
#pragma unroll
    for (int j = 0; j < kSlabRowsPerLane; ++j) {
        s0 += __longlong_as_double((long long)v[j]);
        if (!FWD) s1 += __longlong_as_double((long long)w[j]);
    }
    lanes_add(A.G, [&](auto off) __attribute__((always_inline)) {
        s0 = lane_add<decltype(off)::value>(s0);
        if (!FWD) s1 = lane_add<decltype(off)::value>(s1);
    });
    unsigned long long* result = slab_rows(A, slab) + ((size_t)A.U * A.nch + (duty ? c : 0)) * 2;
    if (FWD) {
        // steps 6-8 about the pooled mean: every unit's squared deviations from its own mean and n times the distance between
        // the two means squared; nothing is subtracted from anything but means
        const double off = s0 * A.inv_M_f64, mean = (double)L.piv[duty ? c : 0] + off;
#pragma unroll
        for (int j = 0; j < kSlabRowsPerLane; ++j) {
            const int k = gl + j * A.G;
            if (k < A.U) {
                const double n = (double)(k + 1 < A.U ? A.rpu : (int)(A.R - (long long)k * A.rpu)) * (double)A.cpc;
                const double d = __longlong_as_double((long long)v[j]) * slab_reciprocal(n) - off;
                s1 += __longlong_as_double((long long)w[j]) + n * (d * d);
            }
        }
        lanes_add(A.G, [&](auto off) __attribute__((always_inline)) { s1 = lane_add<decltype(off)::value>(s1); });
        if (duty && gl == 0) {
            const float hi = (float)mean;
            slab_put(result, hi, (float)(mean - (double)hi));
            slab_put(result + 1, (float)rsqrt_f64(s1 * A.inv_M_f64 + A.eps), 0.f);
        }
    } else if (duty && gl == 0) {
        slab_put(result, (float)s0, (float)s1);
    }
    return true;
}

// The slab's results into L.res (one wavefront).  False: some are missing.
template <bool FWD> __device__ __forceinline__ bool slab_results(const SlabArgs& A, SlabLds& L, int slab, bool patient)
{
    const unsigned long long* result = slab_rows(A, slab) + (size_t)A.U * A.nch * 2;
    return slab_poll(A, patient, [&] {
        bool there = true;
        for (int c = (int)fresh(threadIdx.x) & (kWave - 1); c < A.rch; c += kWave) {
            const unsigned long long v = __hip_atomic_load(result + 2 * c, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const unsigned long long w = FWD ? __hip_atomic_load(result + 2 * c + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) : 0ull;
            there &= !slab_missing(v) && !slab_missing(w);
            L.res[0][c] = __uint_as_float((unsigned)v);
            L.res[1][c] = __uint_as_float((unsigned)(v >> 32));
            if (FWD) L.res[2][c] = __uint_as_float((unsigned)w);
        }
        return there;
    });
}

// After a unit's rows are on their way: counts it in, adds up the channels that are this unit's to add up (u, u + U, ...)
// and waits for the others'.  Every row crosses the chip once and every unit fetches one result per channel; were each unit
// to add up all rows itself, that would be U times as much (7680 pairs of a slab of 268800 x 64 bf16: 4 us a unit).
// Returns false if the unit moves on (its bitmap bit is set).  L.fix: units that moved on before this one completed the
// count; the channels they owe are added up here too.
// `meanwhile()`: run by the wavefronts that fetch ahead once the rows are out.
template <bool FWD, class F> __device__ __forceinline__ bool slab_hand_over(const SlabArgs& A, SlabLds& L, int slab, int u, F meanwhile)
{
    const int t = (int)fresh(threadIdx.x);          // (what is formed from it stays here: see fresh)
    unsigned* cnt = A.sync + kSyncHeader + slab;
    unsigned* bitmap = A.sync + kSyncHeader + A.C + (size_t)slab * A.bitmap_words;
    __syncthreads();                  // every wavefront has issued its row stores
    unsigned old;                     // (of the first thread; given a value for the others it would be waited for here)
    if (t == 0) old = __hip_atomic_fetch_add(cnt, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_amdgcn_readfirstlane(t) >= A.prefetch * kWave) meanwhile();
    const int mine = u + t / A.G * A.U;
    // (whole wavefronts: the first group of each has the lowest channel)
    const bool any = __builtin_amdgcn_readfirstlane(mine) < A.rch;
    const bool done = !any || slab_reduce<FWD>(A, L, slab, mine, false);
    if (t < kWave) {
        const bool up = slab_results<FWD>(A, L, slab, false);
        if (t == 0) {
            L.skip = L.last = L.fix = L.wait = 0;
            if ((old & 0xffffu) == (unsigned)(A.U - 1)) {
                L.last = 1;
                L.wait = !up;
                const int moved = (int)(old >> 16);
                if (moved > 0) {
                    // (their workgroups are about to set their bits: they have seen the count)
                    const unsigned long long t0 = wall_clock64();
                    for (;;) {
                        int have = 0;
                        for (unsigned i = 0; i < A.bitmap_words; ++i) have += __popc(ld_agent(bitmap + i));
                        if (have >= moved) { L.fix = 1; break; }
                        if (wall_clock64() - t0 > kSlabBackstopTicks) {
                            atomicExch(A.sync + 1, 1u);
                            L.skip = 2;               // (the marked units' values stay unwritten: the statistics say so)
                            break;
                        }
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
                } else {
                    L.wait = 1;
                }
            }
        }
    }
    __syncthreads();
    if (L.fix | L.wait) {
        // Every unit has counted itself in, so every row has been issued.  The backstop, if it is ever hit, makes the
        // caller poison the statistics.
        bool sound = true;
        if (L.fix) {
            for (int c = t / A.G; __builtin_amdgcn_readfirstlane(c) < A.rch; c += kSlabThreads / A.G) sound &= slab_reduce<FWD>(A, L, slab, c, true);
        } else if (!done) {
            sound = slab_reduce<FWD>(A, L, slab, mine, true);
        }
        if (t < kWave) sound &= slab_results<FWD>(A, L, slab, true);
        if (!sound) {
            atomicExch(A.sync + 1, 1u);
            L.skip = 2;
        }
        __syncthreads();
    }
    return L.skip != 1;
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
__device__ __forceinline__ SlabGeom slab_geometry(const SlabArgs& A, int slab, int u, int vb = 16)
{
    SlabGeom g;
    const long long row0 = (long long)u * A.rpu, left = A.R - row0;
    g.n = (int)(left < A.rpu ? left : A.rpu);
    g.base = row0 * A.row_bytes + (long long)slab * A.cols * vb;
    return g;
}

// SOLO: consecutive slabs share lines and go to one XCD (workgroups are dealt to the 8 XCDs in turn; measured, slabs of
// 64 bytes x 2100 rows, 8 MB copied through registers: 8.3 us in plain order, 5.8 so).  Bijective for any grid size.
__device__ __forceinline__ int slab_of_block(int b, int G)
{
    const int q = G >> 3, rem = G & 7, xcd = b & 7, i = b >> 3;
    return xcd * q + min(xcd, rem) + i;
}

template <class V> __device__ __forceinline__ void slab_forget(V& v) { asm volatile("" : "+v"(v)); }    // (see forget)

// VB: bytes of a thread's vectors.  8: one workgroup a slab, NCHW with small planes.  A slab starts and ends on whole vectors, so half the
// vector is half the channels: twice the workgroups where 16 bytes give at most half the compute units one (what bounds those
// calls is what one compute unit gets, 50 GB/s of what misses its L1, and its share of the sums), and a workgroup for every slab that would
// else be two units with their hand-over and a launch that prepares it.  Measured, 16 -> 8 bytes, forward / backward us: bf16
// 16 x 256 planes of 13x21 (32 workgroups, 64) 11.7 / 12.1 -> 7.9 / 8.3; 256 x 1024 of 7x7 (two units each of 128 slabs, 256 slabs) 21.6 / 24.3 ->
// 15.5 / 18.2; fp32 113 x 120 of 7x9 8.8 / 8.5 -> 7.0 / 7.3.
template <int VB> struct SlabVector;
template <> struct SlabVector<16> { typedef u32x4 V; };
template <> struct SlabVector<8> { typedef u32x2 V; };

// Several units: the order in which the slabs are taken.  Those in flight together are spread evenly over the row, and a
// round moves on by one slab: neighbouring columns at a long row stride would crowd the memory channels (measured,
// the loads and stores alone, 67200 rows of 4096 bytes: eight neighbouring slabs in flight 154 us, eight spread 114; rows
// of 1024 bytes 115 either way).  Slabs that share lines lie side by side instead, for their lines.  Bijective for any number of slabs.
__device__ __forceinline__ int slab_of_turn(const SlabArgs& A, int turn)
{
    if (A.neighbours) return turn;
    const int q = A.slabs / A.inflight, rem = A.slabs - q * A.inflight;
    const int k = turn / A.inflight, j = turn - k * A.inflight;
    return j * q + min(j, rem) + k;
}

template <bool NT, class V> __device__ __forceinline__ void slab_load(const char* p, V& d)
{
    d = NT ? __builtin_nontemporal_load(reinterpret_cast<const V*>(p)) : *reinterpret_cast<const V*>(p);
}
template <class V> __device__ __forceinline__ void slab_store(char* p, const V& d, int nt)
{
    if (nt) __builtin_nontemporal_store(d, reinterpret_cast<V*>(p));
    else *reinterpret_cast<V*>(p) = d;
}
template <typename T, class V> __device__ __forceinline__ void slab_unpack(const V& d, float (&f)[sizeof(V) / sizeof(T)])
{
    constexpr int EPW = Packed<T>::EPW;
#pragma unroll
    for (int q = 0; q < (int)sizeof(V) / 4; ++q) {
        float g[EPW];
        Packed<T>::unpack(d[q], g);
#pragma unroll
        for (int e = 0; e < EPW; ++e) f[q * EPW + e] = g[e];
    }
}
template <typename T, class V> __device__ __forceinline__ V slab_pack(const float (&f)[sizeof(V) / sizeof(T)])
{
    constexpr int EPW = Packed<T>::EPW;
    V d;
#pragma unroll
    for (int q = 0; q < (int)sizeof(V) / 4; ++q) {
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
__device__ __forceinline__ SlabPass slab_pass(const SlabArgs& A, int n, bool live, int r, int col, int vb = 16)
{
    SlabPass p;
    p.loff = fresh(live ? (unsigned)r * (unsigned)A.row_bytes + (unsigned)(col * vb) : 0u);
    p.nr = live ? (n - r + A.rpp - 1) / A.rpp : 0;
    p.passes = (n + A.rpp - 1) / A.rpp;
    p.step = (long long)A.rpp * A.row_bytes;
    return p;
}

// Start-up stagger: where few slabs are in flight and there are several rounds, slab j of the first round starts j steps
// later, so that some slabs read while others wait or write.  Measured, without -> with, us: two in flight (6 us a step),
// backward of 134400 x 512 bf16 119 -> 106, forward of 268800 x 512 bf16 147 -> 140, fp32 276 -> 271; four (2.5 us),
// backward of 67200 x 1024 fp32 204 -> 193, of 67200 x 2048 bf16 224 -> 210, forward of 134400 x 512 bf16 73.5 -> 69.6.  With
// more in flight they drift apart by themselves (eight, forward of 67200 x 1024 fp32: 129 -> 142 at 2.5 us).
__device__ __forceinline__ void slab_stagger(const SlabArgs& A)
{
    const unsigned long long wait = (unsigned long long)A.stagger * (blockIdx.x / A.U), t0 = wall_clock64();
    while (wall_clock64() - t0 < wait) __builtin_amdgcn_s_sleep(4);
}

// Prefetch (several rounds of units).  While the statistics complete, no load or store of the launch is in flight; the
// register file has no room for the next unit, the LDS has room for 2/5 of it.  Every wavefront but those that poll (their
// polls would queue behind their loads; always the first) fetches its part of the next unit's first passes straight into LDS.
// Measured, without -> with, us: fp32 67200 x 1024 forward 141 -> 129, backward 224 -> 204, fp32 268800 x 512 304 -> 276 and
// 454 -> 440, bf16 268800 x 512 151 -> 146 and 247 -> 239.
// With one slab in flight everyone is in the hand-over at the same time, and what a compute unit fetches stands before its polls, which
// its L1 answers in order: there the backward fetches two passes of the eight (backward, eight -> two: 268800 x 512 bf16 233 -> 222 us, with a
// mask 287 -> 280, fp32 430 -> 416; with two or more in flight the eight are better, fp32 67200 x 1024 194, two 204).
constexpr int kSlabAhead = kSlabWaves - 1;         // wavefronts that fetch ahead
constexpr int kSlabAheadFew = 2;
struct SlabAhead {
    SlabPass ps;
    const char* base[2];
    __device__ __forceinline__ SlabAhead(const SlabArgs& A, int unit, const char* b0, const char* b1)
    {
        const int t = (int)fresh(threadIdx.x), col = t % A.cols, r = t / A.cols;
        const int turn = unit / A.U, slab = slab_of_turn(A, turn);
        const SlabGeom g = slab_geometry(A, slab, unit - turn * A.U);
        ps = slab_pass(A, g.n, r < A.rpp && slab * A.cols + col < A.vecs, r, col);
        base[0] = b0 + g.base;
        base[1] = b1 + g.base;
    }
    // the first N passes, into slots for PRE
    template <int PRE, int TENSORS, int N = PRE> __device__ __forceinline__ void fetch(u32x4* ext)
    {
        const int w = __builtin_amdgcn_readfirstlane((int)(fresh(threadIdx.x) >> 6)) - 1;
#pragma unroll
        for (int i = 0; i < N; ++i)
#pragma unroll
            for (int q = 0; q < TENSORS; ++q) {
                __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)(base[q] + ps.lane(i)),
                                                 (void __attribute__((address_space(3)))*)(ext + ((q * PRE + i) * kSlabAhead + w) * kWave), 16, 0, 0);
                base[q] += ps.advance(i);
            }
    }
};
__device__ __forceinline__ const u32x4& slab_fetched(const u32x4* ext, int slot, int t) { return ext[slot * kSlabAhead * kWave + t - kWave]; }

// ---------------------------------------------------------------------------
// forward
// ---------------------------------------------------------------------------
// P: vectors per thread.  ACT as in the NCHW kernels; the shortcut (ACT == 2) is fetched with x where the
// registers allow (P <= 20), else while the unit is written out.
//
// Statistics.  One pass, under the loads: per column of a thread the sum S of x - f about the thread's first value f, and the
// squared deviations from the thread's own mean, one value at a time (the weights are constants of the unrolled loop):
//     M2 <- M2 + (x - f - S / i)^2 * i / (i + 1),      S <- S + (x - f).
// The unit's mean follows from the sums S + n (f - p) about the channel's pivot p, its first stored value; its squared
// deviations are the sum of M2 + n ((f - p) + S / n - mean)^2 over the threads.  Nothing is a difference
// of large float sums, so it does not matter where the pivot lies.  (A sum of (x - p)^2 with the difference taken off at the
// end loses (mean - p)^2 / variance times the accuracy of a float sum: relative error of 1/sqrt, the worst of many
// channels, pivot 4 standard deviations off 8.8e-7, here 6.1e-8; a few activations among zeros, the
// first of them the pivot, 6.3e-6 and 7.8e-8.)
//
// Launch bounds.  The plan counts one workgroup per compute unit where there are several units, which leaves a wavefront
// 256 registers; only variants that need no more than 128 anyway are held to them.  (P = 18 held to 128 kept 20 to 60
// bytes a lane in memory: forward of 256 x 1024 planes of 7x7 bf16 24.3 us, not held 21.7; of 67200 x 256 channels-last 26.8 and 24.6;
// backward, P = 9, of 26980 x 296 26.8 and 24.5.)  DENSE: held all the same, two workgroups per compute unit, where there are
// more units than compute units: forward of 164 x 800 planes of 11x16 bf16, 500 units, 36.4 us, so 30.7; backward of 149 x 696 of 10x12, 435
// units, 30.3 and 26.1.
template <typename T, int ACT, int P, bool SOLO, bool DENSE, int VB = 16>
__global__ __launch_bounds__(kSlabThreads, DENSE || P * VB / 16 * (ACT == 2 ? 2 : 1) <= (SOLO ? 4 : 12) ? 4 : 2) void slab_forward(SlabArgs A)
{
    static_assert(VB == 16 || SOLO, "8-byte vectors: one workgroup a slab");
    typedef typename SlabVector<VB>::V V;
    constexpr int VEC = VB / (int)sizeof(T);
    constexpr bool EARLY = ACT == 2 && P * VB / 16 <= 20;
    constexpr int PRE = !SOLO && P >= 28 ? 16 : 0;
    __shared__ SlabLds L;
    __shared__ u32x4 ext[PRE ? PRE * kSlabAhead * kWave : 1];
    int fetched = 0;                  // (uniform over a wavefront)
    const char* xb = static_cast<const char*>(A.x);
    const char* rb = static_cast<const char*>(A.dy);
    char* yb = static_cast<char*>(A.out);
    if (SOLO && blockIdx.x == 0 && threadIdx.x == 0) A.sync[1] = 0u;
    if (!SOLO) slab_stagger(A);

    for (int unit = SOLO ? slab_of_block(blockIdx.x, gridDim.x) : (int)blockIdx.x; unit < A.total_units; unit += gridDim.x) {
        // (formed anew for every unit: carried round the loop, what depends on them would cost registers)
        const int t = (int)fresh(threadIdx.x);
        const int col = t % A.cols, r = t / A.cols;
        const int ch = t / A.tpc, sub = t & (A.tpc - 1);  // the channel this thread helps to add up
        const int turn = SOLO ? unit : unit / A.U, u = SOLO ? 0 : unit - turn * A.U;
        const int slab = SOLO ? unit : slab_of_turn(A, turn);
        const int c0 = slab * A.rch;
        const bool live = r < A.rpp && slab * A.cols + col < A.vecs;
        const SlabGeom g = slab_geometry(A, slab, u, VB);
        const SlabPass ps = slab_pass(A, g.n, live, r, col, VB);
        V d[P], s[EARLY ? P : 1];
        // ---- pivots, then the unit's vectors
        const SlabChannels<VEC> cl(A, col);
        float piv[VEC];
        if (A.cpc == 1) {
            V pw;
            slab_load<false>(xb + (long long)slab * A.cols * VB + (live ? (unsigned)(col * VB) : 0u), pw);
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
            if (PRE != 0 && __builtin_amdgcn_readfirstlane(fetched) != 0) {
                unroll_planes<PRE>([&](auto i_) __attribute__((always_inline)) {
                    constexpr int i = decltype(i_)::value;
                    if constexpr (VB == 16) d[i] = slab_fetched(ext, i, t);
                    xu += ps.advance(i);
                });
            } else {
                unroll_planes<PRE>([&](auto i_) __attribute__((always_inline)) {
                    constexpr int i = decltype(i_)::value;
                    slab_load<!SOLO>(xu + ps.lane(i), d[i]);
                    xu += ps.advance(i);
                });
            }
            unroll_planes<P - PRE>([&](auto i_) __attribute__((always_inline)) {
                constexpr int i = PRE + decltype(i_)::value;
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
        // ---- the thread's sums and squared deviations
        float first[VEC], a[VEC], m2[VEC];
        slab_unpack<T>(d[0], first);
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if (ps.nr == 0) first[e] = piv[e];            // (what was loaded is no value of this channel)
            a[e] = m2[e] = 0.f;
        }
        unroll_planes<P - 1>([&](auto i_) __attribute__((always_inline)) {
            constexpr int i = decltype(i_)::value + 1;
            if (i < ps.nr) {
                float f[VEC];
                slab_unpack<T>(d[i], f);
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    const float dv = f[e] - first[e];
                    const float dd = dv - a[e] * (1.0f / (float)i);
                    m2[e] += dd * (dd * ((float)i / (float)(i + 1)));
                    a[e] += dv;
                }
            }
        });
        // ---- the unit's, in one go: what the means of the threads add to the squared deviations, sum n_t (m_t - m)^2, is taken as
        // sum S_t^2 / n_t - S^2 / n, in double precision and from the very S_t = n_t (f - p) + sum (x - f) that S is the sum of, so that the
        // difference is exact to 1e-16 (m / sigma)^2.  S_t as one float would not be exact where f - p is no bfloat16 (mostly zeros, the
        // pivot not among them: 1/sqrt to 1.5e-7, so 4.7e-8): float keeps its two terms apart.
        // Summing twice, the second time about the unit's mean, forward us then / now: bf16 2100 x 512 8.7 / 8.2, 2100 x 2048 10.8 / 10.0,
        // 16 x 256 planes of 13x21 8.4 / 7.8, 256 x 1024 of 7x7 16.5 / 15.5, in units 50960 x 72 18.3 / 17.1; mean + mean_lo 2e-6 / 1.2e-6 at worst.
        constexpr bool APART = std::is_same<T, float>::value;
        constexpr int Q = APART ? 3 : 2;
        float b[Q][VEC];
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            const float off = first[e] - piv[e];
            b[0][e] = APART ? a[e] : a[e] + (float)ps.nr * off;
            b[1][e] = m2[e];
            if constexpr (APART) b[2][e] = off;
        }
        double tot[2];
        {
            const int whole = g.n - (ps.passes - 1) * A.rpp;      // row lanes with a value in every pass; the others have one less
            const double n0 = (double)ps.passes, n1 = n0 - 1.0, inv0 = slab_reciprocal<2>(n0), inv1 = ps.passes > 1 ? slab_reciprocal<2>(n1) : 0.0;
            slab_sum<VEC, Q>(A, L, b, col, r, tot, [&](int i, const float (&x)[Q], double (&o)[2]) __attribute__((always_inline)) {
                double s = (double)x[0];
                if constexpr (APART) s += (i < whole ? n0 : n1) * (double)x[Q - 1];
                o[0] += s;
                o[1] += (double)x[1] + s * s * (i < whole ? inv0 : inv1);
            });
        }
        tot[1] -= tot[0] * tot[0] * slab_reciprocal<2>((double)g.n * (double)A.cpc);
        if (tot[1] < 0.0) tot[1] = 0.0;                           // (a NaN stays)
        if (!SOLO && ch < A.nch && sub == 0) L.piv[ch] = pv;
        // ---- steps 4-5 and 9-10
        bool ok = true, mine = true;
        if (!SOLO) {
            if (ch < A.nch && sub == 0) slab_put_row(A, slab, u, ch, tot[0], tot[1]);
            fetched = 0;
            mine = slab_hand_over<true>(A, L, slab, u, [&] {
                if constexpr (PRE != 0)
                    if (A.prefetch != 0 && unit + (int)gridDim.x < A.total_units) {
                        SlabAhead(A, unit + (int)gridDim.x, xb, xb).template fetch<PRE, 1>(ext);
                        fetched = 1;
                    }
            });
            ok = L.skip != 2;
        }
        if (mine) {
            if (ch < A.nch && sub == 0) {
                float hi, lo, is;
                if (SOLO) {
                    const double mean = (double)pv + tot[0] * A.inv_M_f64;
                    hi = (float)mean;
                    lo = (float)(mean - (double)hi);
                    is = (float)rsqrt_f64(tot[1] * A.inv_M_f64 + A.eps);
                } else {
                    hi = L.res[0][ch];
                    lo = L.res[1][ch];
                    is = L.res[2][ch];
                }
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
            auto value = [&](const V& v, const V& w) __attribute__((always_inline)) {
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
                return slab_pack<T, V>(f);
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
                        V b[B];
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
                        V v, w = {};
                        slab_load<false>(xb + o, v);
                        if constexpr (ACT == 2) slab_load<false>(rb + o, w);
                        slab_store(yb + o, value(v, w), 0);
                    }
                }
            }
        }
        if (!SOLO) {
            if (PRE != 0 && !mine) wait_vector_memory();      // what was fetched ahead has landed (else before the write-out)
            __syncthreads();              // the hand-over's verdicts have been read by everyone
        }
    }
}

// ---------------------------------------------------------------------------
// backward
// ---------------------------------------------------------------------------
// P: vectors per thread and tensor.  ACT != 0: dy is first masked by the stored output (A.aux) being positive; the
// output's vectors are loaded beside the other two where the registers allow (P <= 10), else through the storage x takes
// afterwards.
template <typename T, int ACT, int P, bool SOLO, bool DENSE, int VB = 16>
__global__ __launch_bounds__(kSlabThreads, DENSE || P * VB / 16 * (ACT != 0 ? 3 : 2) <= (SOLO ? 8 : 12) ? 4 : 2) void slab_backward(SlabArgs A)
{
    static_assert(VB == 16 || SOLO, "8-byte vectors: one workgroup a slab");
    typedef typename SlabVector<VB>::V V;
    constexpr int VEC = VB / (int)sizeof(T);
    constexpr bool THREE = ACT != 0 && P * VB / 16 <= (SOLO ? 10 : 6);
    constexpr int PRE = !SOLO && P >= 14 ? 8 : 0;
    __shared__ SlabLds L;
    __shared__ u32x4 ext[PRE ? 2 * PRE * kSlabAhead * kWave : 1];
    int fetched = 0;                  // (uniform over a wavefront)
    const char* xb = static_cast<const char*>(A.x);
    const char* gb = static_cast<const char*>(A.dy);
    const char* ab = static_cast<const char*>(A.aux);
    char* ob = static_cast<char*>(A.out);
    char* zb = static_cast<char*>(A.out2);
    if (SOLO && blockIdx.x == 0 && threadIdx.x == 0) A.sync[1] = 0u;
    if (!SOLO) slab_stagger(A);

    for (int unit = SOLO ? slab_of_block(blockIdx.x, gridDim.x) : (int)blockIdx.x; unit < A.total_units; unit += gridDim.x) {
        // (formed anew for every unit: carried round the loop, what depends on them would cost registers)
        const int t = (int)fresh(threadIdx.x);
        const int col = t % A.cols, r = t / A.cols;
        const int ch = t / A.tpc, sub = t & (A.tpc - 1);  // the channel this thread helps to add up
        const int turn = SOLO ? unit : unit / A.U, u = SOLO ? 0 : unit - turn * A.U;
        const int slab = SOLO ? unit : slab_of_turn(A, turn);
        const int c0 = slab * A.rch;
        const bool live = r < A.rpp && slab * A.cols + col < A.vecs;
        const SlabGeom g = slab_geometry(A, slab, u, VB);
        const SlabPass ps = slab_pass(A, g.n, live, r, col, VB);
        V xd[P], gd[P], yd[THREE ? P : 1];
        auto mask = [&](V& v, const V& y) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < VB / 4; ++q) v[q] = mask_by_positive<T>(v[q], y[q]);
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
            auto load = [&](auto i_, V& dg, V& dx) __attribute__((always_inline)) {
                constexpr int i = decltype(i_)::value;
                slab_load<!SOLO>(gu + ps.lane(i), dg);
                gu += ps.advance(i);
                if constexpr (ACT == 0 || THREE) {
                    slab_load<!SOLO>(xu + ps.lane(i), dx);
                    xu += ps.advance(i);
                }
                if constexpr (ACT != 0) {
                    if constexpr (THREE) slab_load<!SOLO>(yu + ps.lane(i), yd[i]);
                    else slab_load<!SOLO>(yu + ps.lane(i), dx);
                    yu += ps.advance(i);
                }
            };
            // passes [FROM, FROM + N) from the LDS or from memory
            auto first = [&](auto from_, auto n_, bool in_lds) __attribute__((always_inline)) {
                constexpr int from = decltype(from_)::value;
                if (in_lds) {
                    unroll_planes<decltype(n_)::value>([&](auto i_) __attribute__((always_inline)) {
                        constexpr int i = from + decltype(i_)::value;
                        if constexpr (VB == 16) {
                            gd[i] = slab_fetched(ext, i, t);
                            xd[i] = slab_fetched(ext, PRE + i, t);
                        }
                        gu += ps.advance(i);
                        if constexpr (ACT == 0) xu += ps.advance(i);
                        else yu += ps.advance(i);
                    });
                } else {
                    unroll_planes<decltype(n_)::value>([&](auto i_) __attribute__((always_inline)) {
                        constexpr int i = from + decltype(i_)::value;
                        load(IntC<i>{}, gd[i], xd[i]);
                    });
                }
            };
            if constexpr (PRE != 0) {
                first(IntC<0>{}, IntC<kSlabAheadFew>{}, __builtin_amdgcn_readfirstlane(fetched) != 0);
                first(IntC<kSlabAheadFew>{}, IntC<PRE - kSlabAheadFew>{}, __builtin_amdgcn_readfirstlane(fetched) == 2);
            }
            unroll_planes<P - PRE>([&](auto i_) __attribute__((always_inline)) {
                constexpr int i = PRE + decltype(i_)::value;
                load(std::integral_constant<int, i>{}, gd[i], xd[i]);
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
        slab_sum<VEC, 2>(A, L, a, col, r, tot, [](int, const float (&x)[2], double (&o)[2]) __attribute__((always_inline)) {
            o[0] += (double)x[0];
            o[1] += (double)x[1];
        });
        double db = 0.0, dg = 0.0;
        bool ok = true, mine = true;
        if (SOLO) {
            db = tot[0];
            dg = (tot[1] - (double)lv * tot[0]) * (double)is;
        } else {
            if (ch < A.nch && sub == 0) slab_put_row(A, slab, u, ch, tot[0], (tot[1] - (double)lv * tot[0]) * (double)is);
            fetched = 0;
            mine = slab_hand_over<false>(A, L, slab, u, [&] {
                if constexpr (PRE != 0)
                    if (A.prefetch != 0 && unit + (int)gridDim.x < A.total_units) {
                        SlabAhead next(A, unit + (int)gridDim.x, gb, ACT == 0 ? xb : ab);
                        if (A.ahead == 2) next.template fetch<PRE, 2>(ext);
                        else next.template fetch<PRE, 2, kSlabAheadFew>(ext);
                        fetched = A.ahead;
                    }
            });
            ok = L.skip != 2;
        }
        if (mine) {
            if (ch < A.nch && sub == 0) {
                float dbf = SOLO ? (float)db : L.res[0][ch], dgf = SOLO ? (float)dg : L.res[1][ch];
                if (!ok) dbf = dgf = __uint_as_float(0x7fc00000u);
                // dx = gsc * dy + k0 - k2 * (x - mu), see nchw_fused_backward.  SOLO, where a channel may have a handful of
                // values: gsc * (dy - c1) + (k0 - k2 * (x - mu)), so that what cancels is dy and its mean, as stored.  k0 is
                // rounded once: where dy has a mean that is large beside its spread, that rounding is dx's error.
                const float gs = gm * is, kk = gs * is * (dgf * A.inv_M);
                const double c1 = (SOLO ? db : (double)dbf) * A.inv_M_f64;
                L.k0[ch] = (float)((double)kk * (double)lv - (double)gs * (SOLO ? c1 - (double)(float)c1 : c1));
                if (SOLO) L.k3[ch] = (float)c1;
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
            auto value = [&](const V& vx, const V& vg) __attribute__((always_inline)) {
                float fx[VEC], fg[VEC];
                slab_unpack<T>(vx, fx);
                slab_unpack<T>(vg, fg);
#pragma unroll
                for (int e = 0; e < VEC; ++e) {
                    if constexpr (SOLO) fg[e] = gsc[e] * (fg[e] - c1[e]) + (nk2[e] * (fx[e] - mu[e]) + k0[e]);
                    else fg[e] = nk2[e] * (fx[e] - mu[e]) + (gsc[e] * fg[e] + k0[e]);
                }
                return slab_pack<T, V>(fg);
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
                        V vx, vg, vy;
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
        if (!SOLO) {
            if (PRE != 0 && !mine) wait_vector_memory();
            __syncthreads();
        }
    }
}

// X(vectors per thread (and tensor), one unit per slab)
#define CGBN_SLAB_FORWARD_P(X) X(4, true) X(8, true) X(10, true) X(12, true) X(20, true) X(6, false) X(12, false) X(18, false) X(28, false) X(36, false)
#define CGBN_SLAB_BACKWARD_P(X) X(4, true) X(6, true) X(8, true) X(10, true) X(12, true) X(20, true) X(6, false) X(9, false) X(14, false) X(18, false)
// vectors per thread (and tensor) of the variants with 8-byte vectors
#define CGBN_SLAB_NARROW_P(X) X(8) X(12) X(16) X(20) X(28)
// the variants built DENSE too (the forward without a shortcut)
constexpr int kSlabDenseForward = 18, kSlabDenseBackward = 9;

}  // namespace cgbn
