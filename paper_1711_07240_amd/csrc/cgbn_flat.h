// Flat kernels (NCHW): a channel's values as one run of vectors, whatever planes they lie in, dealt evenly to the lanes of one wavefront or of a
// workgroup, and kept in registers between the statistics and the write-out.  One launch, nothing handed over, no prepared workspace.
//
// Bound by the launch and one pass over memory (1 read and 1 write of a tensor forward): small calls take 3.3 ... 4 us, of which about 2.5 are the launch;
// large ones run at 4.5 ... 5.5 TB/s.  The single-launch kernels of cgbn_fused.h move a plane per wavefront at a time and leave a row per plane; where a
// channel is a few short planes most of their lanes idle, and rows, shards and barriers cost more than the data.  Here a channel costs one sum over
// its lanes (two in the forward).  Before / now in us, forward and backward: 4 images of 16 channels of 32x32 fp32 5.6 / 3.7 and 4.8 / 3.8; 2 of 1848 of
// 27x40 bf16 14.6 / 5.9 and 12.9 / 7.5; 2 of 12000 of 24x24 fp32 forward 59.8 / 18.0; 16 of 1720 of 14x22 bf16 22.5 / 9.8 and 18.4 / 11.0.
//
// With one or four wavefronts a channel, 64 registers a lane are the most that leaves the masked backward its three tensors; sixteen have 32.  Vectors are the widest that a plane's bytes allow, so
// that every plane of a channel starts on one; which plane a vector lies in is a quotient by the plane's vectors, formed as a product's high half.
#pragma once

#include "cgbn_slab.h"

namespace cgbn {

struct FlatArgs {
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
    unsigned* sync;       // [1] error word
    double inv_M_f64, eps;
    float inv_M;
    int C;
    int vecs, total;      // vectors of a plane, of a channel
    unsigned magic;       // 2^32 / vecs, rounded up (0: one vector a plane)
    unsigned plane_bytes, image_bytes;
};

// registers of a lane's vectors of one tensor
constexpr int flat_words(int LB, int S) { return S * (LB < 4 ? 4 : LB) / 4; }

// threads of a workgroup: four channels of one wavefront each, or one channel of all its wavefronts
constexpr int flat_threads(int waves) { return waves == 1 ? kThreads : waves * kWave; }

// LB bytes as they are stored (2: one bfloat16, in the low half)
template <int LB> struct FlatVector { typedef uint32_t V __attribute__((ext_vector_type(LB / 4))); };
template <> struct FlatVector<4> { typedef uint32_t V; };
template <> struct FlatVector<2> { typedef uint32_t V; };

template <typename T, int LB, int S> struct FlatUnit {
    static constexpr int E = LB / (int)sizeof(T);            // values of a vector
    typedef typename FlatVector<LB>::V V;
    V v[S];
    static __device__ __forceinline__ V load(const char* p)
    {
        if constexpr (LB == 2) return *reinterpret_cast<const uint16_t*>(p);
        else return *reinterpret_cast<const V*>(p);
    }
    static __device__ __forceinline__ void store(char* p, const V& d)
    {
        if constexpr (LB == 2) *reinterpret_cast<uint16_t*>(p) = (uint16_t)d;
        else *reinterpret_cast<V*>(p) = d;
    }
    // (between passes: or the compiler keeps the values that one pass unpacked for the next, see forget)
    __device__ __forceinline__ void forget_all()
    {
#pragma unroll
        for (int i = 0; i < S; ++i) slab_forget(v[i]);
    }
    static __device__ __forceinline__ void unpack(const V& d, float (&f)[E])
    {
        if constexpr (LB == 2) f[0] = __uint_as_float(d << 16);
        else if constexpr (LB == 4) Packed<T>::unpack(d, f);
        else slab_unpack<T>(d, f);
    }
    static __device__ __forceinline__ V pack(const float (&f)[E])
    {
        if constexpr (LB == 2) return f32_to_bf16(f[0]);
        else if constexpr (LB == 4) return Packed<T>::pack(f);
        else return slab_pack<T, V>(f);
    }
};

// where a lane's vectors lie: its i-th is vector first + i * step of the channel
struct FlatLane {
    int first, step;
    const FlatArgs& A;
    __device__ __forceinline__ bool has(int i) const { return first + i * step < A.total; }
    // byte offset from the channel's first plane; lanes beyond the channel: its first vector, whose values nothing uses
    template <int LB> __device__ __forceinline__ unsigned offset(int i) const
    {
        const int k = has(i) ? first + i * step : 0;
        const int n = A.magic ? (int)__umulhi((unsigned)k, A.magic) : k;
        return (unsigned)n * A.image_bytes + (unsigned)(k - n * A.vecs) * (unsigned)LB;
    }
};

// sums over the lanes of a channel, in double precision, the same in every lane
template <int WAVES> __device__ __forceinline__ double flat_sum(double v, double* part)
{
    lanes_add(kWave, [&](auto off) __attribute__((always_inline)) { v = lane_add<decltype(off)::value>(v); });
    if constexpr (WAVES == 1) return v;
    const int t = (int)threadIdx.x;
    if ((t & (kWave - 1)) == 0) part[t >> 6] = v;
    __syncthreads();
    v = part[0];
#pragma unroll
    for (int w = 1; w < WAVES; ++w) v += part[w];
    return v;
}

// WAVES: wavefronts a channel, 1, 4 or 16.  S: vectors a lane.
template <typename T, int LB, int S, int WAVES, int ACT>
__global__ __launch_bounds__(flat_threads(WAVES), flat_words(LB, S) * (ACT == 2 ? 2 : 1) <= 64 ? 4 : 2) void flat_forward(FlatArgs A)
{
    typedef FlatUnit<T, LB, S> Unit;
    constexpr int E = Unit::E;
    __shared__ double part[2][flat_threads(WAVES) / kWave];
    const int t = (int)threadIdx.x, w = uniform(t >> 6), block = slab_of_block(blockIdx.x, gridDim.x);
    if (blockIdx.x == 0 && t == 0) A.sync[1] = 0u;
    const int c = WAVES == 1 ? block * (kThreads / kWave) + w : block;
    if (c >= A.C) return;
    const FlatLane L{WAVES == 1 ? t & (kWave - 1) : t, WAVES * kWave, A};
    const char* xb = static_cast<const char*>(A.x) + (size_t)c * A.plane_bytes;
    const char* rb = static_cast<const char*>(A.dy) + (size_t)c * A.plane_bytes;
    char* yb = static_cast<char*>(A.out) + (size_t)c * A.plane_bytes;
    Unit x, r;
#pragma unroll
    for (int i = 0; i < S; ++i) x.v[i] = Unit::load(xb + L.template offset<LB>(i));
    if constexpr (ACT == 2) {
#pragma unroll
        for (int i = 0; i < S; ++i) r.v[i] = Unit::load(rb + L.template offset<LB>(i));
    }
    const float pivot = Elem<T>::load1(reinterpret_cast<const T*>(xb)), gamma = load_scalar(A.gamma, c), beta = load_scalar(A.beta, c);
    float acc[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < S; ++i) {
        if (L.has(i)) {
            float f[E];
            Unit::unpack(x.v[i], f);
#pragma unroll
            for (int e = 0; e < E; ++e) acc[(i * E + e) & 3] += f[e] - pivot;
        }
    }
    const double mean = (double)pivot + flat_sum<WAVES>((double)(acc[0] + acc[1]) + (double)(acc[2] + acc[3]), part[0]) * A.inv_M_f64;
    const float mu = (float)mean, mulo = (float)(mean - (double)mu);
#pragma unroll
    for (int q = 0; q < 4; ++q) acc[q] = 0.f;
    x.forget_all();
#pragma unroll
    for (int i = 0; i < S; ++i) {
        if (L.has(i)) {
            float f[E];
            Unit::unpack(x.v[i], f);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                const float dv = f[e] - mu;
                acc[(i * E + e) & 3] += dv * dv;
            }
        }
    }
    // (about mu, which is off by mulo)
    const double sq = flat_sum<WAVES>((double)(acc[0] + acc[1]) + (double)(acc[2] + acc[3]), part[1]) * A.inv_M_f64 - (double)mulo * (double)mulo;
    const float istd = (float)rsqrt_f64((sq < 0.0 ? 0.0 : sq) + A.eps);
    const float gsc = gamma * istd, bsh = beta - gsc * mulo;
    if (L.first == 0) {
        A.mean[c] = mu;
        if (A.mean_lo) A.mean_lo[c] = mulo;
        A.invstd[c] = istd;
    }
    x.forget_all();
    const FlatLane M{(int)fresh((unsigned)L.first), L.step, A};      // (formed anew: kept, offsets and masks would cost a register or two a vector)
#pragma unroll
    for (int i = 0; i < S; ++i) {
        if (M.has(i)) {
            float f[E], h[E];
            Unit::unpack(x.v[i], f);
            if constexpr (ACT == 2) Unit::unpack(r.v[i], h);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                float z = (f[e] - mu) * gsc + bsh;
                if constexpr (ACT == 2) z += h[e];
                if (ACT != 0) z = z < 0.f ? 0.f : z;
                f[e] = z;
            }
            Unit::store(yb + M.template offset<LB>(i), Unit::pack(f));
        }
    }
}

template <typename T, int LB, int S, int WAVES, int ACT>
__global__ __launch_bounds__(flat_threads(WAVES), flat_words(LB, S) * (ACT != 0 ? 3 : 2) <= 96 ? 4 : 2) void flat_backward(FlatArgs A)
{
    typedef FlatUnit<T, LB, S> Unit;
    constexpr int E = Unit::E;
    __shared__ double part[2][flat_threads(WAVES) / kWave];
    const int t = (int)threadIdx.x, w = uniform(t >> 6), block = slab_of_block(blockIdx.x, gridDim.x);
    if (blockIdx.x == 0 && t == 0) A.sync[1] = 0u;
    const int c = WAVES == 1 ? block * (kThreads / kWave) + w : block;
    if (c >= A.C) return;
    const FlatLane L{WAVES == 1 ? t & (kWave - 1) : t, WAVES * kWave, A};
    const size_t at = (size_t)c * A.plane_bytes;
    const char* xb = static_cast<const char*>(A.x) + at;
    const char* gb = static_cast<const char*>(A.dy) + at;
    const char* ab = static_cast<const char*>(A.aux) + at;
    char* ob = static_cast<char*>(A.out) + at;
    char* zb = static_cast<char*>(A.out2) + at;      // (used if A.out2 is not null)
    Unit x, g, y;
#pragma unroll
    for (int i = 0; i < S; ++i) {
        const unsigned o = L.template offset<LB>(i);
        g.v[i] = Unit::load(gb + o);
        x.v[i] = Unit::load(xb + o);
        if constexpr (ACT != 0) y.v[i] = Unit::load(ab + o);
    }
    const float mu = A.mean[c], mulo = A.mean_lo ? A.mean_lo[c] : 0.f, istd = A.invstd[c], gamma = load_scalar(A.gamma, c);
    // chains of at most 16 values, or 32 of bfloat16 (in two of 32 and 64: dgamma of 16 x 512 of 36x40 bf16 1.16 times as far from 64 bits as the
    // single-launch kernels, so 0.88; 16 x 512 of 24x30 fp32 0.95, so 0.74; no slower, 13.8 and 12.2 us)
    constexpr int CH = S * E > 32 ? 4 : 2;
    float a[CH] = {}, b[CH] = {};
#pragma unroll
    for (int i = 0; i < S; ++i) {
        if (L.has(i)) {
            float fx[E], fg[E];
            if constexpr (ACT != 0) {
                if constexpr (LB <= 4) g.v[i] = mask_by_positive<T>(g.v[i], y.v[i]);
                else {
#pragma unroll
                    for (int q = 0; q < LB / 4; ++q) g.v[i][q] = mask_by_positive<T>(g.v[i][q], y.v[i][q]);
                }
            }
            Unit::unpack(x.v[i], fx);
            Unit::unpack(g.v[i], fg);
#pragma unroll
            for (int e = 0; e < E; ++e) {
                a[(i * E + e) % CH] += fg[e];
                b[(i * E + e) % CH] += fg[e] * (fx[e] - mu);
            }
        }
    }
    double suma = (double)a[0] + (double)a[1], sumb = (double)b[0] + (double)b[1];
    if constexpr (CH == 4) {
        suma += (double)a[2] + (double)a[3];
        sumb += (double)b[2] + (double)b[3];
    }
    const double db = flat_sum<WAVES>(suma, part[0]);
    const double dg = (flat_sum<WAVES>(sumb, part[1]) - (double)mulo * db) * (double)istd;
    const float dbf = (float)db, dgf = (float)dg;
    if (L.first == 0) {
        A.dbeta[c] = dbf;
        A.dgamma[c] = dgf;
    }
    // dx = gs * (dy - c1) + (k0 - kk * (x - mu)), see slab_backward
    const float gs = gamma * istd, kk = gs * istd * (dgf * A.inv_M);
    const double c1d = db * A.inv_M_f64;
    const float c1 = (float)c1d, k0 = (float)((double)kk * (double)mulo - (double)gs * (c1d - (double)c1));
    x.forget_all();
    g.forget_all();
    const FlatLane M{(int)fresh((unsigned)L.first), L.step, A};      // (see the forward)
#pragma unroll
    for (int i = 0; i < S; ++i) {
        if (M.has(i)) {
            const unsigned o = M.template offset<LB>(i);
            float fx[E], fg[E];
            Unit::unpack(x.v[i], fx);
            Unit::unpack(g.v[i], fg);
#pragma unroll
            for (int e = 0; e < E; ++e) fg[e] = gs * (fg[e] - c1) + (k0 - kk * (fx[e] - mu));
            Unit::store(ob + o, Unit::pack(fg));
            if (ACT != 0 && A.out2 != nullptr) Unit::store(zb + o, g.v[i]);
        }
    }
}

// X(bytes of a vector, vectors a lane): one wavefront a channel, four, sixteen.  2-byte vectors: bfloat16 alone.
#define CGBN_FLAT_ONE(X) X(16, 4) X(16, 8) X(8, 8) X(8, 16) X(4, 16) X(4, 32)
#define CGBN_FLAT_FOUR(X) CGBN_FLAT_ONE(X) X(16, 16)
#define CGBN_FLAT_FOUR_FORWARD(X) X(8, 32)
#define CGBN_FLAT_SIXTEEN(X) CGBN_FLAT_ONE(X)
#define CGBN_FLAT_BF16(X) X(2, 16) X(2, 32)

}  // namespace cgbn
