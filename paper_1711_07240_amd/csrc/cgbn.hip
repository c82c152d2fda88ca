// Host side of libcgbn: argument validation, launch plan, launches, C ABI.
// See include/cgbn.h for the contract of every entry point.

#include "cgbn.h"
#include "cgbn_kernels.h"
#include "cgbn_fused.h"
#include "cgbn_fused_list.h"
#include "cgbn_slab.h"
#include "cgbn_flat.h"

#include <algorithm>
#include <atomic>
#include <cmath>
#include <cstring>
#include <map>
#include <memory>
#include <mutex>
#include <new>
#include <type_traits>
#include <utility>

// The NCHW single-launch kernels are instantiated in cgbn_fused_inst.hip (one translation
// unit per element type, direction and activation); here they are only declared.
namespace cgbn {
#define CGBN_DECL_FX(LB_, LPPC_, BIG_)                                                              \
    extern template __global__ void nchw_fused_forward<float, LB_, LPPC_, 0, BIG_>(FusedArgs);     \
    extern template __global__ void nchw_fused_forward<float, LB_, LPPC_, 1, BIG_>(FusedArgs);     \
    extern template __global__ void nchw_fused_forward<float, LB_, LPPC_, 2, BIG_>(FusedArgs);     \
    extern template __global__ void nchw_fused_forward<bf16_t, LB_, LPPC_, 2, BIG_>(FusedArgs);    \
    extern template __global__ void nchw_fused_forward<bf16_t, LB_, LPPC_, 0, BIG_>(FusedArgs);    \
    extern template __global__ void nchw_fused_forward<bf16_t, LB_, LPPC_, 1, BIG_>(FusedArgs);
#define CGBN_DECL_BX(LB_, LPPC_, BIG_)                                                              \
    extern template __global__ void nchw_fused_backward<float, LB_, LPPC_, 0, BIG_>(FusedArgs);    \
    extern template __global__ void nchw_fused_backward<float, LB_, LPPC_, 1, BIG_>(FusedArgs);    \
    extern template __global__ void nchw_fused_backward<bf16_t, LB_, LPPC_, 0, BIG_>(FusedArgs);   \
    extern template __global__ void nchw_fused_backward<bf16_t, LB_, LPPC_, 1, BIG_>(FusedArgs);
#define CGBN_DECL_F(LB_, LPPC_) CGBN_DECL_FX(LB_, LPPC_, 0)
#define CGBN_DECL_B(LB_, LPPC_) CGBN_DECL_BX(LB_, LPPC_, 0)
CGBN_FUSED_COMMON(CGBN_DECL_F)
CGBN_FUSED_FORWARD_ONLY(CGBN_DECL_F)
CGBN_FUSED_COMMON(CGBN_DECL_B)
CGBN_FUSED_BACKWARD_ONLY(CGBN_DECL_B)
CGBN_DECL_FX(16, 0, 1)
CGBN_DECL_BX(16, 0, 1)
CGBN_DECL_FX(16, -2, 1)
CGBN_DECL_BX(16, -2, 1)
#define CGBN_DECL_F1(LB_, LPPC_) CGBN_DECL_FX(LB_, LPPC_, 1)
#define CGBN_DECL_B1(LB_, LPPC_) CGBN_DECL_BX(LB_, LPPC_, 1)
CGBN_FUSED_WGP_FORWARD(CGBN_DECL_F1)
CGBN_FUSED_WGP_BACKWARD(CGBN_DECL_B1)
#undef CGBN_DECL_F1
#undef CGBN_DECL_B1
#define CGBN_DECL_F2(LB_, LPPC_) CGBN_DECL_FX(LB_, LPPC_, 2)
#define CGBN_DECL_B2(LB_, LPPC_) CGBN_DECL_BX(LB_, LPPC_, 2)
CGBN_FUSED_BIG_SMALL(CGBN_DECL_F2)
CGBN_FUSED_BIG_SMALL(CGBN_DECL_B2)
#undef CGBN_DECL_F2
#undef CGBN_DECL_B2
#define CGBN_DECL_E(LPPC_, BIG_, T_, ACT_) extern template __global__ void nchw_fused_forward<T_, 16, LPPC_, ACT_, BIG_, true>(FusedArgs);
#define CGBN_DECL_FE(LPPC_, BIG_)                                                               \
    CGBN_DECL_E(LPPC_, BIG_, float, 0) CGBN_DECL_E(LPPC_, BIG_, float, 1) CGBN_DECL_E(LPPC_, BIG_, bf16_t, 0) CGBN_DECL_E(LPPC_, BIG_, bf16_t, 1)
#define CGBN_DECL_SE(LPPC_, BIG_) CGBN_DECL_E(LPPC_, BIG_, float, 2) CGBN_DECL_E(LPPC_, BIG_, bf16_t, 2)
CGBN_FUSED_EDGE_FORWARD(CGBN_DECL_FE)
CGBN_FUSED_EDGE_SHORTCUT(CGBN_DECL_SE)
#undef CGBN_DECL_SE
#undef CGBN_DECL_E
#define CGBN_DECL_E(LPPC_, BIG_, T_, ACT_) extern template __global__ void nchw_fused_backward<T_, 16, LPPC_, ACT_, BIG_, true>(FusedArgs);
#define CGBN_DECL_BE(LPPC_, BIG_)                                                               \
    CGBN_DECL_E(LPPC_, BIG_, float, 0) CGBN_DECL_E(LPPC_, BIG_, float, 1) CGBN_DECL_E(LPPC_, BIG_, bf16_t, 0) CGBN_DECL_E(LPPC_, BIG_, bf16_t, 1)
CGBN_FUSED_EDGE_BACKWARD(CGBN_DECL_BE)
#undef CGBN_DECL_E
#undef CGBN_DECL_FE
#undef CGBN_DECL_BE
// ... the flat kernels in cgbn_flat_inst.hip
#define CGBN_DECL_L(T_, LB_, S_, WAVES_)                                                        \
    extern template __global__ void flat_forward<T_, LB_, S_, WAVES_, 0>(FlatArgs);             \
    extern template __global__ void flat_forward<T_, LB_, S_, WAVES_, 1>(FlatArgs);             \
    extern template __global__ void flat_forward<T_, LB_, S_, WAVES_, 2>(FlatArgs);             \
    extern template __global__ void flat_backward<T_, LB_, S_, WAVES_, 0>(FlatArgs);            \
    extern template __global__ void flat_backward<T_, LB_, S_, WAVES_, 1>(FlatArgs);
#define CGBN_DECL_L8(LB_, S_)                                                                   \
    extern template __global__ void flat_forward<float, LB_, S_, 4, 0>(FlatArgs);               \
    extern template __global__ void flat_forward<float, LB_, S_, 4, 1>(FlatArgs);               \
    extern template __global__ void flat_forward<float, LB_, S_, 4, 2>(FlatArgs);               \
    extern template __global__ void flat_forward<bf16_t, LB_, S_, 4, 0>(FlatArgs);              \
    extern template __global__ void flat_forward<bf16_t, LB_, S_, 4, 1>(FlatArgs);              \
    extern template __global__ void flat_forward<bf16_t, LB_, S_, 4, 2>(FlatArgs);
CGBN_FLAT_FOUR_FORWARD(CGBN_DECL_L8)
#undef CGBN_DECL_L8
#define CGBN_DECL_LF1(LB_, S_) CGBN_DECL_L(float, LB_, S_, 1)
#define CGBN_DECL_LF4(LB_, S_) CGBN_DECL_L(float, LB_, S_, 4)
#define CGBN_DECL_LF16(LB_, S_) CGBN_DECL_L(float, LB_, S_, 16)
#define CGBN_DECL_LB1(LB_, S_) CGBN_DECL_L(bf16_t, LB_, S_, 1)
#define CGBN_DECL_LB4(LB_, S_) CGBN_DECL_L(bf16_t, LB_, S_, 4)
#define CGBN_DECL_LB16(LB_, S_) CGBN_DECL_L(bf16_t, LB_, S_, 16)
CGBN_FLAT_ONE(CGBN_DECL_LF1) CGBN_FLAT_FOUR(CGBN_DECL_LF4) CGBN_FLAT_SIXTEEN(CGBN_DECL_LF16)
CGBN_FLAT_ONE(CGBN_DECL_LB1) CGBN_FLAT_FOUR(CGBN_DECL_LB4) CGBN_FLAT_SIXTEEN(CGBN_DECL_LB16)
CGBN_FLAT_BF16(CGBN_DECL_LB1) CGBN_FLAT_BF16(CGBN_DECL_LB4) CGBN_FLAT_BF16(CGBN_DECL_LB16)
#undef CGBN_DECL_L
#undef CGBN_DECL_LF1
#undef CGBN_DECL_LF4
#undef CGBN_DECL_LF16
#undef CGBN_DECL_LB1
#undef CGBN_DECL_LB4
#undef CGBN_DECL_LB16
// ... and the column-slab kernels in cgbn_slab_inst.hip
#define CGBN_DECL_SF(P_, SOLO_)                                                                 \
    extern template __global__ void slab_forward<float, 0, P_, SOLO_, false>(SlabArgs);         \
    extern template __global__ void slab_forward<float, 1, P_, SOLO_, false>(SlabArgs);         \
    extern template __global__ void slab_forward<float, 2, P_, SOLO_, false>(SlabArgs);         \
    extern template __global__ void slab_forward<bf16_t, 0, P_, SOLO_, false>(SlabArgs);        \
    extern template __global__ void slab_forward<bf16_t, 1, P_, SOLO_, false>(SlabArgs);        \
    extern template __global__ void slab_forward<bf16_t, 2, P_, SOLO_, false>(SlabArgs);
#define CGBN_DECL_SB(P_, SOLO_)                                                                 \
    extern template __global__ void slab_backward<float, 0, P_, SOLO_, false>(SlabArgs);        \
    extern template __global__ void slab_backward<float, 1, P_, SOLO_, false>(SlabArgs);        \
    extern template __global__ void slab_backward<bf16_t, 0, P_, SOLO_, false>(SlabArgs);       \
    extern template __global__ void slab_backward<bf16_t, 1, P_, SOLO_, false>(SlabArgs);
#define CGBN_DECL_SD(T_, ACT_)                                                                  \
    extern template __global__ void slab_forward<T_, ACT_, kSlabDenseForward, false, true>(SlabArgs); \
    extern template __global__ void slab_backward<T_, ACT_, kSlabDenseBackward, false, true>(SlabArgs);
CGBN_DECL_SD(float, 0)
CGBN_DECL_SD(float, 1)
CGBN_DECL_SD(bf16_t, 0)
CGBN_DECL_SD(bf16_t, 1)
#undef CGBN_DECL_SD
CGBN_SLAB_FORWARD_P(CGBN_DECL_SF)
CGBN_SLAB_BACKWARD_P(CGBN_DECL_SB)
#define CGBN_DECL_SN(P_)                                                                        \
    extern template __global__ void slab_forward<float, 0, P_, true, false, 8>(SlabArgs);       \
    extern template __global__ void slab_forward<float, 1, P_, true, false, 8>(SlabArgs);       \
    extern template __global__ void slab_forward<float, 2, P_, true, false, 8>(SlabArgs);       \
    extern template __global__ void slab_forward<bf16_t, 0, P_, true, false, 8>(SlabArgs);      \
    extern template __global__ void slab_forward<bf16_t, 1, P_, true, false, 8>(SlabArgs);      \
    extern template __global__ void slab_forward<bf16_t, 2, P_, true, false, 8>(SlabArgs);      \
    extern template __global__ void slab_backward<float, 0, P_, true, false, 8>(SlabArgs);      \
    extern template __global__ void slab_backward<float, 1, P_, true, false, 8>(SlabArgs);      \
    extern template __global__ void slab_backward<bf16_t, 0, P_, true, false, 8>(SlabArgs);     \
    extern template __global__ void slab_backward<bf16_t, 1, P_, true, false, 8>(SlabArgs);
CGBN_SLAB_NARROW_P(CGBN_DECL_SN)
#undef CGBN_DECL_SN
#undef CGBN_DECL_SF
#undef CGBN_DECL_SB
#undef CGBN_DECL_FX
#undef CGBN_DECL_BX
#undef CGBN_DECL_F
#undef CGBN_DECL_B
}  // namespace cgbn

// Scratch of cgbn_forward_static: one array per device, owned by the loaded library until the process ends.
// In host code this name is only a handle for hipGetSymbolAddress; kernels get the address that call returns.
static __device__ __align__(256) unsigned char scratch[CGBN_STATIC_SCRATCH_BYTES];

namespace {

using namespace cgbn;

// The device address of `scratch` on the current device, looked up once per device.
constexpr int kMaxDevices = 64;
void* g_scratch_ptr[kMaxDevices];
std::mutex g_scratch_lock;
cgbn_status scratch_of_current_device(void** out)
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) {
        (void)hipGetLastError();
        return CGBN_ERR_HIP;
    }
    std::lock_guard<std::mutex> hold(g_scratch_lock);
    if (!g_scratch_ptr[dev]) {
        void* ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess || !ptr) {
            (void)hipGetLastError();
            return CGBN_ERR_HIP;
        }
        g_scratch_ptr[dev] = ptr;
    }
    *out = g_scratch_ptr[dev];
    return CGBN_OK;
}

// ---- launch-shape knobs (cgbn_set_tuning) ---------------------------------
struct Tuning {
    long long chunk_bytes = 32768;       // NCHW: bytes of a plane per workgroup
    long long wave_plane_bytes = 16384;  // NCHW: planes up to this go one per wavefront
    long long tiny_planes = 1;           // NCHW: planes of at most 2 KiB (C a multiple of 8) go several to a workgroup
    long long piece_bytes = 0;           // NHWC reductions: bytes of a pixel run per workgroup; 0 = chosen per shape (see reduce_pieces)
    long long map_piece_bytes = 0;       // NHWC normalise / dx: the same for the elementwise sweeps; 0 = chosen per shape and sweep (see cut_pixels)
    long long reverse = 1;               // alternate sweep direction so a sweep starts on what the last one left in cache
    long long nt_store = 1;              // non-temporal stores for y and dx
    long long fused = 1;                 // register-resident single-launch path where the shape allows it
    long long spin_limit = 1LL << 24;    // polls of a bounded wait in the fused kernels before it gives up
    long long cooperative = 0;           // launch the single-launch kernels cooperatively (co-residency guaranteed by the runtime)
    long long big_lds = 1;               // large planes with few rows/shards: keep more unit data in LDS
    long long one_sweep_stats = 1;       // multi-sweep forward: steps 1-10 from one sweep over x (0: a sweep for the sums, one for the deviations)
    long long fused_groups = 0;          // workgroups of the fused grid (0 = as many as are resident at once)
    long long stagger = 1;               // single-launch kernels: start the channel slots class by class (see choose_stagger)
    long long stagger_us = 0;            // ... start-up delay of the last class (0 = chosen per launch)
    long long stagger_phases = 16;       // ... and the number of classes
    long long flat = 1;                  // NCHW: channels that fit one workgroup's registers go through the flat kernels
    long long wait_us = 100000;          // microseconds after which a device-side wait of the fused kernels gives up
};
// The knobs are process-wide; every call works on ONE copy of them, the one its plan was made under: taken under the lock
// (tuning_now) when the call starts, or when an earlier call of the thread made the plan, if no knob has changed since (`version` counts
// the changes).  So a knob changed by another thread in the middle of a call cannot make the plan, the
// workspace check and the launches of that call disagree.
Tuning g_tune;
std::mutex g_tune_lock;
std::atomic<unsigned> g_tune_version{0};
Tuning tuning_now()
{
    std::lock_guard<std::mutex> hold(g_tune_lock);
    return g_tune;
}
std::atomic<long long> g_last_forward_slab{0}, g_last_backward_slab{0};     // bytes of the vectors of the column-slab kernel it took, or 0
std::atomic<long long> g_last_forward_fused{0}, g_last_backward_fused{0};   // which path the last call took: 1 for a single launch of an NCHW call
std::atomic<long long> g_last_forward_flat{0}, g_last_backward_flat{0};     // ... by a flat kernel
std::atomic<long long> g_last_forward_edge{0}, g_last_backward_edge{0};     // ... by one for planes that are no multiple of 16 bytes
#ifdef CGBN_TRACE
unsigned long long* g_trace = nullptr;
#endif

// Geometry of the register-resident path for one direction (`words` 32-bit
// registers of one tensor per thread: 128 forward, 64 backward).
struct FusedPlan {
    int ok;               // shape can take the path at all (grid size is checked at launch)
    int LB;               // bytes per load: 16 or 8
    int LPPC;             // 0: large planes; else register slots per plane (an instantiated count >= LPP)
    int tp, TL, LPP, IPU, U, rows, rps, G;
    int edge;             // planes start anywhere: 16-byte loads, the values before and behind whole vectors one by one
    int big;              // 1 (large planes) / 2 (small planes): the variant that stages few rows and keeps more unit data in LDS
    long long total_units;
};

// Geometry of the flat path (see cgbn_flat.h); the same for both directions.
struct FlatPlan {
    int waves;            // wavefronts a channel (1, 4 or 16), 0: the shape cannot take the path
    int LB, S;            // bytes of a vector, vectors a lane
    int vecs, total;      // vectors of a plane, of a channel
};

// Geometry of the column-slab path for one direction (see cgbn_slab.h).
struct SlabPlan {
    int ok;               // the shape can take the path, and it is faster than separate sweeps
    int first;            // ... and faster than the single-launch NCHW kernels, where the shape can take those too
    int cols, vecs, rpp, cpc, nch, tpc, slabs, U, rpu;
    int P;                // vectors per thread of the kernel variant
    int vb;               // bytes of a vector
    int shared;           // several rounds of slabs that share lines: neighbours are in flight together (see cut_slabs_in_units)
    long long R, row_bytes, total_units;
};

constexpr int kAnyDevice = -2;
struct Plan {
    Tuning t;             // the knobs this plan was made under (the call's own copy)
    int device, cus;      // the device whose compute units the plan counts on, and how many; kAnyDevice: it does not depend on one
    int N, C, H, W, K, layout, dtype;
    int eb, vec;          // bytes per element; elements per access (NHWC: 1 if C is no multiple of a 16-byte vector, see `group`)
    int HW, ips;
    long long S;
    double M;
    // NCHW
    int wave_mode, L, sp;
    int tiny, tg;         // tiny planes: `tg` planes of consecutive channels per workgroup
    // NHWC
    int cv, TW, ctiles, rpp, PL, pps;
    long long spix;
    // pixel runs of the elementwise sweeps (no rows to keep few), with one, two (dx; a shortcut) and three (masked dx) input tensors
    struct { int PL, pps; long long grid; } map[3];
    // partial sums
    int rows, rps, G;
    long long grid;       // workgroups of one sweep
    // Channels-last, C no multiple of a 16-byte vector: `group` neighbouring pixels are whole vectors, C * group / vec of them, and are
    // taken as one pixel of C * group columns, column j a value of channel j % C.  1: no grouping.  (A thread that loads one
    // value at a time moves 2 or 4 bytes an instruction.)  `may_group`: what grouped() makes of this plan, 1 if nothing.
    int group, may_group;
    FusedPlan ff, fb;     // register-resident path, forward and backward
    FusedPlan ef, ebw;    // ... with 16-byte loads for planes that are no multiple of 16 bytes, and the calls that take them (see edges_pay):
    bool edges[4];        // forward, with a shortcut, backward, masked
    FlatPlan flat;        // the flat path, and the calls that take it before all but column slabs that come first:
    bool flats[4];        // forward, with a shortcut, backward, masked
    SlabPlan sf, sb;      // column-slab path
    SlabPlan sfs, sbm;    // ... of a forward with a shortcut, of a masked backward
    SlabPlan xf, xb, xbm; // the same in several rounds of slabs that share lines (no shortcut): taken where the others are not ok
    SlabPlan nf, nb, nfs, nbm;    // the same with 8-byte vectors: taken in their place where ok
    // workspace layout (byte offsets)
    size_t off_part0, off_part1, off_sh0, off_sh1, off_mlo, off_sync, bytes;
};

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

void make_fused_plan(const Tuning& T, int N, int C, long long HW, int K, int layout, int eb, int words, int lds_words,
                     int lds_words_big, int lds_words_big_small, bool forward, bool edge, FusedPlan* f)
{
    std::memset(f, 0, sizeof(*f));
    if (K > kFusedMaxShards) return;
    if (layout != CGBN_NCHW) return;                   // channels-last shapes: see make_slab_plan
    int LB = 0;
    for (int lb = 16; lb >= 4; lb >>= 1)
        if (HW % (lb / eb) == 0) { LB = lb; break; }
    const bool small_edges = (long long)C * HW * eb % 16 == 0;         // a channel's planes all start at the same byte of a vector
    const long long plane = HW;                        // (HW: what the slots hold of it)
    if (edge) {
        if (LB == 16 || plane * eb <= 1024) return;
        LB = 16;
        HW = HW * eb / 16 * 16 / eb;
        f->edge = 1;
    }
    if (!LB) return;                                   // bfloat16 planes with an odd element count
    const int W = LB / 4, R = words / W, E = LB / eb;
    const long long wave_cap = (long long)R * kWave * E;   // elements one wavefront can hold
    if (LB == 4 && HW > wave_cap) return;              // 4-byte loads only for small planes
    const int ips = N / K;
    const bool small_edges_or_plain = !edge || small_edges;
    f->LB = LB;
    if (edge && !small_edges && HW <= wave_cap) return;
    if (HW <= wave_cap) {
        f->LPP = (int)((HW + (long long)kWave * E - 1) / ((long long)kWave * E));
        // register slots per plane: the smallest instantiated count that holds a plane and
        // leaves at most 16 planes per wavefront
        int lppc = 0;
        for (int cand : kCgbnSlotCounts)
            if (cand >= f->LPP && cand * 16 >= R && cand <= R) { lppc = cand; break; }
        if (!lppc) return;
        if (f->LPP <= cgbn_full_slots(lppc, R)) return;    // (cannot happen: the kernels rely on it, see the table)
        f->LPPC = lppc;
        // with few rows and shards to stage, further whole planes per wavefront go to LDS
        int lds_planes = 0;
        if (T.big_lds && N <= kFusedMaxRowsBig && K <= kFusedMaxShardsBigSmall) {
            bool built = false;
#define CGBN_IS_BUILT(LB_, LPPC_) built = built || (LB == LB_ && lppc == LPPC_);
            CGBN_FUSED_BIG_SMALL(CGBN_IS_BUILT)
#undef CGBN_IS_BUILT
            if (built && !(edge && lppc == 2)) lds_planes = (lds_words_big_small / W) / lppc;
            // ... if that makes the channel's units fewer (else the variant only costs its extra slot checks)
            const int regs_only = 4 * (R / lppc), with_lds = 4 * (R / lppc + lds_planes);
            if ((N + with_lds - 1) / with_lds >= (N + regs_only - 1) / regs_only) lds_planes = 0;
        }
        f->big = lds_planes > 0 ? 2 : 0;
        int per_unit = 4 * (R / lppc + lds_planes);
        f->U = (N + per_unit - 1) / per_unit;
        f->IPU = (N + f->U - 1) / f->U;
        // byte offsets inside a unit are 32-bit
        if ((long long)f->IPU * C * plane * eb > 0x7fffffffLL) return;
        f->rows = N;
        f->rps = ips;
    } else if (LB >= 8 && small_edges_or_plain && HW <= (long long)(R + lds_words / W) * kWave * E) {
        // a plane a few slots too long for a wavefront's registers: still one plane per wavefront, the last
        // slots in LDS (four planes per unit instead of the one a "large plane" unit would hold)
        f->LPP = (int)((HW + (long long)kWave * E - 1) / ((long long)kWave * E));
        f->LPPC = R + lds_words / W;
        f->U = (N + 3) / 4;
        f->IPU = (N + f->U - 1) / f->U;
        if ((long long)f->IPU * C * plane * eb > 0x7fffffffLL) return;
        f->rows = N;
        f->rps = ips;
    } else {
        // large planes: a tile also fills the LDS slots (16-byte loads only); with few rows and shards to
        // stage, the variant with more LDS slots is taken
        const long long gran = (long long)kThreads * E;
        HW = plane;
        for (int big = (LB == 16 && T.big_lds && K <= kFusedMaxShardsBig) ? 1 : 0; big >= 0; --big) {
            const int lw = big ? lds_words_big : lds_words;
            const long long cap = wave_cap * 4 + (LB == 16 ? (long long)(lw / W) * kThreads * E : 0);
            long long tp = (HW + cap - 1) / cap;
            long long TL = (HW + tp - 1) / tp;
            TL = (TL + gran - 1) / gran * gran;
            tp = (HW + TL - 1) / TL;
            if (big && (long long)N * tp > kFusedMaxRowsBig) continue;
            if ((long long)N * tp > kFusedMaxRows) return;
            f->big = big;
            f->tp = (int)tp;
            f->TL = (int)TL;
            f->U = (int)(N * tp);
            f->rows = f->U;
            f->rps = (int)(ips * tp);
            // a plane of at most half the slots: the same channel's planes of two consecutive images per unit
            const long long unit_slots = R + (LB == 16 ? lw / W : 0);
            const long long plane_slots = (HW * eb + (long long)kThreads * LB - 1) / ((long long)kThreads * LB);
            if (LB == 16 && small_edges_or_plain && tp == 1 && N >= 2 && 2 * plane_slots <= unit_slots && (long long)C * HW * eb <= 0xffffffffLL) {
                f->LPPC = -2;
                f->U = (N + 1) / 2;
                f->rows = N;
                f->rps = ips;
            }
            break;
        }
    }
    // Three or four whole planes per workgroup in workgroup-wide slots, where the layout chosen above is one of the
    // large-plane ones (a tile or two planes per workgroup) and leaves the unit markedly emptier (measured, 64 x 256
    // planes of 100 x 100 floats forward 298 -> 284 us; 128 x 512 planes of 100 x 100 bf16 backward 904 -> 846 us)
    if (f->LPPC <= 0 && LB == 16 && small_edges_or_plain && T.big_lds && K <= kFusedMaxShardsBig && N <= kFusedMaxRowsBig && N >= 2 && (long long)C * HW * eb <= 0xffffffffLL) {
        const long long slot_bytes = (long long)kThreads * LB;
        const long long unit_slots = R + lds_words_big / W;                      // of the variant with more unit data in LDS
        const long long plane_bytes = HW * eb, plane_slots = (plane_bytes + slot_bytes - 1) / slot_bytes;
        int best = 0;
        auto consider = [&](int n) { if (unit_slots / n >= plane_slots && n <= N && n > best) best = n; };
#define CGBN_CONSIDER(LB_, LPPC_) consider(-(LPPC_));
        if (forward) { CGBN_FUSED_WGP_FORWARD(CGBN_CONSIDER) } else { CGBN_FUSED_WGP_BACKWARD(CGBN_CONSIDER) }
#undef CGBN_CONSIDER
        // planes a unit holds now
        const double now = f->LPPC == -2 ? 2.0 : 1.0 / (double)(f->tp > 0 ? f->tp : 1);
        if (best > 0 && (double)best >= 1.25 * now && (double)best * (double)plane_bytes >= 0.6 * (double)(unit_slots * slot_bytes)) {
            f->LPPC = -best;
            f->big = 1;
            f->tp = 1;
            f->U = (N + best - 1) / best;
            f->IPU = best;
            f->rows = N;
            f->rps = ips;
        }
    }
    if (f->rows > kFusedMaxRows) return;
    f->total_units = (long long)C * f->U;
    if (f->total_units > 0x7fffffffLL) return;
    int G = 1;
    while (G < kWave && G < f->rps) G <<= 1;
    f->G = G;
    f->ok = 1;
}


// A channel's planes in one wavefront, in a workgroup of four (up to 64 registers a lane: 16 KiB, 64 KiB; with 2- and 4-byte vectors 32) or in one of
// sixteen (32: 128 KiB, with 2-byte vectors 64).  One where there are many short channels, us, one / four: forward 3 x 1954 planes of 14x22 fp32 4.7 / 6.0,
// 2 x 1848 of 27x40 bf16 5.9 / 6.8, 2 x 825 of 8x11 fp32 3.4 / 4.0, 4 x 896 of 32x33 bf16 6.4 / 5.9, 8 x 680 of 14x17 fp32 5.2 / 5.1, 2 x 256 of 13x21
// 4.1 / 4.3; 2 x 512 of 25x42 bf16 backward 6.5 / 5.0, 2 x 2048 9.3 / 9.9.
// Sixteen, of which a compute unit holds one workgroup, where every channel has a compute unit: four with 64 registers / sixteen, 16 x 32 planes of 18x29
// fp32 forward 6.0 / 5.0, 16 x 128 of 36x38 bf16 masked 10.6 / 8.5, 16 x 256 of 24x30 fp32 6.8 / 7.0 and 13.2 / 12.4, 16 x 512 10.5 / 10.7 and 19.1 / 23.1;
// single-launch kernels with hand-overs / sixteen, 32 x 32 of 24x30 fp32 forward 8.7 / 5.6, backward 11.2 / 6.2, 32 x 256 15.0 / 11.2 and 21.5 / 13.8,
// 16 x 256 of 29x50 bf16 11.1 / 8.5 and 12.7 / 10.5, 16 x 512 14.9 / 13.7 and 17.1 / 18.3.  And in waves of workgroups where the planes' vectors have 2 bytes,
// which few other single-launch kernels take: 4 x 2000 of 63x65 47.7 / 40.1 and 73.1 / 55.8, 16 x 512 of 33x35 21.8 / 17.5 and 28.1 / 21.2, 16 x 800 29.0 / 29.9.
// Two waves of them with 16-byte vectors too, whose other kernels have the most rows to hand over: forward, with a shortcut and backward, 32 x 300 of 24x30
// fp32 16.6 / 12.8, 29.1 / 17.9, 24.5 / 17.7; 32 x 512 20.2 / 16.5, 34.4 / 27.2, 36.3 / 27.6; 32 x 512 of 36x46 bf16 25.2 / 19.9, 42.6 / 39.4, 43.0 / 39.0; 4 x 512
// of 96x100 bf16 18.4 / 16.3, 29.3 / 26.0, 23.9 / 23.7.  32 x 800 of 24x32 fp32 33.6 / 37.2, 60.4 / 56.4, 55.7 / 55.7.
// (The compute units of an MI355X, not of the device at hand: plans of NCHW planes beyond the column slabs' ask no device, see make_plan.)
constexpr int kFlatUnits = 256;
void make_flat_plan(int N, int C, long long HW, int eb, FlatPlan* f)
{
    std::memset(f, 0, sizeof(*f));
    const long long plane = HW * eb;
    int LB = 16;
    while (plane % LB != 0) LB /= 2;
    if (LB < eb || plane / LB > 0xffff || (long long)N * C * plane > 0x7fffffffLL) return;
    const long long channel = N * plane, total = N * (plane / LB);
    auto fits = [&](int waves) {
        const long long lane = (total + waves * kWave - 1) / (waves * kWave);
        int S = 0;
#define CGBN_FLAT_FITS(LB_, S_) if (LB == LB_ && lane <= S_ && (S == 0 || S_ < S)) S = S_;
        if (waves == 16) { CGBN_FLAT_SIXTEEN(CGBN_FLAT_FITS) } else { CGBN_FLAT_FOUR(CGBN_FLAT_FITS) CGBN_FLAT_FOUR_FORWARD(CGBN_FLAT_FITS) }
        CGBN_FLAT_BF16(CGBN_FLAT_FITS)
#undef CGBN_FLAT_FITS
        return S;
    };
    int waves = (channel <= 1024 || (channel <= 5000 && C >= 1024)) && total <= 32 * kWave ? 1 : kThreads / kWave, S = fits(waves);
    if (S == 0 || (flat_words(LB, S) > 32 && C <= kFlatUnits)) {
        S = fits(waves = 16);
        if (S == 0 || (C > kFlatUnits && !(C <= 2 * kFlatUnits ? LB == 16 || LB == 2 : LB == 2 && S == 16))) return;
    }
    f->waves = waves;
    f->LB = LB;
    f->S = S;
    f->vecs = (int)(plane / LB);
    f->total = (int)total;
}

int ceil_pow2(int v)
{
    int p = 1;
    while (p < v) p <<= 1;
    return p;
}

// The smallest built variant that takes `need` vectors per thread (0: none does), and the largest there is.
int slab_variant(bool forward, bool solo, long long need)
{
    int best = 0;
#define CGBN_SLAB_BEST(P_, SOLO_) if (SOLO_ == solo && need <= P_ && (best == 0 || P_ < best)) best = P_;
    if (forward) { CGBN_SLAB_FORWARD_P(CGBN_SLAB_BEST) } else { CGBN_SLAB_BACKWARD_P(CGBN_SLAB_BEST) }
#undef CGBN_SLAB_BEST
    return best;
}
int slab_most(bool forward, bool solo)
{
    int most = 0;
#define CGBN_SLAB_MOST(P_, SOLO_) if (SOLO_ == solo && P_ > most) most = P_;
    if (forward) { CGBN_SLAB_FORWARD_P(CGBN_SLAB_MOST) } else { CGBN_SLAB_BACKWARD_P(CGBN_SLAB_MOST) }
#undef CGBN_SLAB_MOST
    return most;
}

// 8-byte words of a plan's rows and results
long long slab_row_words(const SlabPlan& s) { return (long long)s.slabs * s.nch * 2 * (s.U + 1); }

// The matrix (vecs, R, row_bytes, cpc) is given: cuts it into slabs of `cols` vectors and `nch` channels with U units each.
// `row_words`: 8-byte words the workspace has room for (a channel's row is two a unit, its results two more).
bool cut_slabs(SlabPlan* s, int C, int cols, int nch, long long U, long long row_words, int cus, bool forward)
{
    s->vb = 16;
    s->cols = cols;
    s->nch = nch;
    s->rpp = kSlabThreads / cols;
    s->tpc = nch * kWave <= kSlabThreads ? kWave : kSlabThreads / nch;
    s->slabs = (s->vecs + cols - 1) / cols;
    s->rpu = (int)((s->R + U - 1) / U);
    s->U = (int)((s->R + s->rpu - 1) / s->rpu);       // (no empty unit)
    s->P = slab_variant(forward, s->U == 1, ((long long)s->rpu + s->rpp - 1) / s->rpp);
    s->total_units = (long long)s->slabs * s->U;
    s->ok = 0;
    if (s->cpc == 1 && cols > kSlabMaxPixelCols) return false;
    if (!s->P || nch > kSlabMaxChannels || s->slabs > C || s->total_units > 0x3fffffffLL) return false;
    if ((long long)s->rpp * s->row_bytes + (long long)cols * 16 > 0x7fffffffLL) return false;   // 32-bit lane offsets
    if (s->U > 1) {
        if (s->U > cus || s->U > 0xffff) return false;                              // a slab's units are resident together
        if (s->U > kSlabRowsPerLane * kWave) return false;
        if (slab_row_words(*s) > row_words) return false;
        if ((long long)s->slabs * ((s->U + 31) / 32) > C) return false;             // bitmap words
    }
    s->ok = 1;
    return true;
}

// Several units per slab: U so that the launch is shortest.  Rounds are whole; a round of several costs the passes of a unit plus a part that
// every hand-over costs, about that of 10 passes (6 us, against 0.6 us per pass of 512 x 16 bytes on every compute unit).  In one
// round what counts beside the passes, made and (forward that reads x alone) built into the variant, is what each unit adds to the hand-over: its
// row, its count, its fetches.  The weights are fitted to 137 calls of 0.5 to 70 MB, each with 5 to 25 numbers of units; what they pick
// is 1 to 2 % slower than the best in the mean.  Measured, forward / backward us: bf16 8400 x 64 with 255 units of half a pass
// 16.5 / 15.0, 132 of one 14.1 / 13.1, 64 of three 13.1 / 12.4, 12 of eleven 14.5 / 14.8; 8400 x 256 with 64 of three 16.6 / 15.7, 24 of six
// 15.1 / 14.8.  (Two units of half the size per compute unit instead of one: fp32 67200 x 1024 forward / backward 163 / 259 us
// against 142 / 224.)
//   One round: the fewest units of as many passes, so that the last pass is as full as it gets, in whole eights: units are
// dealt to the 8 XCDs in turn, and the same rows of neighbouring slabs then meet in one L2.  Where slabs do not end on line
// boundaries they share those lines: fp32 22400 x 264, 31 units 23.8 / 28.7, 32 units 21.5 / 24.5; 70200 x 112, 63 units 27.7 / 36.3, 64
// units 24.3 / 29.7 (rows of whole lines: no difference).  Such slabs must also all be in flight together (measured, fp32
// 268800 x 136 in four rounds 170 us, the sweeps 101).
//   Such slabs in several rounds (`shared`: at least so many in flight): those in flight are then neighbours, in whole eights of units, so that the
// lines two of them share are fetched by one XCD at about the same time and only those at the ends of the group twice.  See make_shared_plan.
bool cut_slabs_in_units(SlabPlan* s, int C, int cols, int nch, long long row_words, int cus, bool forward, bool second, int shared = 0)
{
    const int rpp = kSlabThreads / cols;
    const long long cap = (long long)rpp * slab_most(forward, false);
    const long long slabs = (s->vecs + cols - 1) / cols;
    const bool lines = cols >= 48 || (s->row_bytes % 128 == 0 && cols % 8 == 0);     // (a wide slab shares little)
    const long long least = (s->R + cap - 1) / cap < 2 ? 2 : (s->R + cap - 1) / cap;
    long long most = cus < s->R ? cus : s->R;
    if (most > kSlabRowsPerLane * kWave) most = kSlabRowsPerLane * kWave;
    if (most > row_words / (2 * slabs * nch) - 1) most = row_words / (2 * slabs * nch) - 1;
    if (shared && most > cus / shared) most = cus / shared;
    const long long top = cus / slabs < most ? cus / slabs : most;
    long long best = 0, best_cost = 0;
    for (int k = 0; k < 12; ++k) {
        // the fewest units and a few more; as many as fill the compute units once, or 3/4, 1/2, 3/8, ... of them
        long long U = k < 4 ? least + k : (k & 1 ? top * 3 >> (k / 2) : top >> (k / 2 - 2));
        if (U < least || U > most) continue;
        long long cost;
        if (slabs * U > cus / U * U) {
            if (shared) {
                U = (U + 7) / 8 * 8;
                if (U > most || 10 * slabs < 7 * ((slabs + cus / U - 1) / (cus / U)) * (cus / U)) continue;
            } else if (!lines) {
                continue;
            }
            const long long grid = cus / U * U, passes = ((s->R + U - 1) / U + rpp - 1) / rpp;
            cost = (slabs * U + grid - 1) / grid * (passes * 60 + 600);
        } else {
            if (shared) continue;                             // (one round: as any other)
            if (!lines && U >= 16 && U / 8 * 8 >= least) U = U / 8 * 8;
            const long long passes = ((s->R + U - 1) / U + rpp - 1) / rpp;
            const long long fewest = (s->R + passes * rpp - 1) / (passes * rpp), eights = (fewest + 7) / 8 * 8;
            if (fewest < 8) U = fewest;
            else if (eights <= U) U = eights;
            if (U < least) continue;
            cost = 255 + (forward && !second ? slab_variant(true, false, passes) * 10 + passes * 10 + U * 75 / 100 : passes * 40 + U / 4) + slabs * U * 60 / 100;
            if (!lines && slabs > 1 && U % 8 != 0) cost = cost * 5 / 4;
        }
        if (best == 0 || cost < best_cost) { best = U; best_cost = cost; }
    }
    if (best < 2 || !cut_slabs(s, C, cols, nch, best, row_words, cus, forward)) return false;
    s->shared = shared > 0;
    // (no unit is empty, so there may be fewer than asked for: they have to be whole eights still)
    if (shared && s->U % 8 != 0) s->ok = 0;
    return s->ok != 0;
}

// channels-last: up to how many pixels a slab is one workgroup.  (Rows shorter than a line: a workgroup shares its lines with few
// others; rows that are no whole lines: units share them.)
long long few_pixels(bool forward, bool second, long long row_bytes)
{
    if (row_bytes <= 64 || (forward && !second)) return 3072;
    if (row_bytes < 128) return !forward && second ? 2304 : 3072;
    if (forward) return row_bytes >= 1024 && row_bytes % 128 != 0 ? 3072 : 2560;
    if (!second) return row_bytes >= 1024 && row_bytes <= 3072 ? 3072 : 2688;
    return row_bytes < 1024 ? 1792 : row_bytes <= 4096 ? 2112 : 1280;
}

// Which calls take the column-slab kernels, and how they are cut.  `second`: the forward adds a shortcut, the backward is
// masked by the stored output: a tensor more.  Channels-last, C a multiple of a 16-byte vector:
//   - few pixels: one workgroup per slab, one launch, nothing to hand over.  Slabs of 2 vectors, backward of one while that
//     gives every compute unit at most one workgroup, since fewer bytes per compute unit then count for more than the half
//     lines (measured, 2 vectors -> 1, with ReLU: bf16 2100 x 512 12.8 -> 11.1, 2100 x 2048 20.2 -> 16.9; beyond, fp32 2100 x 2048 20.5 ->
//     24.0; forward 11.0 -> 12.3).  How few: where several units become faster.  Measured over 16 to 2048 channels of both types,
//     us, one unit / several, e.g. 256 channels fp32: forward of 3000 8.5 / 11.8, of 4200 11.7 / 12.6, of 5000 16.1 / 13.3; with shortcut of
//     2100 9.8 / 13.0, of 2600 13.8 / 13.3; backward of 2600 10.9 / 12.7, of 3000 12.5 / 12.7 (128 channels 13.0 / 11.8); masked of 1500
//     10.0 / 13.1, of 2100 14.6 / 14.4 (128 channels 14.7 / 12.4, 1024 bf16 17.3 / 17.3, 2048 fp32 34.8 / 23.5).
//   - beyond, units of 128-byte columns wherever a slab's units are resident together.  Measured, sweeps -> units: bf16
//     67200 x 256 38 / 49 -> 25 / 30, 16800 x 2048 67 / 94 -> 34 / 52, 268800 x 512 170 / 274 -> 135 / 233; fp32 67200 x 1024
//     154 / 247 -> 126 / 188, 268800 x 1024 599 / 974 -> at most 568 / 908.  Narrower columns lose (half a
//     line per request), wider ones make a slab's rows more than the hand-over bears.
//   - a shortcut that does not fit the registers beside x (P > 20) is fetched batch by batch during the write-out, each batch behind the
//     stores of the one before.  That is slower than the sweeps for float in several rounds (304290 x 192 172 us, so 275; 67200 x 1024
//     201, 209), for float slabs that share lines unless their units are short and in whole eights (224400 x 80 67, 80; 31970 x 456
//     53, 61), and for bf16 in
//     rounds that are not well filled (45560 x 832 5 %); it is faster where rows of more than 4 KiB crowd the sweeps (164724 x 1376 fp32
//     269, 198).
//
// NCHW, planes of at most 512 values, C a multiple of a 16-byte vector's elements (a slab starts and ends on 16 bytes):
//   - images that fit one workgroup: instead of the sweeps always.  Instead of the single-launch kernels where a channel is
//     several of their units, and where a thread holds few vectors and there are 1024 channels, or 128 and 24 images: those
//     kernels move one plane per wavefront at a time and leave most of its lanes idle.  Measured, them -> here, forward / backward us: fp32 256 x 1024 planes of 4x4 100 /
//     135 -> 12 / 14, bf16 16 x 2048 of 8x8 19 / 17 -> 8.3 / 8.0; with few channels and images they stay ahead: fp32 8 x 256
//     of 16x20 6.3 / 5.6 against 6.4 / 6.4, bf16 16 x 256 of 20x20 7.6 / 7.4 against 11.5 / 12.  Not with a second tensor, more than
//     16 passes and few slabs: bf16 20 x 24 of 13x21 with shortcut 12.6 against 14.8, 20 x 48 of 15x23 masked 13.8 against 16.5, 101 x 32 of 7x11
//     12.9 against 16.4 (with more slabs, 228 x 64 of 5x7, 18.7 against 14.7 here).
//   - several units per slab from 6 MB on (below, the hand-over costs what a launch less saves), and there before the
//     single-launch kernels while planes are at most 1 KiB and the tensor 200 MB (backward: 512 bytes, float 800, 100 MB): bf16 256 x 1024 of 7x7 31 / 37 -> 23 /
//     26, of 12x12 110 / 125 -> 49 / 60; fp32 100 x 1024 of 16x20 75 / 97 against 86 / 124.
void make_slab_plan(int N, int C, long long HW, int layout, int eb, long long row_words, int cus, const FusedPlan& f, bool forward,
                    bool second, SlabPlan* s)
{
    std::memset(s, 0, sizeof(*s));
    const int vec = 16 / eb;
    if (C % vec != 0 || (layout == CGBN_NCHW && HW > kSlabThreads)) return;
    if (layout == CGBN_NHWC) {
        s->vecs = C / vec;
        s->R = (long long)N * HW;
        s->row_bytes = (long long)C * eb;
        s->cpc = 1;
        const int pair = s->vecs < 2 || (!forward && s->vecs <= cus) ? 1 : 2;
        if ((s->R <= few_pixels(forward, second, s->row_bytes) || (forward && !second && s->R <= 5120 && s->R * s->row_bytes <= 6000000)) &&
            cut_slabs(s, C, pair, pair * vec, 1, row_words, cus, forward))
            return;
        // about 8 vectors, as even as the row allows
        const int slabs = s->vecs < 12 ? 1 : (s->vecs + 4) / 8, cols = (s->vecs + slabs - 1) / slabs;
        if (cut_slabs_in_units(s, C, cols, ceil_pow2(cols * vec), row_words, cus, forward, second)) {
            if (forward && second && s->P > 20 && s->row_bytes <= 4096) {
                const int inflight = cus / s->U, rounds = (s->slabs + inflight - 1) / inflight;
                if (eb == 4 ? rounds > 1 || !((s->U % 8 == 0 && s->P <= 28) || (s->row_bytes % 128 == 0 && cols == 8))
                            : rounds > 1 && s->total_units * 3 < 2LL * rounds * cus)
                    s->ok = 0;
            }
        } else if (s->R <= 3072) {
            // (more slabs than compute units, sharing lines: still one workgroup each rather than the sweeps)
            cut_slabs(s, C, pair, pair * vec, 1, row_words, cus, forward);
        }
        return;
    }
    const long long row_vecs = (long long)C * HW / vec;
    if (row_vecs > 0x7fffffffLL) return;
    s->vecs = (int)row_vecs;
    s->R = N;
    s->row_bytes = (long long)C * HW * eb;
    s->cpc = (int)HW;
    int nch = vec;                                     // channels per slab: at least 8 vectors, if there are that many
    while (nch * 2 <= kSlabMaxChannels && nch < C && (long long)nch / vec * HW < 8) nch *= 2;
    const int cols = (int)(nch / vec * HW), rpp = kSlabThreads / cols;
    if (N <= rpp * slab_most(forward, true) && cut_slabs(s, C, cols, nch, 1, row_words, cus, forward)) {
        if (second && N > 16 * rpp && s->slabs < (rpp <= 2 ? 16 : 5)) s->ok = 0;
        s->first = !f.ok || f.U > 1 || (C >= 1024 && s->P <= (forward ? 12 : 8)) ||
                   (N >= 24 && C >= 128 && s->P <= (forward ? 8 : 4));
        return;
    }
    if (N * s->row_bytes < 6000000) return;
    if (cut_slabs_in_units(s, C, cols, nch, row_words, cus, forward, second))
        s->first = !f.ok || (f.U > 1 && (forward ? HW * eb <= 1024 && N * s->row_bytes <= 200000000 : HW * eb <= (eb == 2 ? 512 : 800) && N * s->row_bytes <= 100000000));
}

// Channels-last calls that no plan above takes, rows of at least 24 vectors that are no whole lines: in several rounds of 128-byte slabs that share
// lines, where enough of them are in flight and the rounds are at least 70 % full, and where that pays.  Measured over 454 random shapes of 5 to 420 MB, time of the
// sweeps over this one's, geometric mean of the calls taken and, in brackets, of those left, bf16 and fp32: forward 1.14 (0.95) and 1.17 (1.01), backward 1.13
// (0.91) and 1.18 (1.02), masked 1.18 (0.97) and 1.33 (1.02).  fp32 63104 x 1264 (eight and four in flight) 234 / 334 / 645 -> 187 / 281 / 498 us, 23936 x 1168 (16, ten)
// 89 / 134 / 243 -> 64 / 90 / 145.
//   - Rows of more than one tile of the sweeps (256 vectors), which are slower for them: 1.2 to 1.35 whatever the rounds; float beyond 60 slabs in rounds that are
//     not full 0.9 to 1.05, as in more than ten rounds (forward five).
//   - Rows within a line of 8 KiB (shorter ones of 4), of which the same columns of every row crowd few memory channels: 0.8 to 1.05 (26325 x 2040 fp32 masked
//     337 -> 388, 44928 x 1016 backward 160 -> 184).
//   - Shorter rows by how full the rounds are: bf16 forward 1.09 from 71 % with eight and more in flight, from 91 % with fewer, else 0.95 (46898 x 840, 14 slabs
//     by ten, 0.90); backward 1.05 from 81 % (16872 x 1656, 26 by ten, 46 -> 54 us), but for rows of up to 120 vectors (0.97); masked 1.13 from 78 % in at most
//     four rounds, else 0.97.  Float forward 1.14 from 80 % in at most four rounds, else 1.0; backward 1.12 from 84 %, but for rows of up to 107 vectors
//     (four and five in flight: 0.84 to 1.05) and four in flight in six rounds and more (0.84 to 1.04); masked 1.32 always.
//   - A forward before a backward of sweeps, which finds nothing of what this read in the last-level cache: one called directly after the other takes 0.87 to 1.04 of the
//     speed, 0.95 in the mean.  Taken so only where it gains most itself, 1.17 to 1.37 times: rows of several tiles, and from 150 MB on in at most three rounds, 90 % full.
// Fewer in flight: 97244 x 880 (two) backward 321 -> 345, 238080 x 408 (two, one) 235 / 364 -> 321 / 520, bf16 62424 x 1064 (four) masked 223 -> 249; masked float of
// rows of one tile, whose sweeps are faster: 37392 x 904 (six) 225 -> 260.  Rounds two thirds full: bf16 79872 x 496 forward 58 -> 62.  Nine columns a slab: 17920 x 1768
// 65 / 107, so 89 / 114.
bool shared_full(const SlabPlan& x, int cus, int percent)
{
    const int flight = cus / x.U;
    return 100 * x.slabs > percent * ((x.slabs + flight - 1) / flight) * flight;
}
bool shared_pays(const SlabPlan& x, int eb, int cus, bool forward, bool second)
{
    const int flight = cus / x.U, rounds = (x.slabs + flight - 1) / flight;
    auto full = [&](int percent) { return shared_full(x, cus, percent); };
    const bool bf16 = eb == 2, tiles = x.vecs > kThreads;
    if ((x.row_bytes + 128) % (tiles ? 8192 : 4096) < 256) return false;
    if (tiles && (bf16 || second)) return true;
    if (tiles && forward) return x.slabs > 62 ? x.slabs <= 5 * flight && full(85) : 20 * x.slabs <= 101 * flight || full(84);
    if (tiles) return 10 * x.slabs <= 101 * flight && (x.slabs <= 60 || full(78));
    if (forward) return bf16 ? full(flight >= 8 ? 71 : 91) : 100 * x.slabs <= 415 * flight && full(80);
    if (!second) return bf16 ? x.vecs > 120 && full(81) : x.vecs > 107 && full(84) && (flight > 4 || 2 * x.slabs <= 11 * flight);
    return !bf16 || (full(78) && rounds <= 4);
}
void make_shared_plan(int N, int C, long long HW, int eb, long long row_words, int cus, bool forward, bool second, const SlabPlan& s, SlabPlan* x)
{
    std::memset(x, 0, sizeof(*x));
    const int vec = 16 / eb;
    if (s.ok || C % vec != 0 || C / vec < 24) return;
    x->vecs = C / vec;
    x->R = (long long)N * HW;
    x->row_bytes = (long long)C * eb;
    x->cpc = 1;
    const int cols = 8;
    if (x->row_bytes % 128 == 0) return;       // (whole lines)
    const int flight = forward ? 6 : eb == 2 ? 5 : second && x->vecs <= kThreads ? 8 : 4;
    if (cut_slabs_in_units(x, C, cols, ceil_pow2(cols * vec), row_words, cus, forward, second, flight) && !shared_pays(*x, eb, cus, forward, second)) x->ok = 0;
}

// NCHW calls whose plan `s` has 16-byte vectors: one of 8-byte vectors in its place (see SlabVector), where that leaves at least half the compute
// units without a workgroup or a slab is several units.  Measured over 140 random shapes, 16 bytes / 8: forward 1.22, with a shortcut 1.21, backward
// 1.18, masked 1.13 times faster; from 129 to 255 slabs of 16 bytes, where a compute unit would come to hold two of 8, 1.02, 0.97, 0.96, 0.92.
void make_narrow_plan(int N, int C, long long HW, int eb, bool forward, bool second, const SlabPlan& s, int cus, SlabPlan* n)
{
    std::memset(n, 0, sizeof(*n));
    const int vec = 8 / eb;
    if (!s.ok || s.cpc != HW || (s.U == 1 && 2 * s.slabs > cus)) return;
    // (float, four vectors a thread at most: there is little to share out; backward of 67 x 224 planes of 4x5 5.0, so 5.1, masked 5.6, 5.8)
    if (eb == 4 && s.P <= 4 && (!forward || second)) return;
    // (float, masked, many vectors: three tensors' loads on all compute units; 208 x 512 planes of 5x8 10 % slower, 216 x 40 of 4x7 6 %)
    if (eb == 4 && s.P > 8 && !forward && second) return;
    int nch = vec;
    while (nch * 2 <= kSlabMaxChannels && nch < C && (long long)nch / vec * HW < 8) nch *= 2;
    *n = s;
    n->ok = 0;
    n->vb = 8;
    n->vecs = s.vecs * 2;
    n->cols = (int)(nch / vec * HW);
    n->nch = nch;
    n->rpp = kSlabThreads / n->cols;
    n->tpc = nch * kWave <= kSlabThreads ? kWave : kSlabThreads / nch;
    n->slabs = (n->vecs + n->cols - 1) / n->cols;
    n->U = 1;
    n->rpu = N;
    n->total_units = n->slabs;
    n->P = 0;
    const int passes = n->rpp > 0 ? (N + n->rpp - 1) / n->rpp : 0;
#define CGBN_SLAB_BEST(P_) if (passes > 0 && passes <= P_ && n->P == 0) n->P = P_;
    CGBN_SLAB_NARROW_P(CGBN_SLAB_BEST)
#undef CGBN_SLAB_BEST
    if (!n->P || n->slabs > C || (s.U > 1 && n->slabs > cus)) return;
    if ((long long)n->rpp * n->row_bytes + (long long)n->cols * 8 > 0x7fffffffLL) return;
    n->ok = 1;
}

// the current device, -1 if there is none to ask
int current_device()
{
    int dev = 0;
    if (hipGetDevice(&dev) == hipSuccess && dev >= 0) return dev;
    (void)hipGetLastError();
    return -1;
}
// its compute units (256 if there is none to ask)
int compute_units(int dev = current_device())
{
    static std::atomic<int> known[kMaxDevices];
    if (dev < 0 || dev >= kMaxDevices) return 256;
    int cus = known[dev].load(std::memory_order_relaxed);
    if (cus > 0) return cus;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
    known[dev].store(cus, std::memory_order_relaxed);
    return cus;
}

// Pixels per workgroup of the channels-last reduction sweeps.  Measured: these sweeps run
// fastest when the shards are cut into equal pieces and the grid is a whole multiple of the
// compute-unit count (one or two workgroups per unit: 5.7 TB/s against 4.0 with ragged,
// unbalanced pieces), and every further row of partials costs time in the combine step.
// So: the fewest pieces per shard, between `least_bytes` (128 KiB) and 4 MiB each, that fill the last
// round of workgroups best.
long long reduce_pieces(long long spix, int K, int ctiles, int rpp, long long tile_row_bytes, long long least_bytes, int cus)
{
    const long long quantum = 4LL * rpp;                 // four pixels per thread and pass
    const long long max_pixels = (4LL << 20) / tile_row_bytes > quantum ? (4LL << 20) / tile_row_bytes : quantum;
    const long long first = (spix + max_pixels - 1) / max_pixels;      // fewest pieces of at most 4 MiB
    long long best_pps = first;
    double best = -1.0;
    for (long long pps = first; pps <= first + 2LL * cus; ++pps) {
        long long PL = (spix + pps - 1) / pps;
        PL = (PL + quantum - 1) / quantum * quantum;
        if (PL * tile_row_bytes < least_bytes && pps > first) break;   // too short from here on
        const long long grid = (spix + PL - 1) / PL * K * ctiles;
        const long long rounds = (grid + cus - 1) / cus;
        const double fill = (double)grid / (double)(rounds * cus);
        if (fill > best + 0.02) { best = fill; best_pps = pps; }         // ties go to fewer pieces
        if (fill > 0.98) break;
    }
    long long PL = (spix + best_pps - 1) / best_pps;
    return (PL + quantum - 1) / quantum * quantum;
}

// Pixel runs of the channels-last sweeps over `spix` pixels of `cols` columns a shard (p->vec, K given).  False: too many.
bool cut_pixels(const Tuning& T, long long spix, int cols, int K, Plan* p)
{
    p->cv = cols / p->vec;
    p->TW = p->cv < kThreads ? p->cv : kThreads;
    p->ctiles = (p->cv + p->TW - 1) / p->TW;
    p->rpp = kThreads / p->TW;
    p->spix = spix;
    long long PL;
    if (T.piece_bytes > 0) {
        PL = T.piece_bytes / ((long long)cols * p->eb);
        PL -= PL % (4 * p->rpp);                           // four pixels per thread and pass
        if (PL < 4 * p->rpp) PL = 4 * p->rpp;
    } else {
        // (grouped pixels: sweeps are all there is, also for small tensors, and a handful of workgroups would leave the chip idle: pieces from
        // 16 KiB on while two workgroups a compute unit do not come together.  Not beyond: every row costs the combine step; forward of
        // 104 x 72 x 103 x 31 fp32, 1248 rows 81 us, 728 rows 70)
        long long least = 128 << 10;
        if (p->group > 1) least = std::min(least, std::max(16LL << 10, p->S * p->eb / (2LL * p->cus)));
        PL = reduce_pieces(p->spix, K, p->ctiles, p->rpp, (long long)p->TW * p->vec * p->eb, least, p->cus);
    }
    if (PL > p->spix) PL = p->spix;
    p->PL = (int)PL;
    long long pps = (p->spix + PL - 1) / PL;
    if (pps * K > 0x3fffffffLL) return false;
    p->pps = (int)pps;
    p->rows = (int)(pps * K);
    p->rps = (int)pps;
    p->grid = (long long)p->rows * p->ctiles;
    // Pixel runs of the elementwise sweeps: 32 KiB; shorter, but at least four pixels a thread, where that leaves less than two
    // workgroups a compute unit.  Measured, 32 / 64 / 128 KiB, us: with fixed statistics 2 x 200 x 336 x 256 bf16 24.5 / 25.7 / 28.7, fp32 50.2 /
    // 54.0 / 58.5, 4 x 100 x 100 x 64 bf16 3.9 / 4.7 / 6.1; as the last sweep of a forward / backward of 64 x 50 x 84 x 512 bf16 169 / 249, 173 / 256,
    // 176 / 264, fp32 316 / 485, 319 / 502, 325 / 515.
    //   Value by value at most 16 values a thread, two chunks.  Fixed statistics / dx, 32 KiB -> 16 values: 67 x 68 x 69 x 87 bf16 27.3 / 46 ->
    // 24.1 / 31, fp32 331 x 441 x 149 41.1 / 51.6 -> 36.6 / 46.7, 9 x 79 x 85 x 249 20.6 / 33.8 -> 20.2 / 32.1.
    //   Rows of several tiles: 32 KiB of a workgroup's own tile (fixed statistics / dx of 8 x 100 x 50 x 2560 bf16, of the whole row 119 / 163 us, of
    // the tile 98 / 141; fp32 64 x 20 x 20 x 1376 68.4, 65.9), of two fp32 inputs, or more than
    // two tiles, of the whole row (dx of 64 x 20 x 20 x 1376 87 us, of the tile 93; fixed statistics 64 x 40 x 40 x 2056 300, 326).  96 KiB
    // where the last tile is shorter, and its workgroups have less, of bf16: 64 x 40 x 40 x 2560 252 / 348 -> 235 / 337, 64 x 40 x 40 x 2056 270 / 352 -> 234 / 313
    // (fp32 64 x 20 x 20 x 2304 86 us, so 100).
    //   Vectors of float, two inputs: shorter pieces only where one and a half workgroups a compute unit do not come together (dx of
    // 13 to 16 MB, 392 to 490 workgroups of 32 KiB, 8.4 / 9.5 us, of 16 KiB 9.1 / 10.6); three: 16 KiB (masked backward of 64 x 50 x 84 x 512 723 ->
    // 706 us, 64 x 50 x 84 x 1024 1314 -> 1286).
    const bool f32 = p->eb == 4 && p->vec != 1;
    for (int inputs = 1; inputs <= 3; ++inputs) {
        const long long quantum = 4 * p->rpp, enough = f32 && inputs > 1 ? p->cus * 3 / 2 : p->cus * 2;
        const bool row = T.map_piece_bytes > 0 || p->vec == 1 || (f32 && (inputs > 1 || p->ctiles > 2));
        long long bytes = T.map_piece_bytes > 0 ? T.map_piece_bytes : f32 && inputs == 3 ? 16384 : 32768, PL, pps;
        for (;; bytes /= 2) {
            PL = bytes / (row ? (long long)cols * p->eb : (long long)p->TW * p->vec * p->eb);
            if (!row && !f32 && p->cv % p->TW != 0) PL *= 3;
            if (p->vec == 1 && T.map_piece_bytes == 0) PL = std::min(PL, bytes / 2048 * p->rpp);
            PL -= PL % quantum;
            if (PL < quantum) PL = quantum;
            if (PL > p->spix) PL = p->spix;
            pps = (p->spix + PL - 1) / PL;
            if (T.map_piece_bytes > 0 || PL <= quantum || pps * K * p->ctiles >= enough) break;
        }
        // (a launch has less than 2^32 threads: tensors of 70 GB and more, value by value)
        while (pps * K * p->ctiles >= (1LL << 32) / kThreads && PL < p->spix) {
            PL = std::min(2 * PL, p->spix);
            pps = (p->spix + PL - 1) / PL;
        }
        if (pps * K > 0x3fffffffLL || pps * K * p->ctiles > 0x7fffffffLL) return false;
        p->map[inputs - 1] = {(int)PL, (int)pps, pps * K * p->ctiles};
    }
    return p->grid <= 0x7fffffffLL;
}

// The plan with pixels grouped (see Plan::group).  Where a shard is no whole number of groups, the tensor is taken as one shard: the
// calls that use this plan hand out pooled sums only.  False: the tensor is no whole number of groups, or a group more than one tile.
// Measured, value by value -> grouped, forward / backward us: 16 x 60 x 61 x 187 bf16 49.7 / 72.3 -> 32.9 / 34.8, fp32 39.8 / 53.0 -> 35.3 /
// 42.5.
bool group_pixels(const Plan& p, Plan* q)
{
    const int vec = 16 / p.eb;
    int g = vec;
    for (int c = p.C; c % 2 == 0 && g > 1; c /= 2) g /= 2;
    const long long pixels = (long long)p.N * p.HW;
    if (p.S * p.eb < (256 << 10)) return false;        // (fewer, wider rows of threads then cost more than they gain: 2 x 7 x 9 x 50 fp32 11.6 / 9.2 us, grouped 13.6 / 10.9)
    if (g == 1 || pixels % g != 0 || (long long)p.C * g > 0x3fffffffLL) return false;
    *q = p;
    q->vec = vec;
    q->group = g;
    if (pixels / p.K % g != 0) q->K = 1;
    if (!cut_pixels(p.t, pixels / q->K / g, p.C * g, q->K, q)) return false;
    // (several tiles: a channel's columns lie in different workgroups, so every column needs a row; forward / backward of 8 x 50 x 60 x 766
    // bf16 58 / 71 us, value by value 43 / 61)
    return q->ctiles == 1;
}
// Whether a reduction (over dy too, or x alone) groups pixels: a thread that takes few values one by one has little to gain, and the
// wider rows of threads keep fewer workgroups busy.  Measured, values a thread one by one: time one by one, grouped, us: forward bf16
// 16 x 4 x 6 x 414 24: 12.5, 15.6; 24 x 8 x 8 x 414 64: 14.9, 16.4; 15 x 32 x 52 x 13 87: 18.5, 14.6; 8 x 14 x 14 x 302 196: 23.0, 14.3; backward
// 64 x 7 x 8 x 98 28: 14.7, 16.0 (masked 15.9, 16.5); 32 x 7 x 8 x 150 56: 14.6, 14.3; 16 x 8 x 8 x 203 64: 15.1, 14.5 (masked 18.2, 15.1);
// fp32 forward 106 x 4 x 5 x 163 20: 16.4, 17.2; masked 11 x 4 x 6 x 414 24: 10.9, 12.1; 16 x 8 x 8 x 203 64: 15.1, 11.7.
// Where a shard is no whole number of groups its pixels are pooled, which leaves fewer rows to join: always (backward 200 x 5 x 5 x 34 fp32
// 21.3, 11.4; bf16 21.1, 13.6).
bool group_sums(const Plan& p, bool with_dy)
{
    if (p.may_group == 1) return false;
    return p.spix % p.may_group != 0 || p.PL / p.rpp >= (with_dy ? 40 : 80);
}
// ... and an elementwise sweep that reads `tensors` tensors.  (Small fp32 tensors of many channels: a workgroup's constants are as much as its
// data.  dx of 11 x 4 x 6 x 414 3.7 us, grouped 4.2; 32 x 10 x 10 x 414, 5.3 MB, 5.2, 5.7; 4 x 50 x 60 x 414, 20 MB, 13.4, 11.7.)
bool group_map(const Plan& p, int tensors)
{
    return p.may_group > 1 && !(p.eb == 4 && tensors > 1 && p.C > kThreads && p.S * p.eb < (8 << 20));
}
Plan grouped(const Plan& p)
{
    Plan q = p;
    if (p.may_group > 1) group_pixels(p, &q);
    return q;
}

// Which calls on NCHW planes that are no multiple of 16 bytes take the single-launch kernels with 16-byte loads, the values of a plane before and
// behind its whole vectors one by one (`e`), rather than what there is else (`f`: the same kernels with 8- or 4-byte loads; where that is not ok,
// sweeps).  Measured over 1000 random shapes of 0.4 to 400 MB, that time over this one's, geometric means of the calls taken and, in brackets, of those
// left; single calls lie up to 9 % beside that, the same code in another process does where tensors about fill the 256 MB last-level cache:
//   - the sweeps: forward 1.25 (0.93), with a shortcut 1.15 (0.95), backward 1.30 (0.83), masked 1.38 (0.91).  Left to them: fewer than 16 channels of several
//     units, all of whose units read, wait and write together (77 x 8 of 329 x 399 fp32 backward 316 / 497 us, 71 x 8 of 289 x 223 forward 0.67; backwards of up to 13 MB 1.15); tiles that fill
//     too little of a unit (74 x 19 of 109 x 195 bf16 forward 44.5 / 50.5, 20 x 148 of 109 x 103 backward 61.6 / 71.7); few units, which leave the chip idle, and
//     a few more than are resident at once, three a compute unit (58 x 416 of 29 x 45 bf16 forward 45 / 51); many of next to nothing (1 x 3200 of 19 x 31 fp32
//     masked 20.5 / 23.0); with a shortcut, whose write-out waits for it batch by batch, all but large tensors of well filled units (5 x 80 of 211 x 315 fp32
//     76 / 95; 15 x 312 of 43 x 69 bf16 28 / 38; from 100 to 160 MB 0.92 where the units are more than are resident, else 1.1).
//   - 4-byte loads, planes beyond 8 KB (bfloat16 of 8000 bytes 0.78 to 0.95 but for large tensors): forward 1.25; with a shortcut 1.13 from 85 and 100 MB on and bfloat16 channels
//     of one unit, else 0.95; backward 1.08 and masked 1.12, but 0.98 from 12 KB on (masked 1.08 from 60 MB on); few units of several a channel 0.96.  Shorter
//     planes of float where their slots are filled: forward 1.15 from 150 MB on and 1.1 to 1.5 where a channel becomes one unit, else 0.9 to 1.0; with a
//     shortcut 1.2 from 100 MB on, else 0.9; backward 1.08 from 150 MB on, else 0.8 to 1.1; masked 1.05 to 1.25 from 70 MB on without further planes in LDS,
//     else 0.77 to 1.1.
//   - 8-byte loads, which large planes take without further data in LDS: forward beyond 16 KB 1.15, but 0.62 where a plane a wavefront became a plane a workgroup, 0.95
//     where few planes that share one leave the chip idle, and 1.04 from 80 to 160 MB, where a backward that follows then takes longer (a step 0.97); backward 1.14
//     and masked 1.11 where two or three planes share a workgroup, 0.99 and 1.00 for tiles.
bool edges_pay(const FusedPlan& e, const FusedPlan& f, bool built, int C, long long plane_bytes, long long tensor_bytes, int eb, bool forward, bool second)
{
    if (!e.ok) return false;
    const long long unit_bytes = tensor_bytes / e.total_units;
    if (!f.ok || !built) {
        if (plane_bytes <= 2048 && (second || e.U > 1 || e.total_units < 128)) return false;
        if (e.U > 1 && C < 16 && (forward || tensor_bytes > 13000000)) return false;
        if (unit_bytes < 4096 && e.total_units > 1600) return false;
        const long long thin = forward ? (C < 32 ? 70000 : 52000) : second ? (tensor_bytes < 60000000 ? 18000 : 0) : 33000;
        if (e.U > 1 && e.LPPC == 0 && unit_bytes < thin && (!forward || tensor_bytes < 200000000)) return false;
        if (forward && second) return !(e.LPPC > 0 && e.LPPC < 8) && (e.U == 1 || e.total_units <= 768 ? tensor_bytes >= 100000000 : tensor_bytes >= 160000000 && unit_bytes >= 65000);
        if (forward && tensor_bytes < 100000000 && e.total_units > 768 && e.total_units < 900) return false;
        return e.total_units >= (e.U == 1 ? 48 : !forward ? 96 : tensor_bytes >= 45000000 ? 256 : 400);
    }
    if (f.LB == 4) {
        if (e.U > 1 && e.total_units < 256) return false;
        if (!forward && plane_bytes > 12288 && (!second || tensor_bytes < 60000000)) return false;
        const bool shortcut_pays = !(forward && second) || tensor_bytes >= (eb == 2 ? 100000000 : 85000000) || (eb == 2 && e.U == 1);
        if (eb == 2) return plane_bytes > 8192 && shortcut_pays;
        if (plane_bytes >= 9000) return shortcut_pays;
        if (plane_bytes < 4096 || e.LPPC <= 0 || plane_bytes * 100 < (long long)e.LPPC * 1024 * 85) return false;
        if (plane_bytes > 8192) return shortcut_pays;
        if (forward && e.U == 1 && (f.U > 1 || (second && e.total_units <= 500))) return true;
        return !second ? tensor_bytes >= 150000000 : forward ? tensor_bytes >= 100000000 : tensor_bytes >= 70000000 && e.big == 0;
    }
    if (plane_bytes <= 16384 || (forward && second)) return false;
    if (!forward) return (e.LPPC == -3 && e.total_units >= 256 && (eb == 2 || plane_bytes >= 23000)) || (e.LPPC == -2 && e.total_units >= 640 && eb == 2);
    if (e.LPPC < 0) return e.total_units >= 200;
    return e.total_units <= f.total_units && !(e.LPPC == 0 && e.U > 40 && C < 16) && (tensor_bytes < 80000000 || tensor_bytes >= 160000000);
}

// Which (bytes per access, slots per plane) variants exist for an element type, direction and activation: all of
// the list header's, except that the float ReLU backward is not built with 4-byte accesses (one slot count
// excepted; see CGBN_FUSED_RELU_BWD_F32_NARROW).  A shape whose variant is not built takes the multi-sweep kernels.
constexpr bool fused_built(bool f32, bool forward, int act, int LB, int LPPC)
{
    if (f32 && !forward && act == 1 && LB == 4) {
        bool built = false;
#define CGBN_IS_BUILT(LB_, LPPC_) built = built || (LB == LB_ && LPPC == LPPC_);
        CGBN_FUSED_RELU_BWD_F32_NARROW(CGBN_IS_BUILT)
#undef CGBN_IS_BUILT
        return built;
    }
    return true;
}

// The flat kernels take what fits them (60 shapes of random sizes up to 60 MB, 1.60 / 1.39 / 1.89 / 1.43 times as fast forward / backward / with a shortcut / masked in the geometric mean
// as the single-launch kernels and sweeps in their place), but for
// - masked backwards of float planes with 4-byte vectors whose plain backward the single-launch kernels take and whose masked one they are not built
//   for (see fused_built: separate sweeps).  Those whose plain backward they do not take either (planes of more than 4096 values, tiny ones in many
//   images) and those they are built for (24 slots) are flat;
// - backwards with 16-byte vectors of tensors that just outgrow the last-level cache (256 MB, of which a backward's three tensors take three tensors' bytes,
//   a masked one's five): there the single-launch kernels, whose loads are non-temporal and go ahead of the stores, are faster, also when
//   nothing of a call's tensors is cached before it (8 of 3500 of 23x24 fp32, 62 MB, 35.2 / 38.3; with one wavefront a channel they are not: 2 of 12000 of 24x24 fp32
//   48 / 34, which this does not look at yet).  Old / flat in us, 8 images of 23x24 fp32: backward of 44 MB 27.6 / 23.0, 62 MB 35.9 / 39.0, 88 MB 49.1 / 54.2, 141 MB 88.1 / 87.9,
//   212 MB 144 / 131 (16 of 24x30: 147 MB 87.8 / 93.9, 230 MB 145 / 141); masked 26 MB 28.7 / 23.9, 35 MB 35.3 / 37.5, 62 MB 56.6 / 64.2, 88 MB 98.2 / 89.8 (2 of 60x64 bf16 77 MB 78.5 / 85.9; 64 registers a lane: 23 x 1896 of 16x31 fp32,
//   87 MB, 81.0 / 90.8, 16 x 2000 of 24x30 92 MB 98.2 / 96.3); 16 of 24x30 masked 29 MB 32.5 / 30.5, 37 MB
//   36.5 / 43.6, backward 46 MB 27.9 / 25.0, 60 MB 38.1 / 40.4.  (Non-temporal loads here: 18 MB backward 10.6 -> 12.8, masked 15.6 -> 20.0.)
// - forwards of 64 registers a lane of such tensors: 16 of 24x30, 60 MB 28.5 / 19.7, 92 MB 37.1 / 40.6;
// - masked backwards of sixteen wavefronts a channel, 16-byte vectors, of such tensors: 32 x 300 of 24x30 fp32, 28 MB 32.3 / 30.6, 384 36 MB 35.8 / 42.5,
//   4 x 300 of 96x100 bf16, 23 MB 26.9 / 24.1, 384 30 MB 31.2 / 33.7, 512 36.1 / 48.9;
// - backwards of 64 registers a lane in 8-byte vectors: 16 of 18x29 fp32, 400 channels 11.7 / 12.0, 800 17.6 / 19.3.
bool flat_pays(const FlatPlan& f, int C, int direction)
{
    if (f.waves == 0) return false;
    const bool most = flat_words(f.LB, f.S) > 32;
    const long long bytes = (long long)f.total * f.LB * C;
    if (direction >= 2 && f.LB == 8 && most) return false;
    if (f.LB < 16 || direction == 1) return true;
    if (f.waves == 16) return direction != 3 || bytes < 28500000LL;
    if (direction == 0) return !most || bytes < 90000000LL;
    return direction == 2 ? bytes < 50000000LL || bytes > 160000000LL : bytes < 32000000LL || bytes > (most ? 90000000LL : 85000000LL);
}

cgbn_status make_plan(const Tuning& T, int N, int C, int H, int W, int layout, int dtype, int K, Plan* p)
{
    if (N < 1 || C < 1 || H < 1 || W < 1) return CGBN_ERR_SHAPE;
    if (layout != CGBN_NCHW && layout != CGBN_NHWC) return CGBN_ERR_ENUM;
    if (dtype != CGBN_F32 && dtype != CGBN_BF16) return CGBN_ERR_ENUM;
    if (K < 1 || K > N || N % K != 0) return CGBN_ERR_SHARD;
    long long HW = (long long)H * W;
    if (HW > 0x3fffffffLL) return CGBN_ERR_SHAPE;
    long long planes = (long long)N * C;
    if (planes > 0x3fffffffLL) return CGBN_ERR_SHAPE;
    long long S = planes * HW;
    if (S > (1LL << 40)) return CGBN_ERR_SHAPE;
    std::memset(p, 0, sizeof(*p));
    p->t = T;
    p->device = kAnyDevice;
    p->group = p->may_group = 1;
    p->N = N; p->C = C; p->H = H; p->W = W; p->K = K; p->layout = layout; p->dtype = dtype;
    p->eb = dtype == CGBN_F32 ? 4 : 2;
    p->HW = (int)HW;
    p->ips = N / K;
    p->S = S;
    p->M = (double)N * (double)HW;
    const int full_vec = 16 / p->eb;
    if (layout == CGBN_NHWC || (C % full_vec == 0 && HW <= kSlabThreads)) {       // (else neither sweeps nor slab plans need it)
        p->device = current_device();
        p->cus = compute_units(p->device);
    }
    if (layout == CGBN_NCHW) {
        p->vec = full_vec;
        if (T.tiny_planes && HW * p->eb <= kTinyPlaneBytes && C % 8 == 0) {
            // several planes of consecutive channels per workgroup: the most that fit the LDS stage, as a power of two
            int tg = 256;
            while (tg > 8 && (long long)tg * HW * p->eb > kTinyStageBytes) tg >>= 1;
            p->tiny = 1;
            p->tg = tg;
            p->L = (int)HW;
            p->sp = 1;
            p->grid = (long long)N * ((C + tg - 1) / tg);
        } else if (HW * p->eb <= T.wave_plane_bytes) {
            p->wave_mode = 1;
            p->L = (int)HW;
            p->sp = 1;
            p->grid = (planes + 3) / 4;
        } else {
            long long L = T.chunk_bytes / p->eb;
            L -= L % (kThreads * full_vec);                    // whole vectors for every thread
            if (L < kThreads * full_vec) L = kThreads * full_vec;
            if (L > HW) L = HW;
            p->L = (int)L;
            p->sp = (int)((HW + L - 1) / L);
            p->grid = planes * p->sp;
        }
        p->rows = N * p->sp;
        p->rps = p->ips * p->sp;
    } else {
        p->vec = (C % full_vec == 0) ? full_vec : 1;
        if (!cut_pixels(T, (long long)p->ips * HW, C, K, p)) return CGBN_ERR_SHAPE;
    }
    if (p->grid > 0x7fffffffLL || (long long)p->rows * C > (1LL << 33)) return CGBN_ERR_SHAPE;
    int G = 1;
    while (G < kWave && G < p->rps) G <<= 1;
    p->G = G;
    make_fused_plan(T, N, C, HW, K, layout, p->eb, kFusedWords, kFusedLdsWords, kFusedLdsWordsBig, kFusedLdsWordsBigSmall, true, false, &p->ff);
    make_fused_plan(T, N, C, HW, K, layout, p->eb, kFusedWords / 2, kFusedLdsWords / 2, kFusedLdsWordsBig / 2, kFusedLdsWordsBigSmall / 2, false, false, &p->fb);
    make_fused_plan(T, N, C, HW, K, layout, p->eb, kFusedWords, kFusedLdsWords, kFusedLdsWordsBig, kFusedLdsWordsBigSmall, true, true, &p->ef);
    make_fused_plan(T, N, C, HW, K, layout, p->eb, kFusedWords / 2, kFusedLdsWords / 2, kFusedLdsWordsBig / 2, kFusedLdsWordsBigSmall / 2, false, true, &p->ebw);
    // Tiny planes that would fill less than half of the register slots a single-launch variant reserves for a plane
    // run faster through the multi-sweep kernels for tiny planes (measured, 256 images, fwd / bwd us: fp32 7x7 x 1024
    // channels 46 / 58 against 132 / 105; bf16 14x14 x 1024 channels, forward, 85 against 126.  Half full, fp32
    // 14x14: level at 256 channels, the single launch ahead at 1024, 131 / 195 against 153 / 222)
    if (p->tiny) {
        for (FusedPlan* f : {&p->ff, &p->fb})
            if (f->ok && f->LPPC > 0 && 2 * f->LPP < f->LPPC) f->ok = 0;
    }
    int max_rows = p->rows;
    if (p->ff.ok && p->ff.rows > max_rows) max_rows = p->ff.rows;
    if (p->fb.ok && p->fb.rows > max_rows) max_rows = p->fb.rows;
    // the sync area comes first, so that the error word has the same offset in every workspace
    for (FusedPlan* f : {&p->ef, &p->ebw})
        if (f->rows > max_rows) f->ok = 0;                // (no more rows than the other paths have: the workspace stays as it is)
    for (int i = 0; i < 4; ++i) {
        const bool forward = i < 2, second = (i & 1) != 0;
        const FusedPlan& f = forward ? p->ff : p->fb;
        p->edges[i] = edges_pay(forward ? p->ef : p->ebw, f, fused_built(p->eb == 4, forward, second, f.LB, f.LPPC), C, HW * p->eb, S * p->eb, p->eb, forward, second);
    }
    size_t sync = align256(((size_t)kSyncHeader + 4 * (size_t)C) * sizeof(unsigned));
    size_t part = align256((size_t)C * max_rows * sizeof(float));
    size_t sh = align256((size_t)K * C * sizeof(double));
    if (layout == CGBN_NHWC && p->vec == 1) {
        // (its rows may be more, but not so many that the workspace no longer fits the static scratch)
        Plan q;
        if (group_pixels(*p, &q)) {
            const size_t more = align256((size_t)C * (q.rows > max_rows ? q.rows : max_rows) * sizeof(float));
            if (more == part || (more <= std::max(2 * part, (size_t)(512u << 10)) &&
                                 sync + 2 * more + 2 * sh + align256((size_t)C * sizeof(float)) <= (size_t)CGBN_STATIC_SCRATCH_BYTES)) {
                part = more;
                p->may_group = q.group;
            }
        }
    }
    // The column-slab path keeps its rows where the other paths keep theirs and the shard sums (the four arrays are adjacent)
    // and makes that room larger only up to a MiB, or twice the rows of the others while the workspace still fits the static
    // scratch, so that it changes no limit.
    const size_t mlo = align256((size_t)C * sizeof(float)), others = 2 * part + 2 * sh;
    size_t room = others > (1u << 20) ? others : (1u << 20);
    if (sync + others + 2 * part + mlo <= (size_t)CGBN_STATIC_SCRATCH_BYTES && others + 2 * part > room) room = others + 2 * part;
    const long long row_words = (long long)(room / sizeof(double));
    const int cus = p->cus;
    for (const bool forward : {true, false}) {
        SlabPlan &one = forward ? p->sf : p->sb, &two = forward ? p->sfs : p->sbm;
        make_slab_plan(N, C, HW, layout, p->eb, row_words, cus, forward ? p->ff : p->fb, forward, false, &one);
        two = one;
        // (what a second tensor changes: see there)
        if (one.ok && (one.U == 1 ? layout == CGBN_NCHW || one.R > few_pixels(forward, true, one.row_bytes) : forward))
            make_slab_plan(N, C, HW, layout, p->eb, row_words, cus, forward ? p->ff : p->fb, forward, true, &two);
    }
    // (the images that the single-launch kernels take: callers are told that calls of more are separate sweeps)
    if (layout == CGBN_NCHW && N <= kFusedMaxRows && K <= kFusedMaxShards && T.flat) make_flat_plan(N, C, HW, p->eb, &p->flat);
    for (int i = 0; i < 4; ++i) {
        const FusedPlan& f = i < 2 ? p->ff : p->fb;
        p->flats[i] = flat_pays(p->flat, C, i) && !(f.ok && !fused_built(p->eb == 4, i < 2, i & 1, f.LB, f.LPPC));
    }
    if (layout == CGBN_NCHW) {
        make_narrow_plan(N, C, HW, p->eb, true, false, p->sf, cus, &p->nf);
        make_narrow_plan(N, C, HW, p->eb, true, true, p->sfs, cus, &p->nfs);
        make_narrow_plan(N, C, HW, p->eb, false, false, p->sb, cus, &p->nb);
        make_narrow_plan(N, C, HW, p->eb, false, true, p->sbm, cus, &p->nbm);
    }
    if (layout == CGBN_NHWC) {
        make_shared_plan(N, C, HW, p->eb, row_words, cus, false, false, p->sb, &p->xb);
        make_shared_plan(N, C, HW, p->eb, row_words, cus, true, false, p->sf, &p->xf);
        if (p->xf.ok && !p->xb.ok && !p->sb.ok && p->xf.vecs <= kThreads && (S * p->eb < 150000000 || p->xf.slabs > 3 * (cus / p->xf.U) || !shared_full(p->xf, cus, 90)))
            p->xf.ok = 0;                                 // (see shared_pays)
        make_shared_plan(N, C, HW, p->eb, row_words, cus, false, true, p->sbm, &p->xbm);
    }
    for (const SlabPlan* s : {&p->sf, &p->sfs, &p->sb, &p->sbm, &p->xf, &p->xb, &p->xbm})
        if (s->ok && s->U > 1) {
            const size_t need = (size_t)slab_row_words(*s) * sizeof(double);
            if (need > 2 * part + 2 * sh) part = align256((need - 2 * sh + 1) / 2);
        }
    p->off_sync = 0;
    p->off_part0 = sync;
    p->off_part1 = sync + part;
    p->off_sh0 = sync + 2 * part;
    p->off_sh1 = sync + 2 * part + sh;
    p->off_mlo = sync + 2 * part + 2 * sh;
    p->bytes = p->off_mlo + mlo;
    return CGBN_OK;
}

// The plan of a call, from this thread's last plans or made anew.  A plan follows from its key alone: the sizes, the knobs (by
// their version: a plan made while they change is not kept) and, if it counts compute units, the device.  Making one takes 2 us, 9 with a
// large shard channels-last, of the 10 us a small call took on the host; a training run comes back to the same few dozen layers.  Kept by
// four to a hash value, the one longest unused making room: with one to a value up to 7 of the 16 layer
// shapes of a detector, by the image's width, shared one and drove each other out at every step.
struct KeptPlan {
    Plan p, g;            // g: grouped(p)
    int key[7];
    unsigned version;
    unsigned used;        // when it was last taken
    bool valid = false;
    // the plan of a channels-last reduction whose sums are handed out pooled
    const Plan& sums(bool with_dy) const { return group_sums(p, with_dy) ? g : p; }
    const Plan& map(int tensors) const { return group_map(p, tensors) ? g : p; }
};
constexpr int kKeptSets = 128, kKeptWays = 4;
thread_local unsigned g_plans_made = 0;
cgbn_status plan_of(int N, int C, int H, int W, int layout, int dtype, int K, const KeptPlan** out)
{
    static thread_local std::unique_ptr<KeptPlan> kept[kKeptSets][kKeptWays];
    static thread_local unsigned clock = 0;
    const int key[7] = {N, C, H, W, layout, dtype, K};
    unsigned hash = 0;
    for (int v : key) hash = (hash ^ (unsigned)v) * 0x9e3779b1u, hash ^= hash >> 15;
    auto& set = kept[hash % kKeptSets];
    const unsigned version = g_tune_version.load(std::memory_order_acquire);
    int dev = kAnyDevice;          // (asked for only if a plan depends on it)
    for (auto& k : set) {
        if (!k || !k->valid || k->version != version || std::memcmp(k->key, key, sizeof(key)) != 0) continue;
        if (k->p.device != kAnyDevice) {
            if (dev == kAnyDevice) dev = current_device();
            if (k->p.device != dev) continue;
        }
        k->used = ++clock;
        *out = k.get();
        return CGBN_OK;
    }
    std::unique_ptr<KeptPlan>* room = &set[0];
    for (auto& k : set) {
        if (!k || !k->valid || k->version != version) { room = &k; break; }
        if (clock - k->used > clock - (*room)->used) room = &k;
    }
    std::unique_ptr<KeptPlan>& k = *room;
    Plan p;
    const cgbn_status s = make_plan(tuning_now(), N, C, H, W, layout, dtype, K, &p);
    if (s != CGBN_OK) return s;
    ++g_plans_made;
    if (!k) k.reset(new (std::nothrow) KeptPlan);
    if (!k) return CGBN_ERR_HIP;
    k->p = p;
    k->g = grouped(p);
    std::memcpy(k->key, key, sizeof(key));
    k->version = version;
    k->used = ++clock;
    k->valid = g_tune_version.load(std::memory_order_acquire) == version;
    *out = k.get();
    return CGBN_OK;
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

cgbn_status check_ws(const Plan& p, const void* ws, size_t bytes)
{
    if (!ws || ((uintptr_t)ws & 255u) != 0 || bytes < p.bytes) return CGBN_ERR_WORKSPACE;
    return CGBN_OK;
}

cgbn_status launched()
{
    return hipGetLastError() == hipSuccess ? CGBN_OK : CGBN_ERR_HIP;
}

SweepArgs sweep_args(const Plan& p)
{
    SweepArgs A;
    std::memset(&A, 0, sizeof(A));
    A.ch = p.C; A.group = p.group;
    A.S = p.S; A.N = p.N; A.C = p.C * p.group; A.HW = p.HW; A.rows = p.rows;
    A.L = p.L; A.sp = p.sp;
    A.cv = p.cv; A.TW = p.TW; A.ctiles = p.ctiles; A.rpp = p.rpp; A.PL = p.PL; A.pps = p.pps;
    A.spix = p.spix;
    A.tg = p.tg;
    A.pivot_stride = p.layout == CGBN_NCHW ? p.HW : 1;
    A.inv_M = (float)(1.0 / p.M);
    A.nt = (int)p.t.nt_store;
    return A;
}

template <typename T, int OP> void launch_reduce_t(const Plan& p, const SweepArgs& A, hipStream_t st)
{
    dim3 grid((unsigned)p.grid), block(kThreads);
    if (p.layout == CGBN_NCHW) {
        if (p.tiny) hipLaunchKernelGGL((nchw_reduce_tiny<T, OP>), grid, block, 0, st, A);
        else if (p.wave_mode) hipLaunchKernelGGL((nchw_reduce_wave<T, OP>), grid, block, 0, st, A);
        else hipLaunchKernelGGL((nchw_reduce_block<T, OP>), grid, block, 0, st, A);
    } else {
        if (p.vec == 1) hipLaunchKernelGGL((nhwc_reduce<T, 1, OP>), grid, block, 0, st, A);
        else hipLaunchKernelGGL((nhwc_reduce<T, Elem<T>::VEC, OP>), grid, block, 0, st, A);
    }
}

// (see MapConsts)
bool single_consts(const Plan& p) { return p.ctiles == 1 && p.S * p.eb > (256LL << 20); }

template <typename T, int EL> void launch_map_t(const Plan& p, const SweepArgs& A, hipStream_t st)
{
    dim3 block(kThreads);
    if (p.layout == CGBN_NCHW) {
        dim3 grid((unsigned)p.grid);
        if (p.tiny) hipLaunchKernelGGL((nchw_map_tiny<T, EL>), grid, block, 0, st, A);
        else if (p.wave_mode) hipLaunchKernelGGL((nchw_map_wave<T, EL>), grid, block, 0, st, A);
        else hipLaunchKernelGGL((nchw_map_block<T, EL>), grid, block, 0, st, A);
    } else {
        const auto& cut = p.map[el_has_3(EL) ? 2 : el_has_2(EL) ? 1 : 0];
        dim3 grid((unsigned)cut.grid);
        SweepArgs B = A;              // the elementwise sweeps cut the pixel runs their own way
        B.PL = cut.PL;
        B.pps = cut.pps;
        B.single_consts = single_consts(p);
        const bool fixed = EL == EL_FROZEN || EL == EL_SCALE;
        const size_t lds = sizeof(float) * map_const_words<EL>() * (p.group > 1 ? p.C : fixed ? kThreads : 0);
        if (p.vec == 1) hipLaunchKernelGGL((nhwc_map<T, 1, EL, false>), grid, block, 0, st, B);
        else if (p.group == 1) hipLaunchKernelGGL((nhwc_map<T, Elem<T>::VEC, EL, false>), grid, block, lds, st, B);
        else hipLaunchKernelGGL((nhwc_map<T, Elem<T>::VEC, EL, true>), grid, block, lds, st, B);
    }
}

cgbn_status launch_reduce(int op, const Plan& p, const SweepArgs& A, hipStream_t st)
{
    const bool f32 = p.dtype == CGBN_F32;
    switch (op) {
    case OP_SUM:   f32 ? launch_reduce_t<float, OP_SUM>(p, A, st)   : launch_reduce_t<bf16_t, OP_SUM>(p, A, st); break;
    case OP_SQDEV: f32 ? launch_reduce_t<float, OP_SQDEV>(p, A, st) : launch_reduce_t<bf16_t, OP_SQDEV>(p, A, st); break;
    case OP_BWD:   f32 ? launch_reduce_t<float, OP_BWD>(p, A, st)   : launch_reduce_t<bf16_t, OP_BWD>(p, A, st); break;
    case OP_MOMENTS: f32 ? launch_reduce_t<float, OP_MOMENTS>(p, A, st) : launch_reduce_t<bf16_t, OP_MOMENTS>(p, A, st); break;
    default:       f32 ? launch_reduce_t<float, OP_BWD_RELU>(p, A, st) : launch_reduce_t<bf16_t, OP_BWD_RELU>(p, A, st); break;
    }
    return launched();
}

cgbn_status launch_map(int el, const Plan& p, const SweepArgs& A, hipStream_t st)
{
    const bool f32 = p.dtype == CGBN_F32;
    switch (el) {
    case EL_NORM:   f32 ? launch_map_t<float, EL_NORM>(p, A, st)   : launch_map_t<bf16_t, EL_NORM>(p, A, st); break;
    case EL_DX:     f32 ? launch_map_t<float, EL_DX>(p, A, st)     : launch_map_t<bf16_t, EL_DX>(p, A, st); break;
    case EL_FROZEN: f32 ? launch_map_t<float, EL_FROZEN>(p, A, st) : launch_map_t<bf16_t, EL_FROZEN>(p, A, st); break;
    case EL_NORM_RELU: f32 ? launch_map_t<float, EL_NORM_RELU>(p, A, st) : launch_map_t<bf16_t, EL_NORM_RELU>(p, A, st); break;
    case EL_NORM_ADD_RELU: f32 ? launch_map_t<float, EL_NORM_ADD_RELU>(p, A, st) : launch_map_t<bf16_t, EL_NORM_ADD_RELU>(p, A, st); break;
    case EL_DX_RELU: f32 ? launch_map_t<float, EL_DX_RELU>(p, A, st) : launch_map_t<bf16_t, EL_DX_RELU>(p, A, st); break;
    default:        f32 ? launch_map_t<float, EL_SCALE>(p, A, st)  : launch_map_t<bf16_t, EL_SCALE>(p, A, st); break;
    }
    return launched();
}

// `pivot_x`: the activation tensor when the rows hold sums about the channel pivots
// (the plain-sum sweep), else null.
cgbn_status launch_combine(int mode, const Plan& p, char* ws, float* out0, float* out1, float* out2,
                           double* sh0, double* sh1, double eps, const void* pivot_x, hipStream_t st,
                           float* out3 = nullptr)
{
    CombineArgs A;
    std::memset(&A, 0, sizeof(A));
    A.part0 = reinterpret_cast<const float*>(ws + p.off_part0);
    A.part1 = reinterpret_cast<const float*>(ws + p.off_part1);
    A.sh0 = sh0; A.sh1 = sh1;
    A.out0 = out0; A.out1 = out1; A.out2 = out2; A.out3 = out3;
    A.M = p.M; A.eps = eps;
    A.shard_count = p.M / p.K;
    A.x = pivot_x;
    A.pivot_stride = pivot_x ? (p.layout == CGBN_NCHW ? p.HW : 1) : 0;
    A.is_bf16 = p.dtype == CGBN_BF16;
    A.C = p.C; A.rows = p.rows; A.K = p.K; A.rps = p.rps; A.G = p.G;
    if (p.layout == CGBN_NCHW) { A.cs = p.rows; A.rs = 1; } else { A.cs = 1; A.rs = p.C; }
    A.clear_word = reinterpret_cast<unsigned*>(ws + p.off_sync) + 1;
    // values per row partial: a chunk of a plane (the last chunk shorter), a whole plane, or a pixel run of a shard
    if (p.layout == CGBN_NCHW) { A.row_mod = p.sp; A.row_full = (p.wave_mode || p.tiny) ? p.HW : p.L; A.row_total = p.HW; }
    else {
        A.row_mod = p.pps; A.row_full = (long long)p.PL * p.group; A.row_total = p.spix * p.group;
    }
    dim3 block(kThreads);
    if (p.layout == CGBN_NHWC) {       // a row's channels side by side: 16 channels per workgroup
        constexpr int RL = kThreads / kCombineChannels;
        int G = 1;                     // row lanes per shard: as many as the shard count and a shard's rows allow
        while (2 * G * p.K <= RL && 2 * G <= p.rps) G <<= 1;
        A.G = G;
        dim3 grid((unsigned)((p.C + kCombineChannels - 1) / kCombineChannels));
        switch (mode) {
        case CM_MEAN:   hipLaunchKernelGGL((combine_rows_cl<CM_MEAN>), grid, block, 0, st, A); break;
        case CM_INVSTD: hipLaunchKernelGGL((combine_rows_cl<CM_INVSTD>), grid, block, 0, st, A); break;
        case CM_BWD:    hipLaunchKernelGGL((combine_rows_cl<CM_BWD>), grid, block, 0, st, A); break;
        case CM_SHARDS2: hipLaunchKernelGGL((combine_rows_cl<CM_SHARDS2>), grid, block, 0, st, A); break;
        case CM_MOMENTS: hipLaunchKernelGGL((combine_rows_cl<CM_MOMENTS>), grid, block, 0, st, A); break;
        default:        hipLaunchKernelGGL((combine_rows_cl<CM_SHARDS1>), grid, block, 0, st, A); break;
        }
        return launched();
    }
    dim3 grid((unsigned)((p.C + 3) / 4));
    switch (mode) {
    case CM_MEAN:   hipLaunchKernelGGL((combine_rows<CM_MEAN>), grid, block, 0, st, A); break;
    case CM_INVSTD: hipLaunchKernelGGL((combine_rows<CM_INVSTD>), grid, block, 0, st, A); break;
    case CM_BWD:    hipLaunchKernelGGL((combine_rows<CM_BWD>), grid, block, 0, st, A); break;
    case CM_SHARDS2: hipLaunchKernelGGL((combine_rows<CM_SHARDS2>), grid, block, 0, st, A); break;
    case CM_MOMENTS: hipLaunchKernelGGL((combine_rows<CM_MOMENTS>), grid, block, 0, st, A); break;
    default:        hipLaunchKernelGGL((combine_rows<CM_SHARDS1>), grid, block, 0, st, A); break;
    }
    return launched();
}

// ---- register-resident path ------------------------------------------------

// workgroups of `kernel` that are resident at once on the current device (cached per kernel and device)
template <typename KernelT> int resident_groups(KernelT kernel, int threads = kThreads)
{
    static std::mutex lock;
    static std::map<std::pair<const void*, int>, int> cache;
    int dev = 0, per_cu = 0, cus = 0;
    if (hipGetDevice(&dev) != hipSuccess) return 0;
    const std::pair<const void*, int> key(reinterpret_cast<const void*>(kernel), dev);
    std::lock_guard<std::mutex> hold(lock);
    auto it = cache.find(key);
    if (it != cache.end()) return it->second;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess) return 0;
    if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
    cache[key] = per_cu * cus;
    return per_cu * cus;
}

// Start-up stagger of the persistent grid.  All workgroups starting at once run in lock step: every
// channel in flight loads, hands over and writes out at the same time, so the memory system sees a
// read burst, a pause and a write burst per round, and a channel's units, competing with all the
// others, arrive spread out and wait for their last sibling.  Delaying the channel slots class by
// class interleaves those phases.  Measured over 28 launches of 1.3 to 43 rounds (rounds of 23 to
// 61 us): a spread of about 14 us between the first and the last class is at or near the best for
// every launch of at least 4 rounds (forward 2-6 % faster than starting at once, backward 0-6 %);
// spreads proportional to the round are worse at one end or the other, and launches of fewer rounds
// gain nothing or lose what the delay costs, since it is paid once per launch.
// `moved_bytes`: what the launch reads and writes.
void choose_stagger(const Tuning& T, const FusedPlan& f, long long groups, double moved_bytes, FusedArgs& A)
{
    A.stagger_ticks = 0;
    A.stagger_phases = 1;
    const long long slots = groups / f.U, rounds = f.total_units / groups;
    if (!T.stagger || f.U < 2 || slots < 2) return;
    double spread_us = (double)T.stagger_us;
    if (spread_us <= 0.0) {
        if (rounds < 4) return;
        const double round_us = moved_bytes / (double)f.total_units * (double)groups / 4.5e6;   // at 4.5 TB/s
        spread_us = 0.6 * round_us;                 // (short rounds: tiny units)
        if (spread_us > 14.0) spread_us = 14.0;
    }
    const long long phases = slots < T.stagger_phases ? slots : T.stagger_phases;
    A.stagger_phases = (unsigned)phases;
    A.stagger_ticks = (unsigned)(spread_us * 100.0 / (double)(phases - 1));     // 100 MHz clock
}

template <typename KernelT>
cgbn_status launch_fused_kernel(KernelT kernel, const Tuning& T, const FusedPlan& f, FusedArgs& A, int sync_words,
                                hipStream_t st, bool* taken, double moved_bytes)
{
    long long groups = resident_groups(kernel);
    if (T.fused_groups > 0 && T.fused_groups < groups) groups = T.fused_groups;
    if (groups > f.total_units) groups = f.total_units;
    *taken = false;
    if (groups < 1 || f.U > groups) return CGBN_OK;      // a channel's units must all be resident: other path
    // With few channels in flight, a grid that is not a whole number of channels leaves the
    // units of the straddling channel waiting a full round for their siblings: trim it.
    if (T.fused_groups == 0 && groups / f.U < 8) groups = groups / f.U * f.U;
    *taken = true;
    choose_stagger(T, f, groups, moved_bytes, A);
    if (f.U > 1) {      // a channel's only unit hands nothing over: no rows or counters to prepare
        long long want = (A.row_words + kThreads - 1) / kThreads;
        unsigned init_groups = (unsigned)(want < 1 ? 1 : (want > 2048 ? 2048 : want));
        hipLaunchKernelGGL(fused_init, dim3(init_groups), dim3(kThreads), 0, st, A.sync, sync_words,
                           reinterpret_cast<unsigned*>(A.part0), A.row_words);
    }
    if (f.U > 1 && T.cooperative) {
        // Units wait for sibling units, so the whole grid must be resident at once.  Alone on the device it
        // is (the grid is sized for that); a cooperative launch makes the runtime guarantee it also when
        // another such launch is in flight on a different stream, where two half-resident grids could
        // otherwise starve each other until their bounded waits give up.
        void* args[] = {static_cast<void*>(&A)};
        if (hipLaunchCooperativeKernel(reinterpret_cast<const void*>(kernel), dim3((unsigned)groups), dim3(kThreads),
                                       args, 0, st) != hipSuccess) {
            (void)hipGetLastError();
            return CGBN_ERR_HIP;
        }
        return CGBN_OK;
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)groups), dim3(kThreads), 0, st, A);
    return launched();
}

// ACT: 0 plain, 1 ReLU, 2 shortcut + ReLU (forward only)
template <typename T, bool FWD, int ACT>
cgbn_status launch_fused_t(const Tuning& knobs, const FusedPlan& f, FusedArgs& A, int sync_words, hipStream_t st, bool* taken,
                           double moved_bytes)
{
    *taken = false;
    if (f.edge) {
#define CGBN_FUSED_CASEE(LPPC_, BIG_)                                                                        \
        if (f.big == BIG_ && f.LPPC == LPPC_) {                                                              \
            if constexpr (FWD) return launch_fused_kernel(nchw_fused_forward<T, 16, LPPC_, ACT, BIG_, true>, knobs, f, A, sync_words, st, taken, moved_bytes); \
            else return launch_fused_kernel(nchw_fused_backward<T, 16, LPPC_, ACT, BIG_, true>, knobs, f, A, sync_words, st, taken, moved_bytes); \
        }
        if constexpr (FWD && ACT == 2) {
            CGBN_FUSED_EDGE_SHORTCUT(CGBN_FUSED_CASEE)
        } else if constexpr (FWD) {
            CGBN_FUSED_EDGE_FORWARD(CGBN_FUSED_CASEE)
        } else {
            CGBN_FUSED_EDGE_BACKWARD(CGBN_FUSED_CASEE)
        }
#undef CGBN_FUSED_CASEE
        return CGBN_OK;
    }
    if (f.big && f.LB == 16 && f.LPPC == 0) {
        if constexpr (FWD) return launch_fused_kernel(nchw_fused_forward<T, 16, 0, ACT, 1>, knobs, f, A, sync_words, st, taken, moved_bytes);
        else return launch_fused_kernel(nchw_fused_backward<T, 16, 0, ACT, 1>, knobs, f, A, sync_words, st, taken, moved_bytes);
    }
    if (f.big && f.LB == 16 && f.LPPC == -2) {
        if constexpr (FWD) return launch_fused_kernel(nchw_fused_forward<T, 16, -2, ACT, 1>, knobs, f, A, sync_words, st, taken, moved_bytes);
        else return launch_fused_kernel(nchw_fused_backward<T, 16, -2, ACT, 1>, knobs, f, A, sync_words, st, taken, moved_bytes);
    }
#define CGBN_FUSED_CASE1(LB_, LPPC_)                                                                         \
    if (f.big == 1 && f.LB == LB_ && f.LPPC == LPPC_) {                                                      \
        if constexpr (FWD) return launch_fused_kernel(nchw_fused_forward<T, LB_, LPPC_, ACT, 1>, knobs, f, A, sync_words, st, taken, moved_bytes); \
        else return launch_fused_kernel(nchw_fused_backward<T, LB_, LPPC_, ACT, 1>, knobs, f, A, sync_words, st, taken, moved_bytes); \
    }
    if constexpr (FWD) {
        CGBN_FUSED_WGP_FORWARD(CGBN_FUSED_CASE1)
    } else {
        CGBN_FUSED_WGP_BACKWARD(CGBN_FUSED_CASE1)
    }
#undef CGBN_FUSED_CASE1
#define CGBN_FUSED_CASE2(LB_, LPPC_)                                                                         \
    if constexpr (fused_built(std::is_same<T, float>::value, FWD, ACT, LB_, LPPC_))                                                      \
    if (f.big == 2 && f.LB == LB_ && f.LPPC == LPPC_) {                                                      \
        if constexpr (FWD) return launch_fused_kernel(nchw_fused_forward<T, LB_, LPPC_, ACT, 2>, knobs, f, A, sync_words, st, taken, moved_bytes); \
        else return launch_fused_kernel(nchw_fused_backward<T, LB_, LPPC_, ACT, 2>, knobs, f, A, sync_words, st, taken, moved_bytes); \
    }
    CGBN_FUSED_BIG_SMALL(CGBN_FUSED_CASE2)
#undef CGBN_FUSED_CASE2
#define CGBN_FUSED_CASE(LB_, LPPC_)                                                                          \
    if constexpr (fused_built(std::is_same<T, float>::value, FWD, ACT, LB_, LPPC_))                                                      \
    if (f.LB == LB_ && f.LPPC == LPPC_) {                                                                    \
        if constexpr (FWD) return launch_fused_kernel(nchw_fused_forward<T, LB_, LPPC_, ACT, 0>, knobs, f, A, sync_words, st, taken, moved_bytes); \
        else return launch_fused_kernel(nchw_fused_backward<T, LB_, LPPC_, ACT, 0>, knobs, f, A, sync_words, st, taken, moved_bytes); \
    }
    CGBN_FUSED_COMMON(CGBN_FUSED_CASE)
    if constexpr (FWD) {
        CGBN_FUSED_FORWARD_ONLY(CGBN_FUSED_CASE)
    } else {
        CGBN_FUSED_BACKWARD_ONLY(CGBN_FUSED_CASE)
    }
#undef CGBN_FUSED_CASE
    return CGBN_OK;
}

FusedArgs fused_args(const Plan& p, const FusedPlan& f, char* ws)
{
    FusedArgs A;
    std::memset(&A, 0, sizeof(A));
    A.part0 = reinterpret_cast<float*>(ws + p.off_part0);
    A.part1 = reinterpret_cast<float*>(ws + p.off_part1);
    A.sh0 = reinterpret_cast<double*>(ws + p.off_sh0);
    A.sh1 = reinterpret_cast<double*>(ws + p.off_sh1);
    A.sync = reinterpret_cast<unsigned*>(ws + p.off_sync);
    A.row_words = (long long)((p.off_sh0 - p.off_part0) / sizeof(float));   // part0 and part1 are adjacent
    A.total_units = f.total_units;
    A.M = p.M; A.inv_M_f64 = 1.0 / p.M; A.shard_count = p.M / p.K; A.inv_M = (float)(1.0 / p.M);
    A.N = p.N; A.C = p.C; A.HW = p.HW; A.rows = f.rows; A.K = p.K; A.rps = f.rps; A.G = f.G;
    A.U = f.U; A.tp = f.tp; A.TL = f.TL; A.LPP = f.LPP; A.IPU = f.IPU;
    A.nt = (int)p.t.nt_store;
    A.spin_limit = (unsigned)p.t.spin_limit;
    A.wait_ticks = (unsigned long long)p.t.wait_us * 100ull;          // the wall clock counts at 100 MHz
    A.plane_stride = (unsigned)((long long)p.C * p.HW * p.eb);
#ifdef CGBN_TRACE
    A.trace = g_trace;
#endif
    return A;
}

SlabArgs slab_args(const Plan& p, const SlabPlan& s, char* ws)
{
    SlabArgs A;
    std::memset(&A, 0, sizeof(A));
    A.rows = reinterpret_cast<unsigned long long*>(ws + p.off_part0);
    A.sync = reinterpret_cast<unsigned*>(ws + p.off_sync);
    A.R = s.R; A.row_bytes = s.row_bytes;
    A.inv_M_f64 = 1.0 / p.M; A.inv_M = (float)(1.0 / p.M);
    A.vecs = s.vecs; A.cols = s.cols; A.ncols = s.cols * (s.vb / p.eb); A.rpp = s.rpp;
    A.cpc = s.cpc; A.nch = s.nch; A.tpc = s.tpc; A.rch = A.ncols / s.cpc;
    A.C = p.C; A.slabs = s.slabs; A.U = s.U; A.rpu = s.rpu; A.total_units = (int)s.total_units;
    A.G = s.U < kWave ? ceil_pow2(s.U) : kWave;
    A.pivot_stride = p.layout == CGBN_NCHW ? p.HW : 1;
    A.nt = (int)p.t.nt_store && s.U > 1;
    A.spin_limit = (unsigned)p.t.spin_limit;
    A.bitmap_words = (unsigned)((s.U + 31) / 32);
    A.neighbours = s.shared;
    A.cpc_magic = (unsigned)(((1ULL << 32) + s.cpc - 1) / s.cpc);     // (not used for one column per channel)
    return A;
}

template <typename KernelT>
cgbn_status launch_slab_kernel(KernelT kernel, const Plan& p, const SlabPlan& s, SlabArgs A, hipStream_t st)
{
    long long groups = s.total_units;
    if (s.U > 1) {
        const long long resident = resident_groups(kernel, kSlabThreads);
        if (resident < 1) return CGBN_ERR_HIP;
        if (groups > resident) groups = resident;
        if (p.t.fused_groups > 0 && p.t.fused_groups < groups) groups = p.t.fused_groups > s.U ? p.t.fused_groups : s.U;
        // whole slabs only: the units of a straddling slab would wait a round for their siblings
        if (groups > s.U && groups < s.total_units) groups = groups / s.U * s.U;
        A.inflight = (int)(groups / s.U < s.slabs ? groups / s.U : s.slabs);
        if (groups < s.total_units) {
            const int polling = ((A.rch + s.U - 1) / s.U * A.G + kWave - 1) / kWave;      // wavefronts with channels to add up
            A.prefetch = polling < kSlabWaves ? polling : 0;
            A.ahead = A.inflight == 1 ? 1 : 2;           // see SlabAhead
            A.stagger = A.inflight == 2 ? 600u : (A.inflight == 3 || A.inflight == 4 ? 250u : 0u);      // see slab_stagger
        }
        const long long words = 2 * slab_row_words(s);
        long long want = (words + kThreads - 1) / kThreads;
        const unsigned init_groups = (unsigned)(want < 1 ? 1 : (want > 2048 ? 2048 : want));
        hipLaunchKernelGGL(fused_init, dim3(init_groups), dim3(kThreads), 0, st, A.sync, kSyncHeader + 4 * p.C,
                           reinterpret_cast<unsigned*>(A.rows), words);
    }
    hipLaunchKernelGGL(kernel, dim3((unsigned)groups), dim3(kSlabThreads), 0, st, A);
    return launched();
}

template <typename T, bool FWD, int ACT>
cgbn_status launch_slab_t(const Plan& p, const SlabPlan& s, const SlabArgs& A, hipStream_t st)
{
    if (s.vb == 8) {
#define CGBN_SLAB_CASE(P_)                                                                                      \
        if (s.P == P_) {                                                                                        \
            if constexpr (FWD) return launch_slab_kernel(slab_forward<T, ACT, P_, true, false, 8>, p, s, A, st); \
            else return launch_slab_kernel(slab_backward<T, ACT, P_, true, false, 8>, p, s, A, st);             \
        }
        CGBN_SLAB_NARROW_P(CGBN_SLAB_CASE)
#undef CGBN_SLAB_CASE
        return CGBN_ERR_HIP;
    }
    constexpr int dense = FWD ? kSlabDenseForward : kSlabDenseBackward;
    if constexpr (!FWD || ACT != 2)
        if (s.U > 1 && s.P == dense && s.total_units > compute_units()) {
            if constexpr (FWD) return launch_slab_kernel(slab_forward<T, ACT, dense, false, true>, p, s, A, st);
            else return launch_slab_kernel(slab_backward<T, ACT, dense, false, true>, p, s, A, st);
        }
#define CGBN_SLAB_CASE(P_, SOLO_)                                                                               \
    if (s.P == P_ && (s.U == 1) == SOLO_) {                                                                     \
        if constexpr (FWD) return launch_slab_kernel(slab_forward<T, ACT, P_, SOLO_, false>, p, s, A, st);      \
        else return launch_slab_kernel(slab_backward<T, ACT, P_, SOLO_, false>, p, s, A, st);                   \
    }
    if constexpr (FWD) { CGBN_SLAB_FORWARD_P(CGBN_SLAB_CASE) } else { CGBN_SLAB_BACKWARD_P(CGBN_SLAB_CASE) }
#undef CGBN_SLAB_CASE
    return CGBN_ERR_HIP;              // (no such variant: the plan takes its sizes from the same list)
}

FlatArgs flat_args(const Plan& p, char* ws)
{
    FlatArgs A;
    std::memset(&A, 0, sizeof(A));
    A.sync = reinterpret_cast<unsigned*>(ws + p.off_sync);
    A.inv_M_f64 = 1.0 / p.M; A.inv_M = (float)(1.0 / p.M);
    A.C = p.C;
    A.vecs = p.flat.vecs; A.total = p.flat.total;
    A.magic = A.vecs > 1 ? (unsigned)(((1ULL << 32) + A.vecs - 1) / A.vecs) : 0u;
    A.plane_bytes = (unsigned)(p.HW * p.eb); A.image_bytes = (unsigned)((long long)p.C * p.HW * p.eb);
    return A;
}

template <typename T, bool FWD, int ACT> cgbn_status launch_flat_t(const Plan& p, const FlatArgs& A, hipStream_t st)
{
    const FlatPlan& f = p.flat;
    const dim3 grid((unsigned)(f.waves == 1 ? (p.C + 3) / 4 : p.C)), block((unsigned)flat_threads(f.waves));
#define CGBN_FLAT_CASE(LB_, S_, WAVES_)                                                                         \
    if (f.LB == LB_ && f.S == S_ && f.waves == WAVES_) {                                                        \
        if constexpr (FWD) hipLaunchKernelGGL((flat_forward<T, LB_, S_, WAVES_, ACT>), grid, block, 0, st, A);  \
        else hipLaunchKernelGGL((flat_backward<T, LB_, S_, WAVES_, ACT>), grid, block, 0, st, A);               \
        return launched();                                                                                      \
    }
#define CGBN_FLAT_CASE1(LB_, S_) CGBN_FLAT_CASE(LB_, S_, 1)
#define CGBN_FLAT_CASE4(LB_, S_) CGBN_FLAT_CASE(LB_, S_, 4)
#define CGBN_FLAT_CASE16(LB_, S_) CGBN_FLAT_CASE(LB_, S_, 16)
    CGBN_FLAT_ONE(CGBN_FLAT_CASE1) CGBN_FLAT_FOUR(CGBN_FLAT_CASE4) CGBN_FLAT_SIXTEEN(CGBN_FLAT_CASE16)
    if constexpr (FWD) { CGBN_FLAT_FOUR_FORWARD(CGBN_FLAT_CASE4) }
    if constexpr (!std::is_same<T, float>::value) { CGBN_FLAT_BF16(CGBN_FLAT_CASE1) CGBN_FLAT_BF16(CGBN_FLAT_CASE4) CGBN_FLAT_BF16(CGBN_FLAT_CASE16) }
#undef CGBN_FLAT_CASE
#undef CGBN_FLAT_CASE1
#undef CGBN_FLAT_CASE4
#undef CGBN_FLAT_CASE16
    return CGBN_ERR_HIP;              // (no such variant: the plan takes its sizes from the same list)
}

bool eps_ok(float eps) { return std::isfinite(eps) && eps > 0.f; }

#define CGBN_TRY(expr) do { cgbn_status s_ = (expr); if (s_ != CGBN_OK) return s_; } while (0)

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================

extern "C" {

size_t cgbn_workspace_bytes(int N, int C, int H, int W, cgbn_layout layout, cgbn_dtype dtype, int K)
{
    const KeptPlan* k;
    if (plan_of(N, C, H, W, (int)layout, (int)dtype, K, &k) != CGBN_OK) return 0;
    return k->p.bytes;
}

size_t cgbn_workspace_error_offset(int N, int C, int H, int W, cgbn_layout layout, cgbn_dtype dtype, int K)
{
    Plan p;
    if (make_plan(tuning_now(), N, C, H, W, (int)layout, (int)dtype, K, &p) != CGBN_OK) return (size_t)-1;
    return kErrorWordOffset;
}

cgbn_status cgbn_shard_sum(const void* x, int N, int C, int H, int W, cgbn_layout layout, int K,
                           cgbn_dtype dtype, double* s, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !s) return CGBN_ERR_NULL;
    Plan p;
    CGBN_TRY(make_plan(tuning_now(), N, C, H, W, (int)layout, (int)dtype, K, &p));
    if (!aligned16(x)) return CGBN_ERR_ALIGN;
    CGBN_TRY(check_ws(p, workspace, workspace_bytes));
    char* ws = static_cast<char*>(workspace);
    hipStream_t st = static_cast<hipStream_t>(stream);
    SweepArgs A = sweep_args(p);
    A.x = x;
    A.part0 = reinterpret_cast<float*>(ws + p.off_part0);
    CGBN_TRY(launch_reduce(OP_SUM, p, A, st));
    return launch_combine(CM_SHARDS1, p, ws, nullptr, nullptr, nullptr, s, nullptr, 0.0, x, st);
}

cgbn_status cgbn_reduce_mean(const double* s, int K, int C, long long M, float* mean, float* mean_lo, void* stream)
{
    if (!s || !mean) return CGBN_ERR_NULL;
    if (C < 1 || M < 1) return CGBN_ERR_SHAPE;
    if (K < 1) return CGBN_ERR_SHARD;
    dim3 grid((unsigned)((C + kThreads - 1) / kThreads)), block(kThreads);
    hipLaunchKernelGGL((combine_shards<CM_MEAN>), grid, block, 0, static_cast<hipStream_t>(stream),
                       s, (const double*)nullptr, K, C, (double)M, 0.0, mean, mean_lo);
    return launched();
}

cgbn_status cgbn_shard_sqdev(const void* x, int N, int C, int H, int W, cgbn_layout layout, int K,
                             cgbn_dtype dtype, const float* mean, const float* mean_lo, double* v,
                             void* workspace, size_t workspace_bytes, void* stream)
{
    if (!x || !mean || !v) return CGBN_ERR_NULL;
    Plan p;
    CGBN_TRY(make_plan(tuning_now(), N, C, H, W, (int)layout, (int)dtype, K, &p));
    if (!aligned16(x)) return CGBN_ERR_ALIGN;
    CGBN_TRY(check_ws(p, workspace, workspace_bytes));
    char* ws = static_cast<char*>(workspace);
    hipStream_t st = static_cast<hipStream_t>(stream);
    SweepArgs A = sweep_args(p);
    A.x = x; A.mean = mean; A.mean_lo = mean_lo;
    A.part0 = reinterpret_cast<float*>(ws + p.off_part0);
    CGBN_TRY(launch_reduce(OP_SQDEV, p, A, st));
    return launch_combine(CM_SHARDS1, p, ws, nullptr, nullptr, nullptr, v, nullptr, 0.0, nullptr, st);
}

cgbn_status cgbn_reduce_invstd(const double* v, int K, int C, long long M, float eps, float* invstd, void* stream)
{
    if (!v || !invstd) return CGBN_ERR_NULL;
    if (C < 1 || M < 1) return CGBN_ERR_SHAPE;
    if (K < 1) return CGBN_ERR_SHARD;
    if (!eps_ok(eps)) return CGBN_ERR_EPS;
    dim3 grid((unsigned)((C + kThreads - 1) / kThreads)), block(kThreads);
    hipLaunchKernelGGL((combine_shards<CM_INVSTD>), grid, block, 0, static_cast<hipStream_t>(stream),
                       v, (const double*)nullptr, K, C, (double)M, (double)eps, invstd, (float*)nullptr);
    return launched();
}

cgbn_status cgbn_normalize(const void* x, int N, int C, int H, int W, cgbn_layout layout, cgbn_dtype dtype,
                           const float* mean, const float* mean_lo, const float* invstd,
                           const float* gamma, const float* beta, void* y, void* stream)
{
    if (!x || !mean || !invstd || !gamma || !beta || !y) return CGBN_ERR_NULL;
    const KeptPlan* k;
    CGBN_TRY(plan_of(N, C, H, W, (int)layout, (int)dtype, 1, &k));
    const Plan& p = k->map(1);
    if (!aligned16(x) || !aligned16(y)) return CGBN_ERR_ALIGN;
    SweepArgs A = sweep_args(p);
    A.x = x; A.out = y; A.mean = mean; A.mean_lo = mean_lo; A.invstd = invstd; A.gamma = gamma; A.beta = beta;
    return launch_map(EL_NORM, p, A, static_cast<hipStream_t>(stream));
}

cgbn_status cgbn_backward_shard_sums(const void* dy, const void* x, int N, int C, int H, int W,
                                     cgbn_layout layout, int K, cgbn_dtype dtype,
                                     const float* mean, const float* mean_lo, const float* invstd,
                                     double* a, double* b, void* workspace, size_t workspace_bytes, void* stream)
{
    if (!dy || !x || !mean || !invstd || !a || !b) return CGBN_ERR_NULL;
    Plan p;
    CGBN_TRY(make_plan(tuning_now(), N, C, H, W, (int)layout, (int)dtype, K, &p));
    if (!aligned16(x) || !aligned16(dy)) return CGBN_ERR_ALIGN;
    CGBN_TRY(check_ws(p, workspace, workspace_bytes));
    char* ws = static_cast<char*>(workspace);
    hipStream_t st = static_cast<hipStream_t>(stream);
    SweepArgs A = sweep_args(p);
    A.x = x; A.dy = dy; A.mean = mean; A.mean_lo = mean_lo; A.invstd = invstd;
    A.part0 = reinterpret_cast<float*>(ws + p.off_part0);
    A.part1 = reinterpret_cast<float*>(ws + p.off_part1);
    CGBN_TRY(launch_reduce(OP_BWD, p, A, st));
    return launch_combine(CM_SHARDS2, p, ws, nullptr, nullptr, nullptr, a, b, 0.0, nullptr, st);
}

cgbn_status cgbn_backward_reduce(const double* a, const double* b, int K, int C,
                                 float* dbeta, float* dgamma, void* stream)
{
    if (!a || !b || !dbeta || !dgamma) return CGBN_ERR_NULL;
    if (C < 1) return CGBN_ERR_SHAPE;
    if (K < 1) return CGBN_ERR_SHARD;
    dim3 grid((unsigned)((C + kThreads - 1) / kThreads)), block(kThreads);
    hipLaunchKernelGGL((combine_shards<CM_BWD>), grid, block, 0, static_cast<hipStream_t>(stream),
                       a, b, K, C, 1.0, 0.0, dbeta, dgamma);
    return launched();
}

cgbn_status cgbn_backward_dx(const void* dy, const void* x, int N, int C, int H, int W,
                             cgbn_layout layout, cgbn_dtype dtype,
                             const float* mean, const float* mean_lo, const float* invstd,
                             const float* gamma, const float* dgamma, const float* dbeta,
                             void* dx, void* stream)
{
    if (!dy || !x || !mean || !invstd || !gamma || !dgamma || !dbeta || !dx) return CGBN_ERR_NULL;
    const KeptPlan* k;
    CGBN_TRY(plan_of(N, C, H, W, (int)layout, (int)dtype, 1, &k));
    const Plan& p = k->map(2);
    if (!aligned16(x) || !aligned16(dy) || !aligned16(dx)) return CGBN_ERR_ALIGN;
    SweepArgs A = sweep_args(p);
    A.x = x; A.dy = dy; A.out = dx; A.mean = mean; A.mean_lo = mean_lo; A.invstd = invstd;
    A.gamma = gamma; A.dgamma = dgamma; A.dbeta = dbeta;
    return launch_map(EL_DX, p, A, static_cast<hipStream_t>(stream));
}

cgbn_status cgbn_frozen_forward(const void* x, int N, int C, int H, int W, cgbn_layout layout, cgbn_dtype dtype,
                                const float* fixed_mean, const float* fixed_var,
                                const float* gamma, const float* beta, float eps, void* y, void* stream)
{
    if (!x || !fixed_mean || !fixed_var || !gamma || !beta || !y) return CGBN_ERR_NULL;
    const KeptPlan* k;
    CGBN_TRY(plan_of(N, C, H, W, (int)layout, (int)dtype, 1, &k));
    const Plan& p = k->map(1);
    if (!eps_ok(eps)) return CGBN_ERR_EPS;
    if (!aligned16(x) || !aligned16(y)) return CGBN_ERR_ALIGN;
    SweepArgs A = sweep_args(p);
    A.x = x; A.out = y; A.mean = fixed_mean; A.invstd = fixed_var; A.gamma = gamma; A.beta = beta; A.eps = eps;
    return launch_map(EL_FROZEN, p, A, static_cast<hipStream_t>(stream));
}

cgbn_status cgbn_frozen_backward(const void* dy, int N, int C, int H, int W, cgbn_layout layout, cgbn_dtype dtype,
                                 const float* fixed_var, const float* gamma, float eps, void* dx, void* stream)
{
    if (!dy || !fixed_var || !gamma || !dx) return CGBN_ERR_NULL;
    const KeptPlan* k;
    CGBN_TRY(plan_of(N, C, H, W, (int)layout, (int)dtype, 1, &k));
    const Plan& p = k->map(1);
    if (!eps_ok(eps)) return CGBN_ERR_EPS;
    if (!aligned16(dy) || !aligned16(dx)) return CGBN_ERR_ALIGN;
    SweepArgs A = sweep_args(p);
    A.x = dy; A.out = dx; A.invstd = fixed_var; A.gamma = gamma; A.eps = eps;
    return launch_map(EL_SCALE, p, A, static_cast<hipStream_t>(stream));
}

cgbn_status cgbn_update_running_stats(const float* mean, const float* mean_lo, const float* invstd, float eps,
                                      long long M, int C, float momentum, int unbiased,
                                      float* running_mean, float* running_var, void* stream)
{
    if (!mean || !invstd || !running_mean || !running_var) return CGBN_ERR_NULL;
    if (C < 1 || M < 1 || (unbiased && M < 2)) return CGBN_ERR_SHAPE;
    if (!eps_ok(eps)) return CGBN_ERR_EPS;
    if (!(momentum >= 0.f && momentum <= 1.f)) return CGBN_ERR_MOMENTUM;
    const double unbias = unbiased ? (double)M / (double)(M - 1) : 1.0;
    dim3 grid((unsigned)((C + kThreads - 1) / kThreads)), block(kThreads);
    hipLaunchKernelGGL(running_update, grid, block, 0, static_cast<hipStream_t>(stream),
                       mean, mean_lo, invstd, (double)eps, unbias, (double)momentum, running_mean, running_var, C);
    return launched();
}

}  // extern "C"

namespace {

// Algorithm 1, optionally followed by "+ shortcut" and a ReLU (relu == true).  `k`: the call's plan, if its caller has it already.
cgbn_status forward_impl(const void* x, const void* shortcut, bool relu, int N, int C, int H, int W,
                         cgbn_layout layout, int K, const float* gamma, const float* beta, float eps,
                         void* y, float* mean, float* invstd, cgbn_dtype dtype, float* mean_lo,
                         void* workspace, size_t workspace_bytes, void* stream, const KeptPlan* k = nullptr)
{
    if (!x || !gamma || !beta || !y || !mean || !invstd) return CGBN_ERR_NULL;
    if (!k) CGBN_TRY(plan_of(N, C, H, W, (int)layout, (int)dtype, K, &k));
    const Plan& p = k->p;
    if (!eps_ok(eps)) return CGBN_ERR_EPS;
    if (!aligned16(x) || !aligned16(y) || !aligned16(shortcut)) return CGBN_ERR_ALIGN;
    CGBN_TRY(check_ws(p, workspace, workspace_bytes));
    char* ws = static_cast<char*>(workspace);
    hipStream_t st = static_cast<hipStream_t>(stream);
    float* part0 = reinterpret_cast<float*>(ws + p.off_part0);
    double* sh0 = reinterpret_cast<double*>(ws + p.off_sh0);
    float* mlo = reinterpret_cast<float*>(ws + p.off_mlo);
    const int rev = (int)p.t.reverse;

    const SlabPlan& wide = shortcut ? p.sfs : p.xf.ok ? p.xf : p.sf;
    const bool slab = p.t.fused && p.t.one_sweep_stats && wide.ok;
    if (p.t.fused && p.flats[shortcut != nullptr] && !(slab && wide.first)) {
        FlatArgs F = flat_args(p, ws);
        F.x = x; F.dy = shortcut; F.out = y; F.gamma = gamma; F.beta = beta; F.eps = (double)eps;
        F.mean = mean; F.mean_lo = mean_lo; F.invstd = invstd;
        g_last_forward_fused = g_last_forward_flat = 1;
        g_last_forward_slab = g_last_forward_edge = 0;
        const bool f32 = p.dtype == CGBN_F32;
        if (relu && shortcut) return f32 ? launch_flat_t<float, true, 2>(p, F, st) : launch_flat_t<bf16_t, true, 2>(p, F, st);
        if (relu) return f32 ? launch_flat_t<float, true, 1>(p, F, st) : launch_flat_t<bf16_t, true, 1>(p, F, st);
        return f32 ? launch_flat_t<float, true, 0>(p, F, st) : launch_flat_t<bf16_t, true, 0>(p, F, st);
    }
    g_last_forward_flat = g_last_forward_edge = 0;
    for (const FusedPlan* f : {&p.ef, &p.ff}) {
        if (!p.t.fused || !f->ok || (f == &p.ef && !p.edges[shortcut != nullptr]) || (slab && wide.first)) continue;
        FusedArgs F = fused_args(p, *f, ws);
        F.x = x; F.out = y; F.gamma = gamma; F.beta = beta; F.eps = (double)eps; F.aux = shortcut;
        F.mean = mean; F.mean_lo = mlo; F.mean_lo_user = mean_lo; F.invstd = invstd;
        bool taken = false;
        const int sync_words = kSyncHeader + 4 * p.C;
        const bool f32 = p.dtype == CGBN_F32;
        const double moved = (double)p.S * p.eb * (shortcut ? 3.0 : 2.0);
        cgbn_status st_ = relu && shortcut ? (f32 ? launch_fused_t<float, true, 2>(p.t, *f, F, sync_words, st, &taken, moved)
                                                  : launch_fused_t<bf16_t, true, 2>(p.t, *f, F, sync_words, st, &taken, moved))
                        : relu ? (f32 ? launch_fused_t<float, true, 1>(p.t, *f, F, sync_words, st, &taken, moved)
                                      : launch_fused_t<bf16_t, true, 1>(p.t, *f, F, sync_words, st, &taken, moved))
                               : (f32 ? launch_fused_t<float, true, 0>(p.t, *f, F, sync_words, st, &taken, moved)
                                      : launch_fused_t<bf16_t, true, 0>(p.t, *f, F, sync_words, st, &taken, moved));
        g_last_forward_fused = taken;
        g_last_forward_edge = taken && f->edge;
        if (taken) g_last_forward_slab = 0;
        if (taken || st_ != CGBN_OK) return st_;
    }
    g_last_forward_fused = 0;

    g_last_forward_slab = 0;
    if (slab) {
        const SlabPlan& narrow = shortcut ? p.nfs : p.nf;
        const SlabPlan& sp = narrow.ok ? narrow : wide;
        g_last_forward_slab = sp.vb;
        SlabArgs F = slab_args(p, sp, ws);
        F.x = x; F.dy = shortcut; F.out = y; F.gamma = gamma; F.beta = beta; F.eps = (double)eps;
        F.mean = mean; F.mean_lo = mean_lo; F.invstd = invstd;
        const bool f32 = p.dtype == CGBN_F32;
        if (relu && shortcut) return f32 ? launch_slab_t<float, true, 2>(p, sp, F, st) : launch_slab_t<bf16_t, true, 2>(p, sp, F, st);
        if (relu) return f32 ? launch_slab_t<float, true, 1>(p, sp, F, st) : launch_slab_t<bf16_t, true, 1>(p, sp, F, st);
        return f32 ? launch_slab_t<float, true, 0>(p, sp, F, st) : launch_slab_t<bf16_t, true, 0>(p, sp, F, st);
    }

    const Plan &q = k->sums(false), &m = k->map(shortcut ? 2 : 1);
    SweepArgs A = sweep_args(q);
    A.x = x; A.part0 = part0;
    if (p.t.one_sweep_stats) {
        // Steps 1-10 from ONE sweep over x: every row partial is (sum about the pivot, M2 about the row's own
        // mean); the combine step adds the sums (steps 4-5) and turns the M2s into the squared deviations from
        // the pooled mean by the pairwise update M2 + M2' + (mean' - mean)^2 n n'/(n + n') (steps 6-10: the same
        // number, term for term, as summing (x - mean)^2 directly).  Then step 11: 3 sweeps of the tensor instead of 4.
        A.part1 = reinterpret_cast<float*>(ws + p.off_part1);
        CGBN_TRY(launch_reduce(OP_MOMENTS, q, A, st));
        CGBN_TRY(launch_combine(CM_MOMENTS, q, ws, mean, mlo, mean_lo, nullptr, nullptr, (double)eps, x, st, invstd));
        A = sweep_args(m);
        A.x = x; A.mean = mean; A.mean_lo = mlo; A.invstd = invstd; A.gamma = gamma; A.beta = beta; A.out = y;
        A.reverse = rev; A.dy = shortcut;
        return launch_map(!relu ? EL_NORM : shortcut ? EL_NORM_ADD_RELU : EL_NORM_RELU, m, A, st);
    }
    // steps 1-3 then 4-5
    CGBN_TRY(launch_reduce(OP_SUM, q, A, st));
    CGBN_TRY(launch_combine(CM_MEAN, q, ws, mean, mlo, mean_lo, sh0, nullptr, 0.0, x, st));
    // steps 6-8 then 9-10
    A.mean = mean; A.mean_lo = mlo; A.reverse = rev;
    CGBN_TRY(launch_reduce(OP_SQDEV, q, A, st));
    CGBN_TRY(launch_combine(CM_INVSTD, q, ws, invstd, nullptr, nullptr, sh0, nullptr, (double)eps, nullptr, st));
    // step 11
    A = sweep_args(m);
    A.x = x; A.mean = mean; A.mean_lo = mlo; A.invstd = invstd; A.gamma = gamma; A.beta = beta; A.out = y;
    A.dy = shortcut;
    return launch_map(!relu ? EL_NORM : shortcut ? EL_NORM_ADD_RELU : EL_NORM_RELU, m, A, st);
}

// The backward; with `y` (the stored output of the ReLU variant) dy is first masked by y > 0
// and `dshortcut`, if not null, receives the masked dy.
cgbn_status backward_impl(const void* dy, const void* y, const void* x, const float* mean, const float* invstd,
                          const float* gamma, void* dx, void* dshortcut, float* dgamma, float* dbeta,
                          int N, int C, int H, int W, cgbn_layout layout, int K,
                          cgbn_dtype dtype, const float* mean_lo,
                          void* workspace, size_t workspace_bytes, void* stream)
{
    if (!dy || !x || !mean || !invstd || !gamma || !dx || !dgamma || !dbeta) return CGBN_ERR_NULL;
    const bool relu = y != nullptr;
    const KeptPlan* k;
    CGBN_TRY(plan_of(N, C, H, W, (int)layout, (int)dtype, K, &k));
    const Plan& p = k->p;
    if (!aligned16(x) || !aligned16(dy) || !aligned16(dx) || !aligned16(y) || !aligned16(dshortcut)) return CGBN_ERR_ALIGN;
    if (dshortcut && dshortcut == dx) return CGBN_ERR_ALIAS;
    CGBN_TRY(check_ws(p, workspace, workspace_bytes));
    char* ws = static_cast<char*>(workspace);
    hipStream_t st = static_cast<hipStream_t>(stream);
    const int rev = (int)p.t.reverse;

    const SlabPlan& wide = relu ? (p.xbm.ok ? p.xbm : p.sbm) : p.xb.ok ? p.xb : p.sb;
    const bool slab = p.t.fused && wide.ok;
    if (p.t.fused && p.flats[relu ? 3 : 2] && !(slab && wide.first)) {
        FlatArgs F = flat_args(p, ws);
        F.x = x; F.dy = dy; F.aux = y; F.out = dx; F.out2 = dshortcut; F.gamma = gamma;
        F.mean = const_cast<float*>(mean); F.mean_lo = const_cast<float*>(mean_lo); F.invstd = const_cast<float*>(invstd);
        F.dgamma = dgamma; F.dbeta = dbeta;
        g_last_backward_fused = g_last_backward_flat = 1;
        g_last_backward_slab = g_last_backward_edge = 0;
        const bool f32 = p.dtype == CGBN_F32;
        if (relu) return f32 ? launch_flat_t<float, false, 1>(p, F, st) : launch_flat_t<bf16_t, false, 1>(p, F, st);
        return f32 ? launch_flat_t<float, false, 0>(p, F, st) : launch_flat_t<bf16_t, false, 0>(p, F, st);
    }
    g_last_backward_flat = g_last_backward_edge = 0;
    for (const FusedPlan* f : {&p.ebw, &p.fb}) {
        if (!p.t.fused || !f->ok || (f == &p.ebw && !p.edges[relu ? 3 : 2]) || (slab && wide.first)) continue;
        FusedArgs F = fused_args(p, *f, ws);
        F.x = x; F.dy = dy; F.out = dx; F.gamma = gamma; F.aux = y; F.out2 = dshortcut;
        F.mean = const_cast<float*>(mean); F.mean_lo = const_cast<float*>(mean_lo);
        F.invstd = const_cast<float*>(invstd); F.dgamma = dgamma; F.dbeta = dbeta;
        bool taken = false;
        const int sync_words = kSyncHeader + 4 * p.C;
        const bool f32 = p.dtype == CGBN_F32;
        const double moved = (double)p.S * p.eb * (3.0 + (relu ? 1.0 : 0.0) + (dshortcut ? 1.0 : 0.0));
        cgbn_status st_ = relu ? (f32 ? launch_fused_t<float, false, 1>(p.t, *f, F, sync_words, st, &taken, moved)
                                      : launch_fused_t<bf16_t, false, 1>(p.t, *f, F, sync_words, st, &taken, moved))
                               : (f32 ? launch_fused_t<float, false, 0>(p.t, *f, F, sync_words, st, &taken, moved)
                                      : launch_fused_t<bf16_t, false, 0>(p.t, *f, F, sync_words, st, &taken, moved));
        g_last_backward_fused = taken;
        g_last_backward_edge = taken && f->edge;
        if (taken) g_last_backward_slab = 0;
        if (taken || st_ != CGBN_OK) return st_;
    }
    g_last_backward_fused = 0;

    g_last_backward_slab = 0;
    if (slab) {
        const SlabPlan& narrow = relu ? p.nbm : p.nb;
        const SlabPlan& sp = narrow.ok ? narrow : wide;
        g_last_backward_slab = sp.vb;
        SlabArgs F = slab_args(p, sp, ws);
        F.x = x; F.dy = dy; F.aux = y; F.out = dx; F.out2 = dshortcut; F.gamma = gamma;
        F.mean = const_cast<float*>(mean); F.mean_lo = const_cast<float*>(mean_lo); F.invstd = const_cast<float*>(invstd);
        F.dgamma = dgamma; F.dbeta = dbeta;
        const bool f32 = p.dtype == CGBN_F32;
        if (relu) return f32 ? launch_slab_t<float, false, 1>(p, sp, F, st) : launch_slab_t<bf16_t, false, 1>(p, sp, F, st);
        return f32 ? launch_slab_t<float, false, 0>(p, sp, F, st) : launch_slab_t<bf16_t, false, 0>(p, sp, F, st);
    }

    const Plan &q = k->sums(true), &m = k->map(relu ? 3 : 2);
    SweepArgs A = sweep_args(q);
    A.x = x; A.dy = dy; A.mean = mean; A.mean_lo = mean_lo; A.invstd = invstd;
    A.part0 = reinterpret_cast<float*>(ws + p.off_part0);
    A.part1 = reinterpret_cast<float*>(ws + p.off_part1);
    A.reverse = rev;
    A.aux = y;
    CGBN_TRY(launch_reduce(relu ? OP_BWD_RELU : OP_BWD, q, A, st));
    CGBN_TRY(launch_combine(CM_BWD, q, ws, dbeta, dgamma, nullptr,
                            reinterpret_cast<double*>(ws + p.off_sh0), reinterpret_cast<double*>(ws + p.off_sh1),
                            0.0, nullptr, st));
    A = sweep_args(m);
    A.x = x; A.dy = dy; A.mean = mean; A.mean_lo = mean_lo; A.invstd = invstd;
    A.aux = y; A.out2 = dshortcut;
    A.gamma = gamma; A.dgamma = dgamma; A.dbeta = dbeta; A.out = dx;
    return launch_map(relu ? EL_DX_RELU : EL_DX, m, A, st);
}

}  // namespace

extern "C" {

cgbn_status cgbn_forward(const void* x, int N, int C, int H, int W, cgbn_layout layout, int K,
                         const float* gamma, const float* beta, float eps,
                         void* y, float* mean, float* invstd,
                         cgbn_dtype dtype, float* mean_lo,
                         void* workspace, size_t workspace_bytes, void* stream)
{
    return forward_impl(x, nullptr, false, N, C, H, W, layout, K, gamma, beta, eps, y, mean, invstd, dtype, mean_lo,
                        workspace, workspace_bytes, stream);
}

cgbn_status cgbn_forward_static(const void* x, int N, int C, int H, int W, cgbn_layout layout, int K,
                                const float* gamma, const float* beta, float eps,
                                void* y, float* mean, float* invstd,
                                cgbn_dtype dtype, float* mean_lo, void* stream)
{
    // every argument error is answered before the device is asked for its scratch; one plan, and with it one copy of the knobs, for the check
    // and the launches
    if (!x || !gamma || !beta || !y || !mean || !invstd) return CGBN_ERR_NULL;
    const KeptPlan* k;
    CGBN_TRY(plan_of(N, C, H, W, (int)layout, (int)dtype, K, &k));
    if (!eps_ok(eps)) return CGBN_ERR_EPS;
    if (!aligned16(x) || !aligned16(y)) return CGBN_ERR_ALIGN;
    if (k->p.bytes > (size_t)CGBN_STATIC_SCRATCH_BYTES) return CGBN_ERR_SCRATCH;
    void* ws = nullptr;
    CGBN_TRY(scratch_of_current_device(&ws));
    return forward_impl(x, nullptr, false, N, C, H, W, layout, K, gamma, beta, eps, y, mean, invstd, dtype, mean_lo,
                        ws, (size_t)CGBN_STATIC_SCRATCH_BYTES, stream, k);
}

cgbn_status cgbn_backward(const void* dy, const void* x, const float* mean, const float* invstd,
                          const float* gamma, void* dx, float* dgamma, float* dbeta,
                          int N, int C, int H, int W, cgbn_layout layout, int K,
                          cgbn_dtype dtype, const float* mean_lo,
                          void* workspace, size_t workspace_bytes, void* stream)
{
    return backward_impl(dy, nullptr, x, mean, invstd, gamma, dx, nullptr, dgamma, dbeta, N, C, H, W, layout, K,
                         dtype, mean_lo, workspace, workspace_bytes, stream);
}

cgbn_status cgbn_forward_relu(const void* x, const void* shortcut, int N, int C, int H, int W,
                              cgbn_layout layout, int K, const float* gamma, const float* beta, float eps,
                              void* y, float* mean, float* invstd, cgbn_dtype dtype, float* mean_lo,
                              void* workspace, size_t workspace_bytes, void* stream)
{
    return forward_impl(x, shortcut, true, N, C, H, W, layout, K, gamma, beta, eps, y, mean, invstd, dtype, mean_lo,
                        workspace, workspace_bytes, stream);
}

cgbn_status cgbn_backward_relu(const void* dy, const void* y, const void* x, const float* mean, const float* invstd,
                               const float* gamma, void* dx, void* dshortcut, float* dgamma, float* dbeta,
                               int N, int C, int H, int W, cgbn_layout layout, int K,
                               cgbn_dtype dtype, const float* mean_lo,
                               void* workspace, size_t workspace_bytes, void* stream)
{
    if (!y) return CGBN_ERR_NULL;
    return backward_impl(dy, y, x, mean, invstd, gamma, dx, dshortcut, dgamma, dbeta, N, C, H, W, layout, K,
                         dtype, mean_lo, workspace, workspace_bytes, stream);
}

cgbn_status cgbn_workspace_status(const void* workspace, int* gave_up, void* stream)
{
    if (!workspace || !gave_up) return CGBN_ERR_NULL;
    if (((uintptr_t)workspace & 255u) != 0) return CGBN_ERR_WORKSPACE;
    hipLaunchKernelGGL(error_word_to_flag, dim3(1), dim3(kWave), 0, static_cast<hipStream_t>(stream),
                       static_cast<const unsigned*>(workspace), gave_up);
    return launched();
}

const char* cgbn_status_string(cgbn_status status)
{
    switch (status) {
    case CGBN_OK: return "ok";
    case CGBN_ERR_NULL: return "a required pointer is NULL";
    case CGBN_ERR_SHAPE: return "a dimension is < 1 or the tensor is too large";
    case CGBN_ERR_SHARD: return "need 1 <= K <= N and N % K == 0";
    case CGBN_ERR_ENUM: return "layout or dtype out of range";
    case CGBN_ERR_EPS: return "eps must be finite and > 0";
    case CGBN_ERR_WORKSPACE: return "workspace is NULL, not 256-byte aligned or too small";
    case CGBN_ERR_ALIGN: return "activation tensors must be 16-byte aligned";
    case CGBN_ERR_HIP: return "the HIP runtime refused a launch";
    case CGBN_ERR_TUNING: return "unknown tuning key or value out of range";
    case CGBN_ERR_MOMENTUM: return "momentum outside [0, 1]";
    case CGBN_ERR_ALIAS: return "two outputs that must differ are the same buffer";
    case CGBN_ERR_SCRATCH: return "the problem needs more scratch than the library's static array holds";
    }
    return "unknown status";
}

static long long* tuning_slot(const char* key)
{
    if (!key) return nullptr;
    if (!std::strcmp(key, "chunk_bytes")) return &g_tune.chunk_bytes;
    if (!std::strcmp(key, "wave_plane_bytes")) return &g_tune.wave_plane_bytes;
    if (!std::strcmp(key, "tiny_planes")) return &g_tune.tiny_planes;
    if (!std::strcmp(key, "piece_bytes")) return &g_tune.piece_bytes;
    if (!std::strcmp(key, "map_piece_bytes")) return &g_tune.map_piece_bytes;
    if (!std::strcmp(key, "reverse")) return &g_tune.reverse;
    if (!std::strcmp(key, "nt_store")) return &g_tune.nt_store;
    if (!std::strcmp(key, "fused")) return &g_tune.fused;
    if (!std::strcmp(key, "spin_limit")) return &g_tune.spin_limit;
    if (!std::strcmp(key, "fused_groups")) return &g_tune.fused_groups;
    if (!std::strcmp(key, "one_sweep_stats")) return &g_tune.one_sweep_stats;
    if (!std::strcmp(key, "cooperative")) return &g_tune.cooperative;
    if (!std::strcmp(key, "big_lds")) return &g_tune.big_lds;
    if (!std::strcmp(key, "stagger")) return &g_tune.stagger;
    if (!std::strcmp(key, "stagger_us")) return &g_tune.stagger_us;
    if (!std::strcmp(key, "stagger_phases")) return &g_tune.stagger_phases;
    if (!std::strcmp(key, "wait_us")) return &g_tune.wait_us;
    if (!std::strcmp(key, "flat")) return &g_tune.flat;
    return nullptr;
}

cgbn_status cgbn_set_tuning(const char* key, long long value)
{
    long long* slot = tuning_slot(key);
    if (!slot) return CGBN_ERR_TUNING;
    if (slot == &g_tune.reverse || slot == &g_tune.nt_store || slot == &g_tune.fused || slot == &g_tune.one_sweep_stats ||
        slot == &g_tune.cooperative || slot == &g_tune.big_lds || slot == &g_tune.stagger || slot == &g_tune.tiny_planes || slot == &g_tune.flat) {
        if (value != 0 && value != 1) return CGBN_ERR_TUNING;
    } else if (slot == &g_tune.spin_limit) {
        if (value < 0 || value > 0xffffffffLL) return CGBN_ERR_TUNING;
    } else if (slot == &g_tune.stagger_us) {
        if (value < 0 || value > 1000) return CGBN_ERR_TUNING;
    } else if (slot == &g_tune.stagger_phases) {
        if (value < 2 || value > 64) return CGBN_ERR_TUNING;
    } else if (slot == &g_tune.wait_us) {
        if (value < 1 || value > 60000000LL) return CGBN_ERR_TUNING;
    } else if (slot == &g_tune.fused_groups) {
        if (value < 0 || value > (1LL << 20)) return CGBN_ERR_TUNING;
    } else if (slot == &g_tune.wave_plane_bytes) {
        if (value < 0 || value > (1LL << 20)) return CGBN_ERR_TUNING;
    } else if ((slot == &g_tune.piece_bytes || slot == &g_tune.map_piece_bytes) && value == 0) {
        // chosen per shape
    } else if (value < 4096 || value > (1LL << 26)) {
        return CGBN_ERR_TUNING;
    }
    std::lock_guard<std::mutex> hold(g_tune_lock);
    *slot = value;
    g_tune_version.fetch_add(1, std::memory_order_release);
    return CGBN_OK;
}

#ifdef CGBN_TRACE
// performance-work builds only: device buffer of 8 timestamps per unit
void cgbn_debug_set_trace(void* device_buffer) { g_trace = static_cast<unsigned long long*>(device_buffer); }
#endif

cgbn_status cgbn_calibration_copy(const void* src, void* dst, size_t bytes, void* stream)
{
    if (!src || !dst) return CGBN_ERR_NULL;
    if (bytes == 0 || bytes % 16 != 0 || bytes > ((size_t)1 << 40)) return CGBN_ERR_SHAPE;
    if (!aligned16(src) || !aligned16(dst)) return CGBN_ERR_ALIGN;
    const size_t nvec = bytes / 16, per_group = (size_t)kThreads * 8;
    hipLaunchKernelGGL(calibration_copy, dim3((unsigned)((nvec + per_group - 1) / per_group)), dim3(kThreads), 0,
                       static_cast<hipStream_t>(stream), static_cast<const u32x4*>(src), static_cast<u32x4*>(dst), nvec);
    return launched();
}

long long cgbn_plan_get(int N, int C, int H, int W, cgbn_layout layout, cgbn_dtype dtype, int K, const char* key)
{
    Plan p;
    if (!key || make_plan(tuning_now(), N, C, H, W, (int)layout, (int)dtype, K, &p) != CGBN_OK) return -1;
    const bool edge = !std::strncmp(key, "efwd_", 5) || !std::strncmp(key, "ebwd_", 5);
    const bool bwd = !std::strncmp(key + edge, "bwd_", 4);
    if (bwd || !std::strncmp(key + edge, "fwd_", 4)) {
        const FusedPlan& f = edge ? (bwd ? p.ebw : p.ef) : (bwd ? p.fb : p.ff);
        const char* k = key + edge + 4;
        if (!std::strcmp(k, "ok")) return f.ok;
        if (edge && !std::strcmp(k, "taken")) return p.edges[bwd ? 2 : 0];
        if (edge && !std::strcmp(k, "taken2")) return p.edges[bwd ? 3 : 1];
        if (!std::strcmp(k, "LB")) return f.LB;
        if (!std::strcmp(k, "LPPC")) return f.LPPC;
        if (!std::strcmp(k, "LPP")) return f.LPP;
        if (!std::strcmp(k, "IPU")) return f.IPU;
        if (!std::strcmp(k, "U")) return f.U;
        if (!std::strcmp(k, "tp")) return f.tp;
        if (!std::strcmp(k, "TL")) return f.TL;
        if (!std::strcmp(k, "rows")) return f.rows;
        if (!std::strcmp(k, "rps")) return f.rps;
        if (!std::strcmp(k, "G")) return f.G;
        if (!std::strcmp(k, "big")) return f.big;
        if (!std::strcmp(k, "total_units")) return f.total_units;
        // as the kernels form it: where the last plane of a unit that holds several begins
        if (!std::strcmp(k, "last_plane")) return f.LPPC == 0 ? 0 : (long long)cgbn_plane_offset((f.LPPC > 0 ? f.IPU : -f.LPPC) - 1, fused_args(p, f, nullptr).plane_stride);
        return -1;
    }
    if ((key[0] == 's' || key[0] == 'n' || key[0] == 'x') && (!std::strncmp(key + 1, "fwd_", 4) || !std::strncmp(key + 1, "bwd_", 4) ||
                                             !std::strncmp(key + 1, "fwds_", 5) || !std::strncmp(key + 1, "bwdm_", 5))) {
        const bool second = key[4] != '_', narrow = key[0] == 'n';
        if (key[0] == 'x' && key[1] == 'f' && second) return -1;          // (there is none for a forward with a shortcut)
        const SlabPlan& s = key[0] == 'x' ? (key[1] == 'b' ? (second ? p.xbm : p.xb) : p.xf) : key[1] == 'b' ? (second ? (narrow ? p.nbm : p.sbm) : (narrow ? p.nb : p.sb))
                                          : (second ? (narrow ? p.nfs : p.sfs) : (narrow ? p.nf : p.sf));
        const char* k = key + (second ? 6 : 5);
        if (!std::strcmp(k, "ok")) return s.ok;
        if (!std::strcmp(k, "first")) return s.first;
        if (!std::strcmp(k, "cols")) return s.cols;
        if (!std::strcmp(k, "vecs")) return s.vecs;
        if (!std::strcmp(k, "cpc")) return s.cpc;
        if (!std::strcmp(k, "nch")) return s.nch;
        if (!std::strcmp(k, "rpp")) return s.rpp;
        if (!std::strcmp(k, "tpc")) return s.tpc;
        if (!std::strcmp(k, "slabs")) return s.slabs;
        if (!std::strcmp(k, "U")) return s.U;
        if (!std::strcmp(k, "rpu")) return s.rpu;
        if (!std::strcmp(k, "P")) return s.P;
        if (!std::strcmp(k, "R")) return s.R;
        return -1;
    }
    if (!std::strncmp(key, "flat_", 5)) {
        const char* k = key + 5;
        if (!std::strcmp(k, "waves")) return p.flat.waves;
        if (!std::strcmp(k, "LB")) return p.flat.LB;
        if (!std::strcmp(k, "S")) return p.flat.S;
        if (!std::strcmp(k, "vecs")) return p.flat.vecs;
        if (!std::strcmp(k, "total")) return p.flat.total;
        if (!std::strcmp(k, "fwd")) return p.flats[0];
        if (!std::strcmp(k, "fwds")) return p.flats[1];
        if (!std::strcmp(k, "bwd")) return p.flats[2];
        if (!std::strcmp(k, "bwdm")) return p.flats[3];
        return -1;
    }
    if (!std::strcmp(key, "may_group")) return p.may_group;
    if (!std::strcmp(key, "group_sums")) return group_sums(p, false);
    if (!std::strcmp(key, "group_sums_dy")) return group_sums(p, true);
    if (!std::strcmp(key, "group_map")) return group_map(p, 1);
    if (!std::strcmp(key, "group_map2")) return group_map(p, 2);
    if (!std::strncmp(key, "grouped_", 8)) {
        const Plan q = grouped(p);
        const char* k = key + 8;
        if (!std::strcmp(k, "K")) return q.K;
        if (!std::strcmp(k, "cv")) return q.cv;
        if (!std::strcmp(k, "ctiles")) return q.ctiles;
        if (!std::strcmp(k, "rows")) return q.rows;
        if (!std::strcmp(k, "spix")) return q.spix;
        if (!std::strcmp(k, "PL")) return q.PL;
        if (!std::strcmp(k, "pps")) return q.pps;
        return -1;
    }
    if (!std::strcmp(key, "wave_mode")) return p.wave_mode;
    if (!std::strcmp(key, "tiny")) return p.tiny;
    if (!std::strcmp(key, "tg")) return p.tg;
    if (!std::strcmp(key, "L")) return p.L;
    if (!std::strcmp(key, "sp")) return p.sp;
    if (!std::strcmp(key, "vec")) return p.vec;
    if (!std::strcmp(key, "cv")) return p.cv;
    if (!std::strcmp(key, "TW")) return p.TW;
    if (!std::strcmp(key, "ctiles")) return p.ctiles;
    if (!std::strcmp(key, "rpp")) return p.rpp;
    if (!std::strcmp(key, "PL")) return p.PL;
    if (!std::strcmp(key, "pps")) return p.pps;
    if (!std::strcmp(key, "PLm")) return p.map[0].PL;
    if (!std::strcmp(key, "ppsm")) return p.map[0].pps;
    if (!std::strcmp(key, "PLm2")) return p.map[1].PL;
    if (!std::strcmp(key, "ppsm2")) return p.map[1].pps;
    if (!std::strcmp(key, "gridm2")) return p.map[1].grid;
    if (!std::strcmp(key, "single_consts")) return p.layout == CGBN_NHWC && p.eb == 4 && p.vec == 4 && single_consts(p);
    if (!std::strcmp(key, "PLm3")) return p.map[2].PL;
    if (!std::strcmp(key, "ppsm3")) return p.map[2].pps;
    if (!std::strcmp(key, "gridm3")) return p.map[2].grid;
    if (!std::strcmp(key, "rows")) return p.rows;
    if (!std::strcmp(key, "rps")) return p.rps;
    if (!std::strcmp(key, "G")) return p.G;
    if (!std::strcmp(key, "grid")) return p.grid;
    if (!std::strcmp(key, "gridm")) return p.map[0].grid;
    if (!std::strcmp(key, "part_bytes")) return (long long)(p.off_part1 - p.off_part0);
    if (!std::strcmp(key, "shard_bytes")) return (long long)(p.off_sh1 - p.off_sh0);
    return -1;
}

long long cgbn_get_tuning(const char* key)
{
    if (key && !std::strcmp(key, "last_forward_fused")) return g_last_forward_fused.load();
    if (key && !std::strcmp(key, "last_backward_fused")) return g_last_backward_fused.load();
    if (key && !std::strcmp(key, "last_forward_slab")) return g_last_forward_slab.load() != 0;
    if (key && !std::strcmp(key, "last_forward_slab_vector")) return g_last_forward_slab.load();
    if (key && !std::strcmp(key, "last_backward_slab")) return g_last_backward_slab.load() != 0;
    if (key && !std::strcmp(key, "last_backward_slab_vector")) return g_last_backward_slab.load();
    if (key && !std::strcmp(key, "last_forward_flat")) return g_last_forward_flat.load();
    if (key && !std::strcmp(key, "last_forward_edge")) return g_last_forward_edge.load();
    if (key && !std::strcmp(key, "last_backward_flat")) return g_last_backward_flat.load();
    if (key && !std::strcmp(key, "last_backward_edge")) return g_last_backward_edge.load();
    if (key && !std::strcmp(key, "plans_made")) return g_plans_made;
    long long* slot = tuning_slot(key);
    if (!slot) return -1;
    std::lock_guard<std::mutex> hold(g_tune_lock);
    return *slot;
}

}  // extern "C"
