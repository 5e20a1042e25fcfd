// Device code that the kernels' source files share, and the table entry of a recursion kernel.
#pragma once
#include "kernels.h"

namespace lfmmi {
namespace {

template <typename Real>
__device__ __forceinline__ Real wave_sum(Real v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, 64);
    return v;
}

__device__ __forceinline__ float wave_max(float v)
{
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) v = fmaxf(v, __shfl_xor(v, o, 64));
    return v;
}

// Element of an LDS array addressed by the record's index * 4 field.
template <typename Real>
__device__ __forceinline__ Real lds_at(const Real* base, uint32_t index4)
{
    return *reinterpret_cast<const Real*>(reinterpret_cast<const char*>(base) +
                                          index4 * (uint32_t)(sizeof(Real) / 4));
}

// Byte offset of a record's emission value inside a Y buffer: the upper half of
// its key. Plain rows: 4 * pdf. Rows replicated 32 times, so that lane l always
// reads bank l % 32 (conflict-free; small pdf counts only): 128 * pdf + 4 * (l % 32),
// which the upload writes into the device copy of lane l's records.
__device__ __forceinline__ uint32_t y_offset(uint32_t key) { return key >> 16; }

__device__ __forceinline__ float lds_f32(const float* base, uint32_t byte_off)
{
    return *reinterpret_cast<const float*>(reinterpret_cast<const char*>(base) + byte_off);
}

// Arc records on the device: the records of slots 2q and 2q + 1 of a lane lie side
// by side, {key, w, key, w}, pair q of lane l at [q * 64 + l] (a 16-byte load per
// lane streams from L2 at twice the rate of an 8-byte one); slices start at even
// slots. The per-arc leak factors are paired up the same way.
__device__ __forceinline__ const uint4* rec_pairs(const FbParams& p, const OrdDesc& od, const int lane)
{
    return reinterpret_cast<const uint4*>(p.g.recs) + (size_t)(od.rec_at >> 1) * 64 + lane;
}
__device__ __forceinline__ const float2* wb_pairs(const FbParams& p, const OrdDesc& od, const int lane)
{
    return reinterpret_cast<const float2*>(p.g.wb) + (size_t)(od.rec_at >> 1) * 64 + lane;
}
__device__ __forceinline__ uint2 rec_lo(const uint4 r) { return make_uint2(r.x, r.y); }
__device__ __forceinline__ uint2 rec_hi(const uint4 r) { return make_uint2(r.z, r.w); }

// The records of slots first .. first + NSLOT - 1 (`first` even) of this lane into keys and
// weights: all loads go out before any is waited for (one after the other they took 10 us of a
// launch with 24 slots). Slots from `count` on are empty.
template <int NSLOT>
__device__ __forceinline__ void load_records(const FbParams& p, const OrdDesc& od, const int lane,
                                             const int first, const int count, uint32_t (&key)[NSLOT],
                                             float (&w)[NSLOT])
{
    const uint4* recs = rec_pairs(p, od, lane);
    const int last = max((od.total_slots >> 1) - 1, 0);  // (a load past it fetches it again)
    uint4 r[NSLOT / 2];
#pragma unroll
    for (int q = 0; q < NSLOT / 2; ++q)
        r[q] = od.total_slots > 0 ? recs[(size_t)min((first >> 1) + q, last) * 64] : make_uint4(0, 0, 0, 0);
#pragma unroll
    for (int q = 0; q < NSLOT / 2; ++q) {
        const bool on0 = 2 * q < count, on1 = 2 * q + 1 < count;
        key[2 * q] = on0 ? r[q].x : 0u;
        w[2 * q] = on0 ? __uint_as_float(r[q].y) : 0.f;
        key[2 * q + 1] = on1 ? r[q].z : 0u;
        w[2 * q + 1] = on1 ? __uint_as_float(r[q].w) : 0.f;
    }
}

// ---------------------------------------------------------------------------
// Wave-level sums on the DPP cross-lane path (no LDS traffic).
// ---------------------------------------------------------------------------
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ float dpp_add(float v)
{
    // lanes of rows outside ROW_MASK, and lanes whose source is out of range, add 0
    const int moved =
        __builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, ROW_MASK, 0xf, false);
    return v + __int_as_float(moved);
}

// fp64: the two halves of the value travel separately
template <int CTRL, int ROW_MASK>
__device__ __forceinline__ double dpp_add(double v)
{
    const long long bits = __double_as_longlong(v);
    // (with every row written the old value is dead: bound_ctrl lets the compiler drop the
    // two moves that would zero it first)
    constexpr bool kAll = ROW_MASK == 0xf;
    const int lo = __builtin_amdgcn_update_dpp(0, (int)bits, CTRL, ROW_MASK, 0xf, kAll);
    const int hi = __builtin_amdgcn_update_dpp(0, (int)(bits >> 32), CTRL, ROW_MASK, 0xf, kAll);
    return v + __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// After this every lane holds the sum over its row of 16 lanes.
template <typename Real>
__device__ __forceinline__ Real row16_allsum(Real v)
{
    v = dpp_add<0xB1, 0xf>(v);   // quad_perm [1,0,3,2]
    v = dpp_add<0x4E, 0xf>(v);   // quad_perm [2,3,0,1]
    v = dpp_add<0x141, 0xf>(v);  // row_half_mirror
    v = dpp_add<0x140, 0xf>(v);  // row_mirror
    return v;
}

// The value lane `l` holds, as a wave-uniform value.
__device__ __forceinline__ float lane_value(float v, int l)
{
    return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), l));
}
__device__ __forceinline__ double lane_value(double v, int l)
{
    const long long bits = __double_as_longlong(v);
    const int lo = __builtin_amdgcn_readlane((int)bits, l);
    const int hi = __builtin_amdgcn_readlane((int)(bits >> 32), l);
    return __longlong_as_double(((long long)hi << 32) | (unsigned int)lo);
}

// v with lane L holding `value` (wave-uniform) instead. By the compiler's own intrinsic, not by
// inline assembly: a lane write that reads a scalar register two instructions or fewer behind
// the v_readlane that wrote it needs a wait, which the compiler puts in for its own only.
__device__ int writelane_i32(int value, int lane, int old) __asm("llvm.amdgcn.writelane.i32");
template <int L>
__device__ __forceinline__ int write_lane(const int v, const int value)
{
    return writelane_i32(value, L, v);
}

// Sum over the 64 lanes, returned as a wave-uniform value.
template <typename Real>
__device__ __forceinline__ Real wave_sum_uniform(Real v)
{
    v = row16_allsum(v);
    v = dpp_add<0x142, 0xa>(v);  // row_bcast:15 into rows 1 and 3
    v = dpp_add<0x143, 0xc>(v);  // row_bcast:31 into rows 2 and 3
    return lane_value(v, 63);
}

// Wave sums of a and b at once: a 32-lane swap puts a[l] + a[l + 32] in the lower
// half-wave and b[l] + b[l + 32] in the upper one, five DPP steps finish both.
// Lane 31 returns the sum of a, lane 63 the sum of b (other lanes: partial sums).
__device__ __forceinline__ float half_wave_sums(float a, float b)
{
    // lanes 0-31 of [0] keep a, lanes 32-63 of [0] take b's lanes 0-31; [1] the rest
    const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b),
                                                     false, false);
    float v = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    v = row16_allsum(v);
    return dpp_add<0x142, 0xf>(v);  // row_bcast:15: row 1 gets row 0's sum, row 3 row 2's
}
__device__ __forceinline__ double half_wave_sums(double a, double b)
{
    const long long ab = __double_as_longlong(a), bb = __double_as_longlong(b);
    const auto lo = __builtin_amdgcn_permlane32_swap((unsigned)ab, (unsigned)bb, false, false);
    const auto hi = __builtin_amdgcn_permlane32_swap((unsigned)(ab >> 32), (unsigned)(bb >> 32),
                                                     false, false);
    double v = __longlong_as_double(((long long)hi[0] << 32) | lo[0]) +
               __longlong_as_double(((long long)hi[1] << 32) | lo[1]);
    v = row16_allsum(v);
    return dpp_add<0x142, 0xf>(v);
}

// Lane 63 returns the sum over the wave (other lanes: partial sums).
template <typename Real>
__device__ __forceinline__ Real wave_sum_lane63(Real v)
{
    v = row16_allsum(v);
    v = dpp_add<0x142, 0xf>(v);     // row_bcast:15: rows 1 and 3 get the sums of 0 and 2
    return dpp_add<0x143, 0xf>(v);  // row_bcast:31: row 3 gets the sum of rows 0 and 1
}

// LDS access by absolute byte address (the kernel's dynamic LDS starts at 0: it
// declares no static LDS), so that the address register goes straight into the
// ds instruction and constant parts fold into its immediate offset.
typedef __attribute__((address_space(3))) float lds_float_t;
__device__ __forceinline__ float lds_ld(uint32_t addr)
{
    return *reinterpret_cast<const lds_float_t*>(static_cast<uintptr_t>(addr));
}
__device__ __forceinline__ void lds_st(uint32_t addr, float v)
{
    *reinterpret_cast<lds_float_t*>(static_cast<uintptr_t>(addr)) = v;
}
typedef __attribute__((address_space(3))) double lds_double_t;
__device__ __forceinline__ void lds_st(uint32_t addr, double v)
{
    *reinterpret_cast<lds_double_t*>(static_cast<uintptr_t>(addr)) = v;
}
template <typename Real>
__device__ __forceinline__ Real lds_ldr(uint32_t addr)
{
    if constexpr (sizeof(Real) == 8)
        return *reinterpret_cast<const lds_double_t*>(static_cast<uintptr_t>(addr));
    else
        return *reinterpret_cast<const lds_float_t*>(static_cast<uintptr_t>(addr));
}

// N: the largest power of two not above n (0 below the normal range, and nothing beyond 2^126,
// 2^1022 in fp64); inv: its inverse, without a test for totals that are zero or not finite:
// they leave log Z at -inf or NaN whatever the scale is, and the rows that follow at zero
// or not finite.
__device__ __forceinline__ void pow2_scale(const float n, float* N, float* inv)
{
    const uint32_t e = min(__float_as_uint(n) & 0x7f800000u, 0x7e800000u);
    *N = __uint_as_float(e);
    *inv = __uint_as_float(0x7f000000u - e);
}
__device__ __forceinline__ void pow2_scale(const double n, double* N, double* inv)
{
    const uint32_t hi = (uint32_t)((unsigned long long)__double_as_longlong(n) >> 32);
    const uint32_t e = min(hi & 0x7ff00000u, 0x7fd00000u);
    *N = __longlong_as_double((long long)((unsigned long long)e << 32));
    *inv = __longlong_as_double((long long)((unsigned long long)(0x7fe00000u - e) << 32));
}

// ---------------------------------------------------------------------------
// Scales of one sequence, once both of its recursions are done:
//   log Z_b = log(zfin) + sum_t log n_t (+ the frame maxima), and the factor that
//   turns ahat_{t-1} * w * e_t * bhat_t into an occupancy,
//   c_t = exp(A_{t-1} + B_t - log Z'),  A, B = prefix / suffix sums of log n,
// in fp64. Called by every thread of a workgroup (at most 256 of them work);
// scratch: 96 bytes of LDS nobody else uses.
// ---------------------------------------------------------------------------
// Largest difference (nats) between the alpha-side and the beta-side log Z of a
// sequence that counts as rounding: fp32 state vectors on the longest workloads
// here differ by a few 1e-5.
constexpr double kTotalsAgree = 1e-3;

// The prefix sums run over lanes first (shuffles), then over the waves' totals: one thread
// adding up 256 partial sums one after the other took 12 to 15 us at the end of every
// sequence. A thread keeps the logarithms of its first kKeep frames.
template <typename Real>
__device__ void scan_sequence(const FbParams& p, const int b, unsigned char* scratch_raw)
{
    constexpr int kKeep = 4;  // all of them up to 1,023 frames
    double* tot = reinterpret_cast<double*>(scratch_raw);  // [wave][3]
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int workers = min((int)blockDim.x, 256);
    const SeqDesc sd = p.seqs[b];
    const int T = sd.T;
    const int n = T + 1;
    const Real* na = static_cast<const Real*>(p.scal) + sd.scal_at;
    const Real* nb = static_cast<const Real*>(p.scal) + 2 * p.scal_total + sd.scal_at;
    Real* cfac = static_cast<Real*>(p.cfac) + sd.scal_at;
    const int chunk = (n + workers - 1) / workers;
    const bool work = tid < workers;
    const int i0 = work ? min(tid * chunk, n) : n, i1 = min(i0 + chunk, n);
    double la = 0.0, lb = 0.0, lm = 0.0;
    double ka[kKeep], kb[kKeep];
    if (work)
        for (int t = tid; t < T; t += workers) lm += (double)p.rowmax[(size_t)b * p.T + t];
#pragma unroll
    for (int q = 0; q < kKeep; ++q) {
        const bool on = i0 + q < i1;
        ka[q] = on ? log((double)na[i0 + q]) : 0.0;
        kb[q] = on ? log((double)nb[i0 + q]) : 0.0;
        la += ka[q];
        lb += kb[q];
    }
    for (int i = i0 + kKeep; i < i1; ++i) {
        la += log((double)na[i]);
        lb += log((double)nb[i]);
    }
    double ra = la, rb = lb;  // inclusive sums over the wave's lanes
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
        const double xa = __shfl_up(ra, o, 64), xb = __shfl_up(rb, o, 64);
        lm += __shfl_xor(lm, o, 64);
        if (lane >= o) {
            ra += xa;
            rb += xb;
        }
    }
    if (work && lane == 63) {
        double* w = tot + 3 * (tid >> 6);
        w[0] = ra;
        w[1] = rb;
        w[2] = lm;
    }
    __syncthreads();
    double totA = 0.0, totB = 0.0, msum = 0.0;
    ra = __shfl_up(ra, 1, 64);  // exclusive
    rb = __shfl_up(rb, 1, 64);
    if (lane == 0) ra = rb = 0.0;
    for (int w = 0; w < workers >> 6; ++w) {
        if (w == tid >> 6) {
            ra += totA;
            rb += totB;
        }
        totA += tot[3 * w];
        totB += tot[3 * w + 1];
        msum += tot[3 * w + 2];
    }
    const double lz = log((double)static_cast<const Real*>(p.zfin)[b]) + totA;
    // the same total from the beta side: pi . beta'_0. The two agree up to rounding
    // unless a pass lost mass to underflow (a state whose alpha is below the range
    // of Real next to the frame's total while its beta is that much above, or the
    // other way round): such a sequence is flagged, not returned silently wrong
    const double lz_beta = log((double)static_cast<const Real*>(p.zfin)[p.B + b]) + totB;
    const bool nonfinite_in = !(msum == msum);
    const bool dead = !(lz > -INFINITY && lz < INFINITY) || nonfinite_in;
    const bool lossy = !dead && !(fabs(lz - lz_beta) <= kTotalsAgree);
    auto scale = [&](const int i) {
        if (i >= 1) cfac[i] = dead ? (Real)0 : (Real)exp(ra + (totB - rb) - lz);
    };
#pragma unroll
    for (int q = 0; q < kKeep; ++q)
        if (i0 + q < i1) {
            scale(i0 + q);
            ra += ka[q];
            rb += kb[q];
        }
    for (int i = i0 + kKeep; i < i1; ++i) {
        scale(i);
        ra += log((double)na[i]);
        rb += log((double)nb[i]);
    }
    if (tid == 0) {
        int st = 0;
        if (nonfinite_in) st |= 2;
        if (dead) st |= 1;
        if (lossy) st |= 4;
        const float val = nonfinite_in ? __builtin_nanf("") : (float)(lz + msum);
        const float out = p.grad_scale * val;
        if (p.objf_late) {  // k_occ adds them, see add_late_objective
            p.objf_late[b] = out;
            p.status_late[b] = st;
            return;
        }
        p.objf[b] = p.accumulate ? p.objf[b] + out : out;
        if (p.status_out) p.status_out[b] = p.accumulate ? (p.status_out[b] | st) : st;
    }
}

// What a workgroup of a recursion kernel works on. Entries 2i, 2i + 1 of the launch order are the
// two directions of a sequence; a handle's only graph is read without a wait for the sequence.
struct RecWork {
    int b, dir;
    SeqDesc sd;
    OrdDesc od;
};
__device__ __forceinline__ RecWork rec_work(const FbParams& p)
{
    RecWork w;
    w.dir = blockIdx.x & 1;
    int graph = 0;
    if (!p.one_graph) graph = p.seqs[p.order[2 * p.seq_first + blockIdx.x] >> 1].graph;
    w.od = p.g.ords[graph * 3 + w.dir];
    w.b = p.order[2 * p.seq_first + blockIdx.x] >> 1;
    w.sd = p.seqs[w.b];
    return w;
}

// At the end of a recursion kernel, by every thread.
template <typename Real>
__device__ __forceinline__ void finish_sequence(const FbParams& p, const int b, unsigned char* lds_raw)
{
    // The workgroup that finishes a sequence second (alpha or beta) computes its
    // scales: no launch of their own, and no wait for the other sequences.
    // Every wave waits for its trellis rows and scalars to have reached the L2; one thread's fences
    // on either side of the ticket then make them visible device-wide and the other workgroup's
    // visible here (fences by every wave wrote back and invalidated the caches once per wave).
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    __syncthreads();  // ... LDS is free from here on
    int* ticket = reinterpret_cast<int*>(lds_raw);
    if (threadIdx.x == 0) {
        __threadfence();
        *ticket = atomicAdd(p.done + b, 1);
        __threadfence();
    }
    __syncthreads();
    if (*ticket != 1) return;  // workgroup-uniform
    scan_sequence<Real>(p, b, lds_raw + 64);
}

}  // namespace

// ---- kernel variants ---------------------------------------------------------
using RecKernel = void (*)(FbParams);
struct RecVariant {
    int wide, nslot, yrep, leak, max_threads;
    RecKernel fn;
    int hybrid = 0;  // 1: hybrid, 2: hybrid with the large LDS map
    int hubs = 0;    // handles hub slices
    int grouped = 0; // emission by entered state: 1 RecGrouped, 2 RecShort, 3 RecLine; 4 RecLineArc
    int ypass = 0;   // RecLineArc, RecHybrid: staging passes
};
// The straight-line recursion (line.hip): its variants, their number in *n; the one for a kind of
// graph; the LDS one takes.
const RecVariant* line_variants(int* n);
const RecVariant* find_line(bool by_state, bool yrep, int leak, int num_pdfs, int max_wave_slots,
                            int threads);
size_t line_lds_bytes(const RecVariant& v);
// The same for the hybrid recursion without hub slices (hybrid.hip); map 1: 32 KB state vectors, 2: 48 KB.
constexpr int kHybridSlots = 36;  // resident slots of a wave
const RecVariant* hybrid_variants(int* n);
const RecVariant* find_hybrid(bool yrep, int leak, int num_pdfs, int map);

}  // namespace lfmmi
