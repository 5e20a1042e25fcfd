// The recursion as one straight line a step, for graphs of up to 2,048 rows whose waves own one
// or two slices (see kernels.hip for the recursion and the other variants of it).
#include "device.h"

#include <type_traits>

namespace lfmmi {
namespace {

// ---------------------------------------------------------------------------
// The same recursion as one straight line a step, for workgroups whose waves own one or two
// slices. What bounds a step of such graphs is the serial stream of instructions of a wave from
// one barrier to the next (one about every 4.6 clocks, ~20 for a branch, taken or not), not the
// gathers: 2,016 states (442 slots a step, 920 LDS clocks) took 1.05 us a step with RecGrouped, of
// which the tests for slice ends and what follows them were 0.19 and the staging of emissions
// 0.15. Here the code is laid out for the width A of the wave's first slice (the packer puts the
// narrower one first, so A is at most half the slots): no masks and no tests but two for the end
// of the wave's slots. The emission of a lane's row goes from memory into a register two steps
// ahead, with no stop in LDS; the sums of a row stay in registers; the totals of 64 steps collect
// in the lanes of a register.
// LDS map: X0 [0, 8K)  X1 [8K, 16K)  partial sums at 16K: n of wave w at value 32 * set + w, s 16
// further; unused words behind them. RecLineArc: emission rows Y0 [32K, 64K)  Y1 [64K, 96K), the
// last word of each 0.
// A step of that graph now takes 0.72 us (442 gathers of 64 lanes, 140 instructions a wave), a call
// of 64 sequences of 100 to 500 frames 629 -> 452 us; 144 states, 648 arcs: 0.54 -> 0.25 us a step.
// ---------------------------------------------------------------------------
constexpr uint32_t kLineX1 = 8192, kLinePart = 16384, kLineDump = kLinePart + 256;
constexpr uint32_t kLineY0 = 32768, kLineY1 = 65536, kLineYZero = 32764;
constexpr int kLineRows = 2048;

// A 32-bit offset to a scalar base: opaque where it is used, or the compiler widens it to 64 bits
// once and for all (two registers) and adds the base by a vector instruction at every use.
__device__ __forceinline__ uint32_t here(uint32_t& offset)
{
    asm volatile("" : "+v"(offset));
    return offset;
}

template <bool HAS_WB, int NSLOT, int NT>
struct RecLine {
    static_assert(NSLOT % 4 == 0 && NSLOT >= 16, "slots go in groups of four; two tests near the end");
    static constexpr int kGroup = 4, kRing = 8;  // two groups of gathers in flight before a step's sums
    static constexpr int kBlock = 64;            // steps whose totals collect in a register

    uint32_t xa[NSLOT];  // byte address of the gathered state value inside X0
    float wr[NSLOT];     // arc weight (0 in closing and unused slots)
    uint32_t row4[2];    // byte offset of the lane's rows in a state vector
    uint32_t ysrc[2];    // ... of their pdfs in an emission row
    float r[2], g[2];    // alpha: in_wpi of the rows; beta: in_w, in_wpi
    float e[2][2];       // [parity of the step][slice]: emissions of the rows
    typedef const __attribute__((address_space(1))) char* global_bytes_t;
    typedef const __attribute__((address_space(1))) float* global_in_t;
    typedef __attribute__((address_space(1))) char* global_out_bytes_t;
    typedef __attribute__((address_space(1))) float* global_out_t;
    global_bytes_t e2;        // emission row of the step after the next
    global_out_bytes_t trow;  // trellis row this step writes
    float inv, c;             // scale and leak of the vector the last step read
    int keep_n, keep_s;       // lane q: the totals step q of the block found

    __device__ __forceinline__ float emission(const int slice)
    {
        return *(global_in_t)(e2 + here(ysrc[slice]));
    }

    // DIR 0: alpha, 1: beta. PAR = k & 1 as in RecRegs. A: slots of the wave's first slice (0: it
    // owns one slice). `at`: the step's lane in keep_n, keep_s. `count`: the wave's slots.
    template <int PAR, int DIR, int A>
    __device__ __forceinline__ void step(const int at, const float leak_by, const uint32_t read_at,
                                         const uint32_t write_at, const int count)
    {
        constexpr uint32_t xc = PAR ? 0u : kLineX1, xn = PAR ? kLineX1 : 0u;
        constexpr uint32_t pc = kLinePart + (PAR ? 0u : 128u), pn = PAR ? 128u : 0u;
        constexpr bool kTwoSums = DIR == 1 && HAS_WB;
        float pv = lds_ld(pc + read_at);
        float xv[kRing];
#pragma unroll
        for (int i = 0; i < kRing; ++i) xv[i] = lds_ld(xc + xa[i]);
        asm volatile("" ::: "memory");
        pv = row16_allsum(pv);  // every row of 16 lanes: n (of two sums, odd rows: s)
        float nr = pv, Sd = pv;
        if constexpr (kTwoSums) {
            nr = lane_value(pv, 0);
            Sd = lane_value(pv, 16);
        }
        const uint32_t e2n = min(__float_as_uint(nr) & 0x7f800000u, 0x7e800000u);  // see pow2_scale
        inv = __uint_as_float(0x7f000000u - e2n);
        c = leak_by * Sd * inv;
        keep_n = writelane_i32(__builtin_amdgcn_readfirstlane(__float_as_int(nr)), at, keep_n);
        if constexpr (kTwoSums) keep_s = writelane_i32(__float_as_int(Sd), at, keep_s);

        float acc = 0.f, n = 0.f, s = 0.f;
        auto close = [&](const int slice) __attribute__((always_inline)) {
            const float em = e[PAR][slice];
            float x, v;
            if constexpr (DIR == 0) {
                v = x = em * fmaf(inv, acc, c * r[slice]);
                n += x;
            } else {
                v = acc;
                x = em * fmaf(inv, acc, c);
                n = fmaf(r[slice], x, n);
                if constexpr (kTwoSums) s = fmaf(g[slice], x, s);
            }
            lds_st(xn + row4[slice], x);
            *(global_out_t)(trow + here(row4[slice])) = v;
            acc = 0.f;
            e[PAR][slice] = emission(slice);
        };
#pragma unroll
        for (int i = 0; i < NSLOT; i += kGroup) {
            if (i >= NSLOT - 2 * kGroup) {
                int slots = count;
                asm volatile("" : "+s"(slots));  // compare here, in a scalar register
                if (i >= slots) break;
            }
            // issue priority falls as the wave advances (see RecRegs)
            if (i == 0) __builtin_amdgcn_s_setprio(2);
            else if (i == (NSLOT / 12) * 4) __builtin_amdgcn_s_setprio(1);
            else if (i == (NSLOT / 6) * 4) __builtin_amdgcn_s_setprio(0);
            float x[kGroup];
#pragma unroll
            for (int q = 0; q < kGroup; ++q) x[q] = xv[(i + q) % kRing];
            if (i + kRing < NSLOT) {
#pragma unroll
                for (int q = 0; q < kGroup; ++q)
                    xv[(i + q) % kRing] = lds_ld(xc + xa[(i + kRing + q) % NSLOT]);
            }
            // one wait for the group
            asm volatile("" : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]) : "v"(x[3]));
#pragma unroll
            for (int q = 0; q < kGroup; ++q) {
                acc = fmaf(wr[i + q], x[q], acc);
                if (i + q + 1 == A) close(0);
            }
        }
        close(A > 0 ? 1 : 0);
        __builtin_amdgcn_s_setprio(3);
        const float ns = kTwoSums ? half_wave_sums(n, s) : wave_sum_lane63(n);
        lds_st(pn + write_at, ns);
        __syncthreads();
    }

    template <int DIR, int A>
    __device__ __forceinline__ void steps(const int T, const int P, const int rows, const float leak_by,
                                          const float aconst, const uint32_t read_at,
                                          const uint32_t write_at, const int count, float* scalN,
                                          float* scalS, const int wave, const int lane)
    {
        constexpr bool kTwoSums = DIR == 1 && HAS_WB;
        const ptrdiff_t estep = (DIR == 0 ? 4 : -4) * (ptrdiff_t)P;
        const ptrdiff_t tstep = (DIR == 0 ? 4 : -4) * (ptrdiff_t)rows;
        auto advance = [&](const int k) __attribute__((always_inline)) {
            if (k + 2 + DIR < T) e2 += estep;
            trow += tstep;
        };
        for (int k0 = 1; k0 <= T; k0 += kBlock) {
            const int end = min(k0 + kBlock - 1, T);
            int k = k0;
            for (; k + 1 <= end; k += 2) {
                step<1, DIR, A>(k - k0, leak_by, read_at, write_at, count);
                advance(k);
                step<0, DIR, A>(k + 1 - k0, leak_by, read_at, write_at, count);
                advance(k + 1);
            }
            if (k <= end) step<1, DIR, A>(k - k0, leak_by, read_at, write_at, count);
            // alpha: of the vector that step k read; beta: the scale of the rows that it stored
            if (wave == 0 && lane <= end - k0) {
                const float nr = __int_as_float(keep_n);
                float N, unused;
                pow2_scale(nr, &N, &unused);
                const int to = DIR == 0 ? k0 - 1 + lane : T - k0 - lane;
                scalN[to] = N;
                scalS[to] = kTwoSums ? __int_as_float(keep_s) : (DIR == 0 ? nr : aconst * nr);
            }
        }
    }

    template <int DIR>
    __device__ __forceinline__ void run(const FbParams& p, const SeqDesc& sd, const OrdDesc& od,
                                        const int b)
    {
        constexpr bool kTwoSums = DIR == 1 && HAS_WB;
        const int tid = threadIdx.x;
        const int lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int nwaves = blockDim.x >> 6;
        const int T = sd.T;
        const int P = p.P;
        const int rows = od.num_slices * 64;
        float* trel = static_cast<float*>(DIR == 0 ? p.alpha : p.beta) +
                      (DIR == 0 ? sd.alpha_at : sd.beta_at);
        float* scalN = static_cast<float*>(p.scal) + (size_t)(DIR * 2) * p.scal_total + sd.scal_at;
        float* scalS = scalN + p.scal_total;
        const int32_t* so = p.g.slice_off + od.slice_off_at;
        const float eps = p.leak;
        const float* erows = p.emis + (size_t)b * p.T * P;

        int s0 = 0, s1 = 0;  // the wave's slices: none, one or two
        if (wave < od.num_waves) {
            s0 = p.g.wave_first[od.wave_first_at + wave];
            s1 = p.g.wave_first[od.wave_first_at + wave + 1];
        }
        const int first = so[s0];
        const int count = so[s1] - first;
        const int width0 = s1 - s0 == 2 ? so[s0 + 1] - first : 0;
        load_records<NSLOT>(p, od, lane, first, count, xa, wr);
        const int closing0 = HAS_WB ? width0 - 1 : -1, closing1 = HAS_WB ? count - 1 : -1;
#pragma unroll
        for (int i = 0; i < NSLOT; ++i) {
            xa[i] = xa[i] & 0xffffu;
            if (HAS_WB && (i == closing0 || i == closing1)) wr[i] = 0.f;  // holds no arc
            asm volatile("" : "+v"(xa[i]), "+v"(wr[i]));
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int row = min(s0 + q, max(s1 - 1, 0)) * 64 + lane;
            row4[q] = (uint32_t)row * 4u;
            ysrc[q] = (uint32_t)p.g.row_pdf[od.vec_at + row] * 4u;
            r[q] = (float)(DIR == 0 ? p.g.in_wpi : p.g.in_w)[od.vec_at + row];
            g[q] = kTwoSums ? (float)p.g.in_wpi[od.vec_at + row] : 0.f;
            e[0][q] = e[1][q] = 0.f;
        }
        keep_n = keep_s = 0;
        if (tid < 64) lds_st(kLinePart + tid * 4, 0.f);
        __syncthreads();

        // Frame whose emissions meet the rows that step k stores, as in RecGrouped
        auto frame_of = [&](int k) { return max(0, min(DIR == 0 ? k - 1 : T - k - 1, T - 1)); };
        auto total = [&](float a, float bsum, const uint32_t to) {  // this wave's partial sums
            a = wave_sum_uniform(a);
            bsum = wave_sum_uniform(bsum);
            if (lane == 0) {
                lds_st(to + wave * 4, a);
                lds_st(to + (16 + wave) * 4, bsum);
            }
        };
        // ---- step 0: v_0 = init into X0, partial sums into set 0
        {
            float n = 0.f, s = 0.f;
            const int ti = DIR == 0 ? 0 : T;
            for (int sl = s0; sl < s1; ++sl) {
                const int row = sl * 64 + lane;
                const float v = p.g.vinit[od.vec_at + row];
                lds_st(row * 4, v);
                trel[(size_t)ti * rows + row] = v;
                n += v;
                s += p.g.va[od.vec_at + row] * v;
            }
            // beta: into set 1 first, the vector itself needs the totals
            total(n, s, kLinePart + (DIR == 0 ? 0u : 128u));
            if (T > 0) {
#pragma unroll
                for (int k = 1; k <= 2; ++k) {
                    e2 = (global_bytes_t)(erows + (size_t)frame_of(k) * P);
                    e[k & 1][0] = emission(0);
                    e[k & 1][1] = emission(1);
                }
                e2 = (global_bytes_t)(erows + (size_t)frame_of(3) * P);
            }
            __syncthreads();
            if constexpr (DIR == 1) {
                const float pv = row16_allsum(lds_ld(kLinePart + (32u + (lane & 31)) * 4u));
                const float nr = lane_value(pv, 0), Sd = lane_value(pv, 16);
                float N;
                pow2_scale(nr, &N, &inv);
                c = eps * Sd * inv;
                if (tid == 0) {
                    scalN[T] = N;
                    scalS[T] = Sd;
                }
                n = s = 0.f;
                const float* em = erows + (size_t)max(T - 1, 0) * P;
                for (int q = 0; q < s1 - s0 && T > 0; ++q) {
                    const uint32_t at = (uint32_t)((s0 + q) * 64 + lane) * 4u;
                    const int vec = od.vec_at + (s0 + q) * 64 + lane;
                    const float u = em[p.g.row_pdf[vec]] * (inv * lds_ld(at) + c);
                    lds_st(at, u);
                    n += (float)p.g.in_w[vec] * u;
                    if (kTwoSums) s += (float)p.g.in_wpi[vec] * u;
                }
                total(n, s, kLinePart);
                __syncthreads();
            }
        }
        trow = (global_out_bytes_t)(trel + (size_t)(DIR == 0 ? 1 : T - 1) * rows);
        const float aconst = od.a_const;
        const float leak_by = DIR == 0 || kTwoSums ? eps : eps * aconst;
        const uint32_t read_at = (uint32_t)(lane & (kTwoSums ? 31 : 15)) * 4u;
        // where the end-of-step sums go: n from lane 63; of two sums n from lane 31, s from 63
        const bool says = kTwoSums ? (lane & 31) == 31 : lane == 63;
        const uint32_t write_at =
            says ? kLinePart + ((uint32_t)wave + (kTwoSums && lane == 63 ? 16u : 0u)) * 4u
                 : kLineDump + (uint32_t)lane * 4u;
        if (s1 > s0) {
#define LFMMI_LINE_STEPS(A)                                                                      \
    case A:                                                                                      \
        if constexpr (A <= NSLOT / 2)                                                            \
            steps<DIR, A>(T, P, rows, leak_by, aconst, read_at, write_at, count, scalN, scalS,   \
                          wave, lane);                                                           \
        break;
            switch (width0) {
                LFMMI_LINE_STEPS(0) LFMMI_LINE_STEPS(2) LFMMI_LINE_STEPS(4) LFMMI_LINE_STEPS(6)
                LFMMI_LINE_STEPS(8) LFMMI_LINE_STEPS(10) LFMMI_LINE_STEPS(12) LFMMI_LINE_STEPS(14)
                LFMMI_LINE_STEPS(16) LFMMI_LINE_STEPS(18)
                LFMMI_LINE_STEPS(20) LFMMI_LINE_STEPS(22) LFMMI_LINE_STEPS(24)
            }
#undef LFMMI_LINE_STEPS
        } else {
            for (int k = 1; k <= T; ++k) __syncthreads();
        }

        // ---- last scalars (alpha) and the closing dot product; beta's last rows are read
        // back from the trellis, each by the thread that stored it
        {
            if constexpr (DIR == 0) {
                const uint32_t pc = kLinePart + ((T & 1) ? 128u : 0u);
                const float nr = lane_value(row16_allsum(lds_ld(pc + (lane & 15) * 4u)), 0);
                float N;
                pow2_scale(nr, &N, &inv);
                c = eps * nr * inv;
                if (tid == 0) {
                    scalN[T] = N;
                    scalS[T] = nr;
                }
            }
            float z = 0.f;
            for (int sl = s0; sl < s1; ++sl) {
                const int row = sl * 64 + lane;
                const float raw = DIR == 0 ? lds_ld(((T & 1) ? kLineX1 : 0u) + row * 4) : trel[row];
                const float v = raw * inv + c * p.g.vb[od.vec_at + row];
                z += p.g.vfin[od.vec_at + row] * v;
            }
            z = wave_sum_uniform(z);
            __syncthreads();
            if (lane == 0) lds_st(kLinePart + wave * 4, z);
            __syncthreads();
            if (tid == 0) {
                float Z = 0.f;
                for (int w = 0; w < nwaves; ++w) Z += lds_ld(kLinePart + w * 4);
                static_cast<float*>(p.zfin)[(size_t)DIR * p.B + b] = Z;
            }
        }
    }
};

// ---------------------------------------------------------------------------
// The straight line for graphs whose arcs carry pdfs of their own: two gathers an arc, as in
// RecRegs (LEAK 0 and 2 there), the emission row in LDS (32 copies of it with YREP). Bound by the
// vector instructions of a step as much as by the gathers. What it saves against RecRegs is the
// tests for slice ends, waits for the last step's trellis stores ahead of the staging of the next
// emission row, and the branches of that staging: every wave stages an equal share of the row.
// n is the power of two below the total, as in RecGrouped (its inverse needs no reciprocal).
// Time of a step with RecRegs / here, one sequence: 20 states 0.55 / 0.27 us; 300 states, 3,000 arcs
// 0.67 / 0.45; 600, 5,400 0.83 / 0.59; 1,237, 8,659 (initial probabilities that differ) 0.87 / 0.80;
// 2,000, 20,000 1.08 / 0.98 (there the waves' 22 slots of three vector instructions bound it); 300
// pdfs, plain rows 1.27 / 1.17. A call of 64 sequences of 100 to 500 frames, 2,000 states: 653 -> 588.
// YPASS: staging passes (YREP: quads of copies, else values).
// ---------------------------------------------------------------------------
template <bool YREP, int YPASS, int LEAK, int NSLOT, int NT>
struct RecLineArc {
    static_assert(LEAK == 0 || LEAK == 2, "no leak factors per arc");
    static constexpr bool ROWS = LEAK == 2;
    static constexpr int kRing = 4;    // slots whose gathers are in flight ahead of a step's sums
    static constexpr int kAhead = 2;   // ... and ahead of the slots in use
    static constexpr int kStageAt = 4;
    static constexpr int kBlock = 64;
    static_assert(NSLOT % 2 == 0 && NSLOT >= 16, "slots go in pairs; tests near the end");

    uint32_t xa[NSLOT];  // byte address of the gathered state value inside X0
    uint32_t ya[NSLOT];  // ... of the emission value, in Y0
    float wr[NSLOT];
    uint32_t row4[2];
    float a[2];              // ROWS: the rows' initial probabilities
    float yreg[YPASS];       // emission values this lane stages, a step ahead
    uint32_t ysrc[YPASS];    // byte offset of such a value inside an emission row
    uint32_t ydst[YPASS];    // YREP: where its copies go in Y0 (else: at the same offset)
    typedef const __attribute__((address_space(1))) char* global_bytes_t;
    typedef const __attribute__((address_space(1))) float* global_in_t;
    typedef __attribute__((address_space(1))) char* global_out_bytes_t;
    typedef __attribute__((address_space(1))) float* global_out_t;
    typedef float lds_pair_t __attribute__((ext_vector_type(2)));
    global_bytes_t e2;
    global_out_bytes_t trow;
    int keep_n;

    __device__ __forceinline__ void load_y()
    {
#pragma unroll
        for (int i = 0; i < YPASS; ++i) yreg[i] = *(global_in_t)(e2 + here(ysrc[i]));
    }
    template <int BUF>
    __device__ __forceinline__ void store_y()
    {
#pragma unroll
        for (int i = 0; i < YPASS; ++i) {
            constexpr uint32_t buf = BUF ? kLineY1 - kLineY0 : 0u;
            if constexpr (YREP) {  // four adjacent words, a pair at a time: see RecRegs::store_y
                typedef __attribute__((address_space(3))) lds_pair_t* lds_pair_at;
                const lds_pair_t two = {yreg[i], yreg[i]};
                const uint32_t at = here(ydst[i]);
                *(lds_pair_at)(static_cast<uintptr_t>(at + buf)) = two;
                *(lds_pair_at)(static_cast<uintptr_t>((at ^ 8u) + buf)) = two;
            } else {
                lds_st(kLineY0 + buf + ysrc[i], yreg[i]);
            }
        }
    }

    template <int PAR, int A>
    __device__ __forceinline__ void step(const int at, const float leak_by, const uint32_t read_at,
                                         const uint32_t write_at, const int count)
    {
        constexpr uint32_t xc = PAR ? 0u : kLineX1, xn = PAR ? kLineX1 : 0u;
        constexpr uint32_t yc = PAR ? 0u : kLineY1 - kLineY0;
        constexpr uint32_t pc = kLinePart + (PAR ? 0u : 128u), pn = PAR ? 128u : 0u;
        float pv = lds_ld(pc + read_at);
        float xv[kRing], ev[kRing];
#pragma unroll
        for (int i = 0; i < kRing; ++i) {
            xv[i] = lds_ld(xc + xa[i]);
            ev[i] = lds_ld(yc + ya[i]);
        }
        asm volatile("" ::: "memory");
        pv = row16_allsum(pv);
        const uint32_t e2n = min(__float_as_uint(pv) & 0x7f800000u, 0x7e800000u);  // see pow2_scale
        const float inv = __uint_as_float(0x7f000000u - e2n);
        const float c = leak_by * pv * inv;
        keep_n = writelane_i32(__builtin_amdgcn_readfirstlane(__float_as_int(pv)), at, keep_n);

        float acc1 = 0.f, acc2 = 0.f, n = 0.f;
        auto close = [&](const int slice) __attribute__((always_inline)) {
            const float v = fmaf(inv, acc1, c * acc2);
            lds_st(xn + row4[slice], v);
            *(global_out_t)(trow + here(row4[slice])) = v;
            if constexpr (ROWS) n = fmaf(a[slice], v, n);
            else n += v;
            acc1 = acc2 = 0.f;
        };
#pragma unroll
        for (int i = 0; i < NSLOT; i += 2) {
            if (i >= NSLOT - 8 && i % 4 == 0) {
                int slots = count;
                asm volatile("" : "+s"(slots));  // compare here, in a scalar register
                if (i >= slots) break;
            }
            // issue priority falls as the wave advances (see RecRegs)
            if (i == 0) __builtin_amdgcn_s_setprio(2);
            else if (i == (NSLOT / 6) * 2) __builtin_amdgcn_s_setprio(1);
            else if (i == (NSLOT / 3) * 2) __builtin_amdgcn_s_setprio(0);
            if (i == kStageAt) {  // the row of step k + 1 to LDS, the loads for step k + 2
                store_y<PAR>();
                load_y();
            }
            float x0 = xv[i % kRing], x1 = xv[(i + 1) % kRing];
            float e0 = ev[i % kRing], e1 = ev[(i + 1) % kRing];
            if (i + kAhead < NSLOT && i + kAhead >= kRing) {  // (the opening burst is in flight)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    xv[(i + kAhead + q) % kRing] = lds_ld(xc + xa[(i + kAhead + q) % NSLOT]);
                    ev[(i + kAhead + q) % kRing] = lds_ld(yc + ya[(i + kAhead + q) % NSLOT]);
                }
            }
            asm volatile("" : "+v"(x0), "+v"(e0) : "v"(x1), "v"(e1));  // one wait for the pair
            auto arc = [&](const float w, const float e, const float x) __attribute__((always_inline)) {
                if constexpr (ROWS) {  // emission times value first: see RecRegs::add_arc
                    acc1 = fmaf(w, e * x, acc1);
                    acc2 = fmaf(w, e, acc2);
                } else {
                    const float t = w * e;
                    acc1 = fmaf(t, x, acc1);
                    acc2 += t;
                }
            };
            arc(wr[i], e0, x0);
            arc(wr[i + 1], e1, x1);
            if (i + 2 == A) close(0);
        }
        close(A > 0 ? 1 : 0);
        __builtin_amdgcn_s_setprio(3);
        lds_st(pn + write_at, wave_sum_lane63(n));
        __syncthreads();
    }

    // A < 0: a wave that owns no slice helps to stage emissions.
    template <int A>
    __device__ __forceinline__ void steps(const int T, const ptrdiff_t estep, const ptrdiff_t tstep,
                                          const float leak_by, const float sconst,
                                          const uint32_t read_at, const uint32_t write_at,
                                          const int count, float* sN, float* sS, const int sstep,
                                          const int wave, const int lane)
    {
        auto advance = [&](const int k) __attribute__((always_inline)) {
            if (k + 2 < T) e2 += estep;
            trow += tstep;
        };
        auto one = [&](auto par, const int at) __attribute__((always_inline)) {
            if constexpr (A >= 0) {
                step<decltype(par)::value, A>(at, leak_by, read_at, write_at, count);
            } else {
                store_y<decltype(par)::value>();
                load_y();
                __syncthreads();
            }
        };
        for (int k0 = 1; k0 <= T; k0 += kBlock) {
            const int end = min(k0 + kBlock - 1, T);
            int k = k0;
            for (; k + 1 <= end; k += 2) {
                one(std::integral_constant<int, 1>(), k - k0);
                advance(k);
                one(std::integral_constant<int, 0>(), k + 1 - k0);
                advance(k + 1);
            }
            if (k <= end) one(std::integral_constant<int, 1>(), k - k0);
            if (A >= 0 && wave == 0 && lane <= end - k0) {  // of the vectors that the steps read
                const float nr = __int_as_float(keep_n);
                float N, unused;
                pow2_scale(nr, &N, &unused);
                sN[(k0 - 1 + lane) * sstep] = N;
                sS[(k0 - 1 + lane) * sstep] = sconst * nr;
            }
        }
    }

    __device__ __forceinline__ void run(const FbParams& p, const SeqDesc& sd, const OrdDesc& od,
                                        const int b, const int dir)
    {
        const int tid = threadIdx.x;
        const int lane = tid & 63;
        const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
        const int nwaves = blockDim.x >> 6;
        const int T = sd.T;
        const int P = p.P;
        const int rows = od.num_slices * 64;
        float* trel = static_cast<float*>(dir == 0 ? p.alpha : p.beta) +
                      (dir == 0 ? sd.alpha_at : sd.beta_at);
        float* scalN = static_cast<float*>(p.scal) + (size_t)(dir * 2) * p.scal_total + sd.scal_at;
        float* scalS = scalN + p.scal_total;
        const int32_t* so = p.g.slice_off + od.slice_off_at;
        const float eps = p.leak;
        const float* erows = p.emis + (size_t)b * p.T * P;

        int s0 = 0, s1 = 0;  // the wave's slices: none, one or two
        if (wave < od.num_waves) {
            s0 = p.g.wave_first[od.wave_first_at + wave];
            s1 = p.g.wave_first[od.wave_first_at + wave + 1];
        }
        const int first = so[s0];
        const int count = so[s1] - first;
        const int width0 = s1 - s0 == 2 ? so[s0 + 1] - first : 0;
        load_records<NSLOT>(p, od, lane, first, count, ya, wr);
#pragma unroll
        for (int i = 0; i < NSLOT; ++i) {
            xa[i] = ya[i] & 0xffffu;
            ya[i] = kLineY0 + (i < count ? y_offset(ya[i]) : kLineYZero);
            asm volatile("" : "+v"(xa[i]), "+v"(ya[i]), "+v"(wr[i]));
        }
#pragma unroll
        for (int q = 0; q < 2; ++q) {
            const int row = min(s0 + q, max(s1 - 1, 0)) * 64 + lane;
            row4[q] = (uint32_t)row * 4u;
            a[q] = ROWS ? p.g.va[od.vec_at + row] : 0.f;
        }
        {  // an equal share of the row for every wave, in whole groups of eight quads or values
            const int units = YREP ? P * 8 : P;
            const int share = ((units + nwaves - 1) / nwaves + 7) & ~7;
#pragma unroll
            for (int i = 0; i < YPASS; ++i) {
                // lanes past the share and shares past the row repeat the work of others
                const int q = (wave * share + (i * 64 + lane) % share) % units;
                ysrc[i] = (uint32_t)(YREP ? q >> 3 : q) * 4u;
                ydst[i] = kLineY0 + (uint32_t)q * (YREP ? 16u : 4u) +
                          (YREP ? (uint32_t)((q >> 3) & 1) * 8u : 0u);
                yreg[i] = 0.f;
            }
        }
        keep_n = 0;
        if (tid == 0) {
            lds_st(kLineY0 + kLineYZero, 0.f);
            lds_st(kLineY1 + kLineYZero, 0.f);
        }
        if (tid < 64) lds_st(kLinePart + tid * 4, 0.f);
        __syncthreads();

        // ---- step 0: v_0 = init into X0, partial sums into set 0
        {
            float n = 0.f;
            const int ti = dir == 0 ? 0 : T;
            for (int sl = s0; sl < s1; ++sl) {
                const int row = sl * 64 + lane;
                const float v = p.g.vinit[od.vec_at + row];
                lds_st(row * 4, v);
                trel[(size_t)ti * rows + row] = v;
                n += ROWS ? p.g.va[od.vec_at + row] * v : v;
            }
            n = wave_sum_uniform(n);
            if (lane == 0) lds_st(kLinePart + wave * 4, n);
            // rows of steps 1 (into Y0 now) and 2 (into registers); frame of step k: alpha k - 1,
            // beta T - k, kept inside the sequence
            auto frame_of = [&](int k) { return max(0, min(dir == 0 ? k - 1 : T - k, T - 1)); };
            if (T > 0) {
                e2 = (global_bytes_t)(erows + (size_t)frame_of(1) * P);
                load_y();
                store_y<0>();
                e2 = (global_bytes_t)(erows + (size_t)frame_of(2) * P);
                load_y();
                e2 = (global_bytes_t)(erows + (size_t)frame_of(3) * P);
            }
            __syncthreads();
        }
        trow = (global_out_bytes_t)(trel + (size_t)(dir == 0 ? 1 : T - 1) * rows);
        const ptrdiff_t estep = (dir == 0 ? 4 : -4) * (ptrdiff_t)P;
        const ptrdiff_t tstep = (dir == 0 ? 4 : -4) * (ptrdiff_t)rows;
        // s = sconst * n; the leak's share of a row is leak_by * n / N times its second sum
        const float sconst = ROWS ? 1.f : od.a_const;
        const float leak_by = ROWS ? eps : eps * sconst * od.b_const;
        const uint32_t read_at = (uint32_t)(lane & 15) * 4u;
        const uint32_t write_at =
            lane == 63 ? kLinePart + (uint32_t)wave * 4u : kLineDump + (uint32_t)lane * 4u;
        float* const sN = scalN + (dir == 0 ? 0 : T);  // the scalars of step 0
        float* const sS = scalS + (dir == 0 ? 0 : T);
        const int sstep = dir == 0 ? 1 : -1;
#define LFMMI_LINE_STEPS(A)                                                                        \
    case A:                                                                                        \
        if constexpr (A <= NSLOT / 2)                                                              \
            steps<A>(T, estep, tstep, leak_by, sconst, read_at, write_at, count, sN, sS, sstep,    \
                     wave, lane);                                                                  \
        break;
        switch (s1 > s0 ? width0 : -1) {
            LFMMI_LINE_STEPS(-1)
            LFMMI_LINE_STEPS(0) LFMMI_LINE_STEPS(2) LFMMI_LINE_STEPS(4) LFMMI_LINE_STEPS(6)
            LFMMI_LINE_STEPS(8) LFMMI_LINE_STEPS(10) LFMMI_LINE_STEPS(12) LFMMI_LINE_STEPS(14)
        }
#undef LFMMI_LINE_STEPS

        // ---- last scalars and the closing dot product
        {
            const float nr =
                lane_value(row16_allsum(lds_ld(kLinePart + ((T & 1) ? 128u : 0u) + (lane & 15) * 4u)), 0);
            float N, inv;
            pow2_scale(nr, &N, &inv);
            const float c = eps * sconst * nr * inv;
            if (tid == 0) {
                const int tp = dir == 0 ? T : 0;
                scalN[tp] = N;
                scalS[tp] = sconst * nr;
            }
            float z = 0.f;
            for (int sl = s0; sl < s1; ++sl) {
                const int row = sl * 64 + lane;
                const float v = lds_ld(((T & 1) ? kLineX1 : 0u) + row * 4) * inv +
                                c * p.g.vb[od.vec_at + row];
                z += p.g.vfin[od.vec_at + row] * v;
            }
            z = wave_sum_uniform(z);
            __syncthreads();  // every wave has read the partial sums
            if (lane == 0) lds_st(kLinePart + wave * 4, z);
            __syncthreads();
            if (tid == 0) {
                float Z = 0.f;
                for (int w = 0; w < nwaves; ++w) Z += lds_ld(kLinePart + w * 4);
                static_cast<float*>(p.zfin)[(size_t)dir * p.B + b] = Z;
            }
        }
    }
};

template <bool HAS_WB, int NSLOT, int NT>
__global__ void __launch_bounds__(NT) k_rec_line(FbParams p)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const RecWork work = rec_work(p);
    const int b = work.b, dir = work.dir;
    const SeqDesc sd = work.sd;
    const OrdDesc od = work.od;
    RecLine<HAS_WB, NSLOT, NT> r;
    if (dir == 0) r.template run<0>(p, sd, od, b);
    else r.template run<1>(p, sd, od, b);
    finish_sequence<float>(p, b, lds_raw);
}

template <bool YREP, int YPASS, int LEAK, int NSLOT, int NT>
__global__ void __launch_bounds__(NT) k_rec_line_arc(FbParams p)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const RecWork work = rec_work(p);
    const int b = work.b, dir = work.dir;
    const SeqDesc sd = work.sd;
    const OrdDesc od = work.od;
    RecLineArc<YREP, YPASS, LEAK, NSLOT, NT> r;
    r.run(p, sd, od, b, dir);
    finish_sequence<float>(p, b, lds_raw);
}

#define LFMMI_LINE(NSLOT, WB, NT) {0, NSLOT, 0, WB, NT, k_rec_line<WB == 1, NSLOT, NT>, 0, 0, 3}
#define LFMMI_LINE_ARC(YREP, YPASS, LEAK, NSLOT) \
    {0, NSLOT, YREP, LEAK, 1024, k_rec_line_arc<YREP != 0, YPASS, LEAK, NSLOT, 1024>, 0, 0, 4, YPASS}
#define LFMMI_LINE_ARCS(NSLOT)                                                          \
    LFMMI_LINE_ARC(1, 1, 0, NSLOT), LFMMI_LINE_ARC(1, 2, 0, NSLOT), LFMMI_LINE_ARC(0, 3, 0, NSLOT), \
    LFMMI_LINE_ARC(1, 1, 2, NSLOT), LFMMI_LINE_ARC(1, 2, 2, NSLOT), LFMMI_LINE_ARC(0, 3, 2, NSLOT)
const RecVariant kLineVariants[] = {
    LFMMI_LINE(16, 0, 1024), LFMMI_LINE(24, 0, 1024), LFMMI_LINE(32, 0, 1024),
    LFMMI_LINE(36, 0, 1024), LFMMI_LINE(48, 0, 512),
    LFMMI_LINE(16, 1, 1024), LFMMI_LINE(24, 1, 1024), LFMMI_LINE(32, 1, 1024),
    LFMMI_LINE(36, 1, 1024), LFMMI_LINE(48, 1, 512),
    LFMMI_LINE_ARCS(16), LFMMI_LINE_ARCS(24), LFMMI_LINE_ARCS(28),
};
#undef LFMMI_LINE
#undef LFMMI_LINE_ARC
#undef LFMMI_LINE_ARCS

}  // namespace

// The smallest variant for this kind of graph that holds max_wave_slots, or null.
const RecVariant* find_line(bool by_state, bool yrep, int leak, int num_pdfs, int max_wave_slots,
                            int threads)
{
    const int units = yrep ? num_pdfs * 8 : num_pdfs;
    const RecVariant* best = nullptr;
    for (const RecVariant& v : kLineVariants) {
        if (v.grouped != (by_state ? 3 : 4) || v.leak != leak || v.nslot < max_wave_slots ||
            threads > v.max_threads)
            continue;
        if (!by_state && (v.yrep != (yrep ? 1 : 0) || units > v.ypass * v.max_threads)) continue;
        if (!best || v.nslot < best->nslot || (v.nslot == best->nslot && v.ypass < best->ypass)) best = &v;
    }
    return best;
}

const RecVariant* line_variants(int* n)
{
    *n = (int)(sizeof kLineVariants / sizeof kLineVariants[0]);
    return kLineVariants;
}

size_t line_lds_bytes(const RecVariant& v)
{
    return v.grouped == 4 ? kLineY1 + 32768 : kLineDump + 384;
}

int rec_line_slots(bool by_state, bool yrep, int leak, int num_pdfs, int max_wave_slots, int threads)
{
    const RecVariant* v = find_line(by_state, yrep, leak, num_pdfs, max_wave_slots, threads);
    return v ? v->nslot : 0;
}

int rec_line_max_rows() { return kLineRows; }

}  // namespace lfmmi
