// The recursion of graphs with more arcs than the registers hold, without hub slices (see RecRegs in
// kernels.hip, whose hybrid form this replaces there).
#include "device.h"

namespace lfmmi {
namespace {

// ---------------------------------------------------------------------------
// The first NSLOT slots of a wave stay in registers, both LDS addresses of a slot in one of them, the
// records of the others come from L2 in every step. Protocol, LDS maps and arithmetic of an arc are
// those of RecRegs (LEAK 0 and 2 there; BIG: 48 KB state vectors, 16 KB emission rows). What is
// different is what a wave issues besides its slots, and when:
//   - the records of its first two streamed pairs are asked for while the resident slots are worked
//     on, not when those are done (an L2 latency of every step);
//   - every wave stages an equal share of the next emission row, with no branches;
//   - n is the power of two below the total, and the totals of 64 steps are stored together;
//   - memory is addressed by a scalar base and a 32-bit offset.
// Calls with the hybrid form of RecRegs and the fences of every wave / with this one and one thread's:
// 5,000 states, 50,000 arcs, 32 sequences of 200 to 1,600 frames 4,961 / 4,648 us (a step 3.0 -> 2.75 us);
// of 100 to 500, initial probabilities that differ 1,827 / 1,684; 7,398 states, B = 128 3,179 / 2,811;
// 10,000 states, 3,000 pdfs, B = 128 6,083 / 5,765 (5,765 to 6,060 on other cards: streamed slots and
// occupancies keep every compute unit busy).
// ---------------------------------------------------------------------------
template <bool YREP, int YPASS, int LEAK, int NSLOT, bool BIG>
struct RecHybrid {
    static constexpr bool ROWS = LEAK == 2;
    static_assert(LEAK == 0 || LEAK == 2, "no leak factors per arc");
    static_assert(!BIG || !YREP, "the large map: plain emission rows");
    static constexpr uint32_t kX1 = BIG ? 49152u : 32768u;
    static constexpr uint32_t kY0 = BIG ? 98304u : 65536u;
    static constexpr uint32_t kY1 = BIG ? 114688u : 98304u;
    static constexpr uint32_t kYZero = BIG ? 16380u : 32764u;  // see rec_zero_word()
    static constexpr uint32_t kPart = 131072u, kDump = kPart + 256u;
    static_assert((kY0 & 0xffff7fffu) == 0x10000u, "see y_of()");
    static constexpr int kTailSlots = 4;  // before these a wave may find that it has no more
    static constexpr int kStageAt = 12;
    static constexpr int kBlock = 64;
    static_assert(NSLOT % 2 == 0 && kStageAt < NSLOT - kTailSlots && NSLOT <= 64, "pairs; every wave stages");
    typedef const __attribute__((address_space(1))) char* global_bytes_t;
    typedef const __attribute__((address_space(1))) float* global_in_t;
    typedef __attribute__((address_space(1))) char* global_out_bytes_t;
    typedef __attribute__((address_space(1))) float* global_out_t;
    typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
    typedef const __attribute__((address_space(1))) u32x4_t* global_u32x4_t;
    typedef float lds_pair_t __attribute__((ext_vector_type(2)));
    typedef __attribute__((address_space(3))) lds_pair_t* lds_pair_at;

    uint32_t key[NSLOT];  // the state value's address in X0, above it the emission value's less 64 KB
    float wr[NSLOT];
    float yreg[YPASS];
    uint32_t ysrc[YPASS], ydst[YPASS];
    int keep_n;
    int so_tab, stream_end;  // lane l: the end of the wave's l-th streamed slice; of all of them
    global_bytes_t e2;
    global_out_bytes_t trow;
    global_bytes_t rbase;    // the wave's streamed pairs
    int last;                // index of the last of them
    uint32_t lane16;

    static __device__ __forceinline__ uint32_t here(uint32_t& offset)
    {
        asm volatile("" : "+v"(offset));  // (see line.hip)
        return offset;
    }
    static __device__ __forceinline__ void add_arc(const float w, const float e, const float x,
                                                   float& acc1, float& acc2)
    {
        if constexpr (ROWS) {  // emission times value first: see RecRegs::add_arc
            acc1 = fmaf(w, e * x, acc1);
            acc2 = fmaf(w, e, acc2);
        } else {
            const float t = w * e;
            acc1 = fmaf(t, x, acc1);
            acc2 += t;
        }
    }
    __device__ __forceinline__ void load_y()
    {
#pragma unroll
        for (int i = 0; i < YPASS; ++i) {
            // (two passes of copies: out of the other address, or two registers too many)
            if constexpr (YREP && YPASS > 1) yreg[i] = *(global_in_t)(e2 + ((here(ydst[i]) >> 7) << 2));
            else yreg[i] = *(global_in_t)(e2 + here(ysrc[i]));
        }
    }
    template <uint32_t BUF>
    __device__ __forceinline__ void store_y()
    {
#pragma unroll
        for (int i = 0; i < YPASS; ++i) {
            if constexpr (YREP) {  // four adjacent words, a pair at a time: see RecRegs::store_y
                const lds_pair_t two = {yreg[i], yreg[i]};
                const uint32_t at = here(ydst[i]);
                *(lds_pair_at)(static_cast<uintptr_t>(at + BUF)) = two;
                *(lds_pair_at)(static_cast<uintptr_t>((at ^ 8u) + BUF)) = two;
            } else {
                lds_st(BUF + here(ysrc[i]), yreg[i]);
            }
        }
    }
    __device__ __forceinline__ uint4 pair_at(const int q) const
    {
        const u32x4_t v = *(global_u32x4_t)(rbase + ((uint32_t)q * 1024u + lane16));
        return make_uint4(v.x, v.y, v.z, v.w);
    }

    template <int PAR>
    __device__ __forceinline__ void step(const int at, const float leak_by, const uint32_t read_at,
                                         const uint32_t write_at, const int lane, const uint64_t mask,
                                         const uint32_t row4_first, const int nsl, const int sl_stream,
                                         const int sl_end, const int first_streamed, const int32_t* so)
    {
        constexpr uint32_t xc = PAR ? 0u : kX1, xn = PAR ? kX1 : 0u;
        constexpr uint32_t yc = PAR ? 0u : kY1 - kY0, yn = PAR ? kY1 : kY0;
        constexpr uint32_t pc = kPart + (PAR ? 0u : 128u), pn = PAR ? 128u : 0u;
        // opaque once a step: the addresses are taken out of the keys where they are used
#pragma unroll
        for (int i = 0; i < NSLOT; ++i) asm volatile("" : "+v"(key[i]));
        // the upper half of the register below a 1: 64 KB + the stored half; what else leads to the
        // buffer of this parity folds into the offset field of the read
        auto y_of = [&](const uint32_t k) {
            return (yc + kY0 - 0x10000u) + __builtin_amdgcn_alignbit(1u, k, 16u);
        };
        auto resident_y = [&](const uint32_t k) { return yc + __builtin_amdgcn_alignbit(1u, k, 16u); };
        float pv = lds_ld(pc + read_at);
        float xv[2], ev[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            xv[i] = lds_ld(xc + (key[i] & 0xffffu));
            ev[i] = lds_ld(resident_y(key[i]));
        }
        asm volatile("" ::: "memory");
        pv = row16_allsum(pv);
        const uint32_t e2n = min(__float_as_uint(pv) & 0x7f800000u, 0x7e800000u);  // see pow2_scale
        const float inv = __uint_as_float(0x7f000000u - e2n);
        const float c = leak_by * pv * inv;
        keep_n = writelane_i32(__builtin_amdgcn_readfirstlane(__float_as_int(pv)), at, keep_n);

        float acc1 = 0.f, acc2 = 0.f, n = 0.f;
        uint64_t left = mask;
        int next_close = left ? __builtin_ctzll(left) : 64;
        uint32_t row4 = row4_first;
        uint4 q0, q1;
#pragma unroll
        for (int i = 0; i < NSLOT; i += 2) {
            if (i >= NSLOT - kTailSlots) {
                int slots = nsl;
                asm volatile("" : "+s"(slots));  // compare here, in a scalar register
                if (i >= slots) break;
            }
            // issue priority falls as the wave advances (see RecRegs)
            if (i == 0) __builtin_amdgcn_s_setprio(2);
            else if (i == (NSLOT / 6) * 2) __builtin_amdgcn_s_setprio(1);
            else if (i == (NSLOT / 3) * 2) __builtin_amdgcn_s_setprio(0);
            if (i == kStageAt) {  // the row of step k + 1 to LDS, the loads for step k + 2; first records
                store_y<yn>();
                load_y();
                q0 = pair_at(0);
                q1 = pair_at(min(1, last));
            }
            float x0 = xv[0], x1 = xv[1], e0 = ev[0], e1 = ev[1];
            if (i + 2 < NSLOT) {
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    xv[q] = lds_ld(xc + (key[(i + 2 + q) % NSLOT] & 0xffffu));
                    ev[q] = lds_ld(resident_y(key[(i + 2 + q) % NSLOT]));
                }
            }
            asm volatile("" : "+v"(x0), "+v"(e0) : "v"(x1), "v"(e1));  // one wait for the pair
            add_arc(wr[i], e0, x0, acc1, acc2);
            add_arc(wr[i + 1], e1, x1, acc1, acc2);
            if (__builtin_expect(i + 1 == next_close, 0)) {  // wave-uniform: a slice ends
                const float v = fmaf(inv, acc1, c * acc2);
                lds_st(xn + row4, v);
                *(global_out_t)(trow + here(row4)) = v;
                if constexpr (ROWS) n = fmaf(wr[i + 1], v, n);  // the closing slot's w is a[row]
                else n += v;
                acc1 = acc2 = 0.f;
                row4 += 256u;
                left &= left - 1;
                next_close = left ? __builtin_ctzll(left) : 64;
            }
        }
        // The wave's other slices (the first of them may have begun in the registers). Pairs of slots
        // in a flat sequence, four pairs in registers: two are being used while the two after them
        // load, and the eight gathers of two pairs go out before the first is waited for. Loads past
        // the wave's last pair repeat it (in bounds, never used).
        int i = first_streamed;  // even
        if (i < stream_end) {
            int sl = sl_stream;
            auto slice_end = [&](const int s) {  // one past the last slot of slice `s`
                if (s >= sl_end) return stream_end;
                return s - sl_stream < 64 ? __builtin_amdgcn_readlane(so_tab, s - sl_stream) : so[s + 1];
            };
            int o1 = slice_end(sl);
            auto close = [&](const uint32_t closing_w) {  // w of the slice's last slot
                const float v = fmaf(inv, acc1, c * acc2);
                uint32_t to = (uint32_t)(sl * 64 + lane) * 4u;
                lds_st(xn + to, v);
                *(global_out_t)(trow + here(to)) = v;
                if constexpr (ROWS) n = fmaf(__uint_as_float(closing_w), v, n);
                else n += v;
                acc1 = acc2 = 0.f;
                ++sl;
                o1 = slice_end(sl);
            };
            auto two_pairs = [&](const uint4 qa, const uint4 qb, const bool b_valid) {
                float e0 = lds_ld(y_of(qa.x)), x0 = lds_ld(xc + (qa.x & 0xffffu));
                float e1 = lds_ld(y_of(qa.z)), x1 = lds_ld(xc + (qa.z & 0xffffu));
                float ee2 = lds_ld(y_of(qb.x)), x2 = lds_ld(xc + (qb.x & 0xffffu));
                float e3 = lds_ld(y_of(qb.z)), x3 = lds_ld(xc + (qb.z & 0xffffu));
                // one wait for the eight: the first use names the value loaded last
                asm volatile("" : "+v"(x0), "+v"(e0), "+v"(x1), "+v"(e1), "+v"(x2), "+v"(ee2)
                             : "v"(x3), "v"(e3));
                add_arc(__uint_as_float(qa.y), e0, x0, acc1, acc2);
                add_arc(__uint_as_float(qa.w), e1, x1, acc1, acc2);
                i += 2;
                if (i == o1) close(qa.w);
                if (b_valid) {
                    add_arc(__uint_as_float(qb.y), ee2, x2, acc1, acc2);
                    add_arc(__uint_as_float(qb.w), e3, x3, acc1, acc2);
                    i += 2;
                    if (i == o1) close(qb.w);
                }
            };
            uint4 q2 = pair_at(min(2, last));
            uint4 q3 = pair_at(min(3, last));
            for (int pr = 0; pr <= last; pr += 4) {
                two_pairs(q0, q1, pr + 1 <= last);
                q0 = pair_at(min(pr + 4, last));
                q1 = pair_at(min(pr + 5, last));
                if (pr + 2 <= last) two_pairs(q2, q3, pr + 3 <= last);
                q2 = pair_at(min(pr + 6, last));
                q3 = pair_at(min(pr + 7, last));
            }
        }
        __builtin_amdgcn_s_setprio(3);
        lds_st(pn + write_at, wave_sum_lane63(n));
        __syncthreads();
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

        int s0 = 0, s1 = 0;
        if (wave < od.num_waves) {
            s0 = p.g.wave_first[od.wave_first_at + wave];
            s1 = p.g.wave_first[od.wave_first_at + wave + 1];
        }
        const int first = so[s0];
        // resident: the wave's first NSLOT slots; the slices that end there make the mask, the one
        // that straddles the limit is finished from L2
        const int nsl = min(so[s1] - first, NSLOT);
        uint64_t mask = 0;
        int sl_stream = s0;
        while (sl_stream < s1 && so[sl_stream + 1] - first <= nsl) {
            mask |= (uint64_t)1 << (so[sl_stream + 1] - 1 - first);
            ++sl_stream;
        }
        so_tab = so[max(min(sl_stream + lane, s1 - 1), 0) + 1];
        stream_end = so[s1];
        {
            const int from = first + nsl;  // even
            last = max(((stream_end - from) >> 1) - 1, 0);
            // (a wave with nothing to stream asks for its first records, unused)
            const uint64_t rb = reinterpret_cast<uint64_t>(rec_pairs(p, od, 0)) +
                                (uint64_t)((from < stream_end ? from : min(first, od.total_slots - 2)) >> 1) * 1024u;
            rbase = (global_bytes_t)(((uint64_t)(uint32_t)__builtin_amdgcn_readfirstlane((int)(rb >> 32)) << 32) |
                                     (uint32_t)__builtin_amdgcn_readfirstlane((int)rb));
            lane16 = (uint32_t)lane * 16u;
        }
        load_records<NSLOT>(p, od, lane, first, nsl, key, wr);
#pragma unroll
        for (int i = 0; i < NSLOT; ++i) {
            const uint32_t y = kY0 + (i < nsl ? y_offset(key[i]) : kYZero);
            key[i] = (key[i] & 0xffffu) | ((y - 0x10000u) << 16);
            asm volatile("" : "+v"(key[i]), "+v"(wr[i]));
        }
        {  // an equal share of the emission row for every wave, in whole groups of eight quads or values
            const int units = YREP ? P * 8 : P;
            const int share = ((units + nwaves - 1) / nwaves + 7) & ~7;
#pragma unroll
            for (int i = 0; i < YPASS; ++i) {
                // lanes past the share and shares past the row repeat the work of others
                const int q = (wave * share + (i * 64 + lane) % share) % units;
                ysrc[i] = (uint32_t)(YREP ? q >> 3 : q) * 4u;
                ydst[i] = (uint32_t)q * 16u + (uint32_t)((q >> 3) & 1) * 8u;
                yreg[i] = 0.f;
            }
        }
        keep_n = 0;
        if (tid == 0) {
            lds_st(kY0 + kYZero, 0.f);
            lds_st(kY1 + kYZero, 0.f);
        }
        if (tid < 64) lds_st(kPart + tid * 4, 0.f);
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
            if (lane == 0) lds_st(kPart + wave * 4, n);
            // rows of steps 1 (into Y0 now) and 2 (into registers); frame of step k: alpha k - 1,
            // beta T - k, kept inside the sequence
            auto frame_of = [&](int k) { return max(0, min(dir == 0 ? k - 1 : T - k, T - 1)); };
            if (T > 0) {
                e2 = (global_bytes_t)(erows + (size_t)frame_of(1) * P);
                load_y();
                store_y<kY0>();
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
        const uint32_t write_at = lane == 63 ? kPart + (uint32_t)wave * 4u : kDump + (uint32_t)lane * 4u;
        const uint32_t row4_first = (uint32_t)(s0 * 64 + lane) * 4u;
        const int sstep = dir == 0 ? 1 : -1;
        float* const sN = scalN + (dir == 0 ? 0 : T);
        float* const sS = scalS + (dir == 0 ? 0 : T);
        for (int k0 = 1; k0 <= T; k0 += kBlock) {
            const int end = min(k0 + kBlock - 1, T);
            int k = k0;
            for (; k + 1 <= end; k += 2) {
                step<1>(k - k0, leak_by, read_at, write_at, lane, mask, row4_first, nsl, sl_stream, s1,
                        first + nsl, so);
                if (k + 2 < T) e2 += estep;
                trow += tstep;
                step<0>(k + 1 - k0, leak_by, read_at, write_at, lane, mask, row4_first, nsl, sl_stream, s1,
                        first + nsl, so);
                if (k + 3 < T) e2 += estep;
                trow += tstep;
            }
            if (k <= end)
                step<1>(k - k0, leak_by, read_at, write_at, lane, mask, row4_first, nsl, sl_stream, s1,
                        first + nsl, so);
            if (wave == 0 && lane <= end - k0) {  // of the vectors that the steps read
                const float nr = __int_as_float(keep_n);
                float N, unused;
                pow2_scale(nr, &N, &unused);
                sN[(k0 - 1 + lane) * sstep] = N;
                sS[(k0 - 1 + lane) * sstep] = sconst * nr;
            }
        }

        // ---- last scalars and the closing dot product
        {
            const float nr =
                lane_value(row16_allsum(lds_ld(kPart + ((T & 1) ? 128u : 0u) + (lane & 15) * 4u)), 0);
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
                const float v = lds_ld(((T & 1) ? kX1 : 0u) + row * 4) * inv + c * p.g.vb[od.vec_at + row];
                z += p.g.vfin[od.vec_at + row] * v;
            }
            z = wave_sum_uniform(z);
            __syncthreads();  // every wave has read the partial sums
            if (lane == 0) lds_st(kPart + wave * 4, z);
            __syncthreads();
            if (tid == 0) {
                float Z = 0.f;
                for (int w = 0; w < nwaves; ++w) Z += lds_ld(kPart + w * 4);
                static_cast<float*>(p.zfin)[(size_t)dir * p.B + b] = Z;
            }
        }
    }
};

template <bool YREP, int YPASS, int LEAK, int NSLOT, bool BIG>
__global__ void __launch_bounds__(1024) k_rec_hybrid(FbParams p)
{
    extern __shared__ __align__(16) unsigned char lds_raw[];
    const RecWork work = rec_work(p);
    const int b = work.b, dir = work.dir;
    const SeqDesc sd = work.sd;
    const OrdDesc od = work.od;
    RecHybrid<YREP, YPASS, LEAK, NSLOT, BIG> r;
    r.run(p, sd, od, b, dir);
    finish_sequence<float>(p, b, lds_raw);
}

#define LFMMI_HYBRID(YREP, YPASS, LEAK, MAP)                                                        \
    {0, kHybridSlots, YREP, LEAK, 1024, k_rec_hybrid<YREP != 0, YPASS, LEAK, kHybridSlots, MAP == 2>, MAP, 0, 0, YPASS}
const RecVariant kHybridVariants[] = {
    LFMMI_HYBRID(1, 1, 0, 1), LFMMI_HYBRID(1, 2, 0, 1), LFMMI_HYBRID(0, 3, 0, 1), LFMMI_HYBRID(0, 3, 0, 2),
    LFMMI_HYBRID(1, 1, 2, 1), LFMMI_HYBRID(1, 2, 2, 1), LFMMI_HYBRID(0, 3, 2, 1), LFMMI_HYBRID(0, 3, 2, 2),
};
#undef LFMMI_HYBRID

}  // namespace

const RecVariant* hybrid_variants(int* n)
{
    *n = (int)(sizeof kHybridVariants / sizeof kHybridVariants[0]);
    return kHybridVariants;
}

const RecVariant* find_hybrid(bool yrep, int leak, int num_pdfs, int map)
{
    const int units = yrep ? num_pdfs * 8 : num_pdfs;
    for (const RecVariant& v : kHybridVariants)
        if (v.yrep == (yrep ? 1 : 0) && v.leak == leak && v.hybrid == map && units <= v.ypass * 1024) return &v;
    return nullptr;
}

}  // namespace lfmmi
