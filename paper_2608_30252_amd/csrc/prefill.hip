// prefill.hip -- memory-prefill attention: the draft's one masked pass over a
// prefix that builds its initial compact memory (Sec. 3.3 prefill; the
// appendix on memory prefill).
//
// The prefill mask applies the same write policy as decoding, so every query
// of the pass attends exactly the set it would attend during decoding:
//   raw token at position p : sinks [0, min(S, p+1)), the slots materialised
//                             in passes of earlier tokens (1 .. slots_after(p)),
//                             and the window [max(S, p-W+1), p];
//   memory slot g_m         : the sinks, slots 1..m (itself included) and the
//                             W raw tokens before its position id b_m = S + m r:
//                             [max(S, b_m - W), b_m - 1].
// Keys come from two places: the memory segment (sinks in rows 0..S-1, slot m
// in row S + m - 1) and the prefix's raw K/V (position x in row x).  For every
// query the visible keys are one prefix of the memory segment, [0, mem_hi),
// and one interval of raw rows, [raw_lo, raw_hi).
//
// Both products run on the matrix cores (v_mfma_f32_16x16x32_bf16, fp32
// accumulation).  A workgroup of four waves owns one (sequence, KV head) unit
// and a block of query tokens; its rows are (token, query head of the GQA
// group) pairs in 16-token blocks, each wave holding NB of them with their
// query fragments in registers for the whole pass.  Keys stream in 64-key
// tiles through two LDS stages, the next tile's direct loads
// (global_load_lds_dwordx4) in flight while one is used:
//   * K rows land with their 16-byte chunks XOR-swizzled so the A operand reads
//     of S^T = K Q^T are conflict-free; the A rows are permuted so that each
//     lane's S^T accumulators hold the 8 consecutive keys that the PV product's
//     B operand needs (no shuffle of probabilities);
//   * V rows land as they are (16-byte chunks XOR-swizzled by row), and the A
//     operand of O^T = V^T P^T -- 8 consecutive keys of one feature -- comes
//     from two transposing LDS reads (ds_read_b64_tr_b16: lane 4e + a of a
//     16-lane group names features 4a .. 4a+3 of key row e, and lane 4a + b
//     receives feature 4a + b of the four rows);
//   * online softmax per query row without a running maximum: probabilities are
//     taken against the row's reference maximum as it stands, and only when a
//     lane's sum of 8 exceeds 16 (some row has outgrown its reference by 2 .. 16
//     times) do the maxima move, o and l rescale and the step's probabilities
//     get taken again.  Masks apply in place, on the tiles that are not inside
//     every row's range; one barrier per tile.
// What bounds it at d 64: vector issue.  A 64-key tile of a wave takes 32 matrix
// products, 32 fma, 32 exponentials (four issue slots each), 32 adds and 16
// conversions, and nothing else of weight: no maxima (a fifth of the vector work
// before), no address arithmetic (stage and half are instruction offsets), no
// staging registers (128 registers: four waves per SIMD instead of three).
// 32K prefix, 32/8 heads, 2048 slots: 785 -> 627 us; 4 ragged prefixes at d 128,
// W 128: 492 -> 406 us (two waves per SIMD there: latency-bound); one of 330
// tokens at d 128: 18.1 -> 16.2.  Measured
// and not kept: 64 rows per wave (685 us against 703 on long windows, but twice the time
// with one query head per KV head), 32-key tiles in three stages at d 128 (419 - 426).
// Query blocks of every unit are dealt round-robin over the units (with a
// multiple of 8 units all blocks of one KV head share an XCD and its L2), the
// heaviest blocks first.
#include <type_traits>

#include "mad_device.h"
#include "mad_internal.h"

namespace mad {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_v;
typedef __attribute__((ext_vector_type(4))) float f32x4_v;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_v;

template <int D>
struct PrefillCfg {
    static constexpr int KT = 64;                     // keys per tile (128 spills registers at d 64)
    static constexpr int KH = KT / 32;                 // 32-key halves of a tile
    static constexpr int RB = D * 2;                   // bytes per K row
    static constexpr int CPR = RB / 16;                // 16-byte chunks per K row
    static constexpr int KTILE = KT * RB;              // K tile bytes
    static constexpr int STAGE = 2 * KTILE;            // K tile + V tile (same size)
    static constexpr int SMEM = 2 * STAGE;
    static constexpr int LPW = KTILE / 1024 / 4;       // K (and V) loads per wave per tile
};

typedef short v4s_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4s_t lds_read_tr16(const unsigned char *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s_t *)(p));
}

// Lanes l, l^16, l^32, l^48 hold the same query row.  v_permlane16_swap and
// v_permlane32_swap (VALU lane swaps, no LDS round trip) give every lane the
// values of lanes l & ~16 and l | 16 (resp. 32), so two swaps reduce over the four.
__device__ __forceinline__ float prefill_row_max(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1]));
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float prefill_row_sum(float v) {
    const auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = __uint_as_float(a[0]) + __uint_as_float(a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

constexpr float kLazySum = 16.f;  // rescale threshold of the online softmax: a lane's sum of 8 probabilities
constexpr float kNoMax = 3e38f;   // minus the reference maximum (log2 units) of a row without keys: 2^(s + this) overflows

// the largest value of the wave, wave-uniform: lane swaps on the vector ALU (six
// rounds of LDS shuffles took 1 us of a workgroup's prologue)
__device__ __forceinline__ int wave_max_i32(int v) {
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0xB1, 0xF, 0xF, true));    // quad_perm [1, 0, 3, 2]
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0x4E, 0xF, 0xF, true));    // quad_perm [2, 3, 0, 1]
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0x141, 0xF, 0xF, true));   // row_half_mirror
    v = max(v, __builtin_amdgcn_mov_dpp(v, 0x140, 0xF, 0xF, true));   // row_mirror
    const auto a = __builtin_amdgcn_permlane16_swap((unsigned)v, (unsigned)v, false, false);
    v = max((int)a[0], (int)a[1]);
    const auto b = __builtin_amdgcn_permlane32_swap((unsigned)v, (unsigned)v, false, false);
    return __builtin_amdgcn_readfirstlane(max((int)b[0], (int)b[1]));
}

__device__ __forceinline__ int prefill_slots_after(int t, int S, int ru, int u) {
    return t <= S ? 0 : (t - S) / ru * u;
}

// Occupancy: four waves per SIMD at head_dim 64 (128 registers), two at 128.
template <int D, int G, int NB>
__global__ __launch_bounds__(256, D == 64 ? 4 : 2) void prefill_kernel(const PrefillArgs a) {
    using C = PrefillCfg<D>;
    constexpr int KST = D / 32, DB = D / 16;
    constexpr int TBW = 4 * NB / G;   // 16-token blocks per workgroup
    constexpr int QT = 16 * TBW;      // query tokens per workgroup
    static_assert(4 * NB % G == 0, "row blocks cover whole token blocks");
    extern __shared__ __align__(16) unsigned char smem[];

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lg = lane >> 4;
    const int unit = blockIdx.x % a.units;
    const int qb = a.nrb + a.nsb - 1 - (int)(blockIdx.x / a.units);   // slot blocks, then raw blocks, late first
    const int b = unit / a.Hkv, c = unit - b * a.Hkv;
    const bool slot_kind = qb >= a.nrb;
    const int S = a.S, W = a.W, r = a.r, u = a.u, ru = a.r * a.u;
    const int nq = slot_kind ? a.Mtot[b] : a.P[b];
    const int q0 = (slot_kind ? qb - a.nrb : qb) * QT;   // first token: raw position, or slot index - 1
    if (q0 >= nq) return;                                 // the whole workgroup: no barrier crossed
    const int qlast = min(nq, q0 + QT) - 1;

    // ---- the workgroup's key ranges: the union of its rows' ranges ----
    int mem_hi, raw_lo, raw_hi;
    if (!slot_kind) {
        mem_hi = qlast < S ? qlast + 1 : S + prefill_slots_after(qlast, S, ru, u);
        raw_lo = max(S, q0 - W + 1);
        raw_hi = qlast + 1;
    } else {
        mem_hi = S + qlast + 1;
        raw_lo = max(S, S + (q0 + 1) * r - W);
        raw_hi = S + (qlast + 1) * r;
    }
    if (raw_hi < raw_lo) raw_hi = raw_lo;
    const int n_mem_t = (mem_hi + C::KT - 1) / C::KT;
    const int nt = n_mem_t + (raw_hi - raw_lo + C::KT - 1) / C::KT;

    const bf16_t *mk = reinterpret_cast<const bf16_t *>(a.mk) + b * a.m_seq + c * a.m_head;
    const bf16_t *mv = reinterpret_cast<const bf16_t *>(a.mv) + b * a.m_seq + c * a.m_head;
    const bf16_t *rk = reinterpret_cast<const bf16_t *>(a.rk) + b * a.r_seq + c * a.r_head;
    const bf16_t *rv = reinterpret_cast<const bf16_t *>(a.rv) + b * a.r_seq + c * a.r_head;
    // ---- tile loader: direct loads into LDS, the next tile's into the idle stage ----
    auto tile_base = [&](int t, bool &is_mem, int &end) -> int {
        is_mem = t < n_mem_t;
        if (is_mem) {
            end = mem_hi;
            return t * C::KT;
        }
        end = raw_hi;
        return raw_lo + (t - n_mem_t) * C::KT;
    };
    // Wave load inst = LPW wave + j brings 1 KB: lane l's LDS slot is chunk cidx % CPR of row cidx / CPR
    // (cidx = 64 inst + l), which holds the row's chunk slot ^ swizzle(row).  A pair's second load adds
    // 1024 to both of its addresses (an instruction offset), so its lane offset leaves that out.
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    uint32_t k_off[C::LPW], v_off[C::LPW];
    #pragma unroll
    for (int j = 0; j < C::LPW; ++j) {
        const int cidx = (wave * C::LPW + j) * 64 + lane, row = cidx / C::CPR, slot = cidx % C::CPR;
        k_off[j] = row * C::RB + ((slot ^ k_swz<D>(row)) << 4) - 1024 * (j & 1);
        v_off[j] = row * C::RB + ((slot ^ v_swz<D>(row)) << 4) - 1024 * (j & 1);
    }
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_addr(smem)) + wv * C::LPW * 1024;
    auto load_tile = [&](int t, auto stage_const) {
        constexpr int ST = decltype(stage_const)::value * C::STAGE;
        bool is_mem;
        int end;
        const int base = tile_base(t, is_mem, end);
        const bf16_t *ks = (is_mem ? mk : rk) + (size_t)base * D, *vs = (is_mem ? mv : rv) + (size_t)base * D;
        if (base + C::KT <= end) {
            #pragma unroll
            for (int j = 0; j < C::LPW; j += 2) {
                lds_stream16_x2<false>(ks, k_off[j], k_off[j + 1], lds0 + ST + j * 1024);
                lds_stream16_x2<false>(vs, v_off[j], v_off[j + 1], lds0 + ST + C::KTILE + j * 1024);
            }
        } else {
            // rows past the range load a valid row (masked): the pair's offsets from 1 KB before the base, so
            // that neither is negative once its row is clamped
            const unsigned char *k1 = reinterpret_cast<const unsigned char *>(ks) - 1024;
            const unsigned char *v1 = reinterpret_cast<const unsigned char *>(vs) - 1024;
            uint32_t ko[C::LPW], vo[C::LPW];
            #pragma unroll
            for (int j = 0; j < C::LPW; ++j) {
                const int cidx = (wave * C::LPW + j) * 64 + lane, row = cidx / C::CPR, slot = cidx % C::CPR;
                const uint32_t at = min(row, end - 1 - base) * C::RB + ((j & 1) ? 0 : 1024);
                ko[j] = at + ((slot ^ k_swz<D>(row)) << 4);
                vo[j] = at + ((slot ^ v_swz<D>(row)) << 4);
            }
            #pragma unroll
            for (int j = 0; j < C::LPW; j += 2) {
                lds_stream16_x2<false>(k1, ko[j], ko[j + 1], lds0 + ST + j * 1024);
                lds_stream16_x2<false>(v1, vo[j], vo[j + 1], lds0 + ST + C::KTILE + j * 1024);
            }
        }
    };

    load_tile(0, std::integral_constant<int, 0>());   // in flight while the queries are read

    const bf16_t *qbase = reinterpret_cast<const bf16_t *>(slot_kind ? a.q_slot : a.q_raw) +
                          (size_t)b * (slot_kind ? a.slot_cap : a.q_cap) * a.Hq * D;

    // ---- this lane's rows: query fragments and visible ranges ----
    bf16x8_v qf[NB][KST];
    int m_lim[NB], r_lo[NB], r_hi[NB];
    #pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int j = wave + 4 * i, g = j % G, tb = j / G;
        const int tok = q0 + tb * 16 + lr;
        if (tok <= qlast) {
            const bf16_t *qrow = qbase + ((size_t)tok * a.Hq + c * G + g) * D;
            #pragma unroll
            for (int ks = 0; ks < KST; ++ks) qf[i][ks] = *reinterpret_cast<const bf16x8_v *>(qrow + ks * 32 + 8 * lg);
            if (!slot_kind) {
                m_lim[i] = tok < S ? tok + 1 : S + prefill_slots_after(tok, S, ru, u);
                r_lo[i] = max(S, tok - W + 1);
                r_hi[i] = tok < S ? r_lo[i] : tok + 1;
            } else {
                const int bm = S + (tok + 1) * r;
                m_lim[i] = S + tok + 1;
                r_lo[i] = max(S, bm - W);
                r_hi[i] = bm;
            }
        } else {
            #pragma unroll
            for (int ks = 0; ks < KST; ++ks) qf[i][ks] = bf16x8_v{0, 0, 0, 0, 0, 0, 0, 0};
            m_lim[i] = 0;
            r_lo[i] = r_hi[i] = 0;
        }
    }

    // the wave's tiles without a mask: the tightest of its rows' ranges
    int mem_full = m_lim[0], lo_full = r_lo[0], hi_full = r_hi[0];
    #pragma unroll
    for (int i = 1; i < NB; ++i) {
        mem_full = min(mem_full, m_lim[i]);
        lo_full = max(lo_full, r_lo[i]);
        hi_full = min(hi_full, r_hi[i]);
    }
    mem_full = -wave_max_i32(-mem_full);
    lo_full = wave_max_i32(lo_full);
    hi_full = -wave_max_i32(-hi_full);

    f32x4_v o[DB][NB];
    // per row: the reference maximum (unscaled scores), minus it in log2 units, the running sum
    float m_run[NB], nms[NB], l_run[NB];
    #pragma unroll
    for (int i = 0; i < NB; ++i) {
        m_run[i] = -INFINITY;
        nms[i] = kNoMax;
        l_run[i] = 0.f;
        #pragma unroll
        for (int db = 0; db < DB; ++db) o[db][i] = f32x4_v{0.f, 0.f, 0.f, 0.f};
    }
    const float cs = a.scale_log2;

    // LDS offsets of this lane's operand reads within a stage (the half of the tile and the second
    // row of a V pair are instruction offsets)
    int k_at[2][KST], v_at[DB];
    #pragma unroll
    for (int blk = 0; blk < 2; ++blk) {
        const int kr = 8 * (lr >> 2) + 4 * blk + (lr & 3);
        #pragma unroll
        for (int ks = 0; ks < KST; ++ks) k_at[blk][ks] = kr * C::RB + (((4 * ks + lg) ^ k_swz<D>(kr)) << 4);
    }
    #pragma unroll
    for (int db = 0; db < DB; ++db) {
        const int r0 = 8 * lg + (lr >> 2), byte = db * 32 + 8 * (lr & 3);
        v_at[db] = C::KTILE + r0 * C::RB + (((byte >> 4) ^ v_swz<D>(r0)) << 4) + (byte & 8);
    }

    auto compute = [&](int t, auto stage_const) {
        const unsigned char *st = smem + decltype(stage_const)::value * C::STAGE;
        bool is_mem;
        int end;
        const int base = tile_base(t, is_mem, end);
        const bool full = is_mem ? base + C::KT <= mem_full : base >= lo_full && base + C::KT <= min(hi_full, end);
        #pragma unroll
        for (int h = 0; h < C::KH; ++h) {
            // S^T = K Q^T for keys 32h .. 32h+31 of the tile: A row m of block blk is key
            // 32h + 8(m/4) + 4 blk + m%4, so accumulator element e&3 of block e>>2 in lane
            // group lg is key 32h + 8 lg + e
            f32x4_v sacc[2][NB];
            #pragma unroll
            for (int blk = 0; blk < 2; ++blk) {
                bf16x8_v kf[KST];
                #pragma unroll
                for (int ks = 0; ks < KST; ++ks)
                    kf[ks] = *reinterpret_cast<const bf16x8_v *>(st + k_at[blk][ks] + h * 32 * C::RB);
                #pragma unroll
                for (int i = 0; i < NB; ++i) {
                    sacc[blk][i] = f32x4_v{0.f, 0.f, 0.f, 0.f};
                    #pragma unroll
                    for (int ks = 0; ks < KST; ++ks)
                        sacc[blk][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[ks], qf[i][ks], sacc[blk][i], 0, 0, 0);
                }
            }
            if (!full) {
                // edge tile: element e is key base + 32h + 8lg + e; mask in place
                #pragma unroll
                for (int i = 0; i < NB; ++i) {
                    const int lo = is_mem ? 0 : r_lo[i], hi = min(end, is_mem ? m_lim[i] : r_hi[i]);
                    const int k0 = base + 32 * h + 8 * lg, a0 = lo - k0, b0 = hi - k0;
                    #pragma unroll
                    for (int e = 0; e < 8; ++e) {
                        const bool ok = (e >= a0) & (e < b0);   // no short circuit: straight-line selects
                        sacc[e >> 2][i][e & 3] = ok ? sacc[e >> 2][i][e & 3] : -INFINITY;
                    }
                }
            }
            // Probabilities against the reference maximum as it stands, p = 2^(s c - m c): one fma into the
            // exponential, and no maximum is taken.  A lane's sum above kLazySum (or a NaN) says that
            // some row has outgrown its reference: only then the maxima move, o and l are rescaled and the
            // probabilities taken again.  Rows that saw no key yet have a reference that any score outgrows.
            float ps[NB];
            uint32_t pk[NB][4];
            auto probabilities = [&](int i) {
                float p[8];
                #pragma unroll
                for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(sacc[e >> 2][i][e & 3], cs, nms[i]));
                ps[i] = ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
                #pragma unroll
                for (int e = 0; e < 4; ++e) pk[i][e] = cvt_pk_bf16(p[2 * e], p[2 * e + 1]);
            };
            bool grown = false;
            #pragma unroll
            for (int i = 0; i < NB; ++i) {
                probabilities(i);
                grown |= !(ps[i] <= kLazySum);
            }
            if (__any(grown)) {
                #pragma unroll
                for (int i = 0; i < NB; ++i) {
                    float mt = -INFINITY;
                    #pragma unroll
                    for (int e = 0; e < 8; ++e) mt = fmaxf(mt, sacc[e >> 2][i][e & 3]);
                    const float mn = fmaxf(m_run[i], prefill_row_max(mt));
                    const float alpha = mn == m_run[i] ? 1.f : __builtin_amdgcn_exp2f((m_run[i] - mn) * cs);
                    m_run[i] = mn;
                    nms[i] = mn == -INFINITY ? kNoMax : -mn * cs;
                    l_run[i] *= alpha;
                    #pragma unroll
                    for (int db = 0; db < DB; ++db) o[db][i] *= alpha;
                    probabilities(i);
                }
            }
            bf16x8_v pf[NB];
            #pragma unroll
            for (int i = 0; i < NB; ++i) {
                l_run[i] += ps[i];
                pf[i] = __builtin_bit_cast(bf16x8_v, u32x4_v{pk[i][0], pk[i][1], pk[i][2], pk[i][3]});
            }
            // O^T += V^T P^T: A = V^T rows (features db*16 + lr), keys 32h + 8 lg .. +7,
            // from the transposing reads of key rows 32h + 8 lg + {0..3} and {4..7}
            #pragma unroll
            for (int db = 0; db < DB; ++db) {
                const v4s_t lo = lds_read_tr16(st + v_at[db] + h * 32 * C::RB);
                const v4s_t hi = lds_read_tr16(st + v_at[db] + (h * 32 + 4) * C::RB);
                const bf16x8_v vf = __builtin_bit_cast(bf16x8_v, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
                #pragma unroll
                for (int i = 0; i < NB; ++i) o[db][i] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf, pf[i], o[db][i], 0, 0, 0);
            }
        }
    };

    // The loads of tile t + 1 go out before tile t is used and have landed by its end (the waits are
    // explicit: the compiler does not count direct loads).  Two tiles a round, so that every LDS
    // address has its stage as a constant.
    wait_vm(0);
    __syncthreads();
    for (int t = 0; t < nt; t += 2) {
        if (t + 1 < nt) load_tile(t + 1, std::integral_constant<int, 1>());
        compute(t, std::integral_constant<int, 0>());
        if (t + 1 >= nt) break;
        wait_vm(0);
        __syncthreads();
        if (t + 2 < nt) load_tile(t + 2, std::integral_constant<int, 0>());
        compute(t + 1, std::integral_constant<int, 1>());
        wait_vm(0);
        __syncthreads();
    }

    // ---- normalise and store: lane (lr, lg) holds features db*16 + 4 lg .. +3 of row lr ----
    bf16_t *obase = reinterpret_cast<bf16_t *>(slot_kind ? a.o_slot : a.o_raw) +
                    (size_t)b * (slot_kind ? a.slot_cap : a.q_cap) * a.Hq * D;
    float *lbase = slot_kind ? a.lse_slot : a.lse_raw;
    #pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int j = wave + 4 * i, g = j % G, tb = j / G;
        const int tok = q0 + tb * 16 + lr;
        const float lt = prefill_row_sum(l_run[i]);
        if (tok > qlast) continue;
        const float inv = lt > 0.f ? 1.f / lt : 0.f;
        const size_t head = (size_t)tok * a.Hq + c * G + g;
        #pragma unroll
        for (int db = 0; db < DB; ++db) {
            const f32x4_v v = o[db][i];
            *reinterpret_cast<uint2 *>(obase + head * D + db * 16 + 4 * lg) =
                make_uint2(cvt_pk_bf16(v[0] * inv, v[1] * inv), cvt_pk_bf16(v[2] * inv, v[3] * inv));
        }
        if (lbase && lg == 0)
            lbase[(size_t)b * (slot_kind ? a.slot_cap : a.q_cap) * a.Hq + head] =
                lt > 0.f ? (m_run[i] * a.scale_log2 + log2f(lt)) * kLn2 : -INFINITY;
    }
}

// ------------------------------------------------------------------ host ----

// 16-row blocks per wave (two workgroups per CU)
static constexpr int prefill_nb(int) { return 2; }

int prefill_tokens_per_block(int d, int G) { return 16 * 4 * prefill_nb(d) / G; }

template <int D, int G>
static hipError_t launch_t(const PrefillArgs &a, hipStream_t st) {
    using C = PrefillCfg<D>;
    constexpr int NB = prefill_nb(D);
    dim3 grid((unsigned)(a.units * (a.nrb + a.nsb))), block(256);
    hipLaunchKernelGGL((prefill_kernel<D, G, NB>), grid, block, C::SMEM, st, a);
    return hipGetLastError();
}

template <int D>
static hipError_t launch_g(const PrefillArgs &a, int G, hipStream_t st) {
    switch (G) {
        case 1: return launch_t<D, 1>(a, st);
        case 2: return launch_t<D, 2>(a, st);
        case 4: return launch_t<D, 4>(a, st);
        case 8: return launch_t<D, 8>(a, st);
    }
    return hipErrorInvalidValue;
}

hipError_t launch_prefill(const PrefillArgs &a, int d, int G, hipStream_t st) {
    if (d == 64) return launch_g<64>(a, G, st);
    if (d == 128) return launch_g<128>(a, G, st);
    return hipErrorInvalidValue;
}

}  // namespace mad
