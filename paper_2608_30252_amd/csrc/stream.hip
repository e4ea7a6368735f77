// stream.hip -- bandwidth-bound bf16 attention over long key/value streams: the
// target's (gamma+1)-query verify attention over its full KV cache (Sec. 2.1
// draft-verify paradigm; Sec. 3.3: the verifier keeps the full KV), query t of
// the T = gamma+1 new tokens seeing rows 0 .. len-T+t.  Also the draft's decode
// attention (decode.hip) where its launch is long or has many query heads per
// KV head (T = 1; a row's keys are its memory, its window ring and the new
// token, which is appended).
//
// Work decomposition.  A unit is one (sequence, KV head); its query tile is the
// T*G rows (t, g) -> row t*G + g, padded to 16-row blocks.  The keys of every
// unit are cut into slabs (32 KB of K + V), and the slabs of all units, in unit
// order, are dealt to one workgroup per CU in equal contiguous runs.  Ragged
// batches therefore keep every CU busy to the end: with a fixed number of
// splits per unit, sized by the longest sequence, 16 sequences of 600 .. 12000
// keys ran at 3.5 TB/s.  A run covers whole units, the tail of its first unit
// and the head of its last; whole units are finished by their workgroup,
// small pieces of a unit are merged by the last workgroup to arrive at it (one
// arrival counter per unit), so such a call is a single launch; where a unit
// has many or large pieces a second launch merges them (plan_stream).
//
// Both products run on the matrix cores (v_mfma_f32_16x16x32_bf16, fp32
// accumulation):
//   * S^T = K Q^T takes K rows as the A operand.  Key rows are assigned to the
//     A rows with a fixed permutation so that the S^T accumulator already holds,
//     in every lane, the 8 consecutive keys that the next product needs;
//   * O^T = V^T P^T takes its A operand (8 consecutive keys of one feature)
//     either from V rows of d features (two transposing LDS reads,
//     ds_read_b64_tr_b16) or from a key-contiguous V^T cache (one run of cap
//     keys per feature); the probabilities come from the lane's own scores
//     (rounded to bf16);
//   * online softmax per query row: the row's 8 scores of a 32-key step sit in
//     one lane, the row max needs two cross-lane exchanges.
// The eight waves share a four-stage LDS ring of slabs filled by direct loads
// (global_load_lds_dwordx4, issued by all waves), so 96 KB are in flight per
// CU.  Wave w < KS*NB owns 16-row block w % NB and key group w / NB of every
// slab; consecutive waves -- on different SIMDs -- take different row blocks,
// and one wave's exponentials overlap another's matrix products.  K rows land
// with their 16-byte chunks XOR-swizzled by row (k_swz, v_swz), V^T rows by
// feature, so every operand read is conflict-free.  The ring runs on
// across units: the next unit's slabs and its query rows (direct loads into a
// small LDS area, older than the unit's first slab) are in flight while the
// current unit finishes.
#include <type_traits>

#include "mad_device.h"
#include "mad_internal.h"

namespace mad {

// phase marks of the diagnostic trace build: 0 entry, 1 the run's last slab done and,
// where the launch merges, 2 its pieces acknowledged, 3 the arrivals known, 4 merged
MAD_TRACE_BUFFER(mad_trace_verify)

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8_v;
typedef __attribute__((ext_vector_type(4))) float f32x4_v;
typedef __attribute__((ext_vector_type(4))) unsigned int u32x4_v;

// Lanes l, l^16, l^32, l^48 hold the same query row: two lane swaps reduce over the four.
__device__ __forceinline__ float max_over_row_lanes(float v) { return pair_max<32>(pair_max<16>(v)); }
__device__ __forceinline__ float sum_over_row_lanes(float v) { return pair_sum<32>(pair_sum<16>(v)); }

template <int D, int NB>
struct StreamCfg {
    static constexpr int SLAB = stream_slab(D);            // keys per slab
    static constexpr int RB = D * 2;                       // bytes per K (and V) row
    static constexpr int CPR = D / 8;                      // 16-byte chunks per row
    static constexpr int KBYTES = SLAB * RB;               // K bytes per slab (= V bytes)
    static constexpr int STAGE = 2 * KBYTES;
    static constexpr int NST = 4;                          // ring stages
    static constexpr int NWV = 8;                          // waves
    static constexpr int IPW = STAGE / 1024 / NWV;         // direct loads per wave per slab
    static constexpr int RP = NB * 16;                     // padded query rows
    static constexpr int KS = SLAB / 32 < NWV / NB ? SLAB / 32 : (NWV / NB >= 4 ? 4 : 2);   // key groups of a slab
    static constexpr int KPG = SLAB / KS;                  // keys per group: 32, or 64 in two steps
    static constexpr int VROW = SLAB * 2, VCH = SLAB / 8;  // bytes and chunks of a V^T row in a stage
    static constexpr int QBYTES = RP * RB;
    static constexpr int QSLOTS = RP * RB >= 16384 ? 1 : 2;   // query areas (LDS holds one at 64 rows, d 128)
    static constexpr int OFF_Q = NST * STAGE;
    static constexpr int OFF_ML = OFF_Q + QSLOTS * QBYTES;
    static constexpr int SMEM = OFF_ML + KS * RP * 8;
    static constexpr int XPASS = KS * RP * D * 4 > STAGE ? 2 : 1;   // passes of the key groups' exchange through one stage
    static_assert((NST * STAGE & (NST * STAGE - 1)) == 0 && IPW % 2 == 0 && KS * NB <= NWV && KPG % 32 == 0, "waves");
    static_assert(KS * RP * D * 4 <= XPASS * STAGE, "the key groups' exchange fits one stage");
    static_assert(SMEM + 2 * MAD_MAX_VERIFY_ROWS * 4 + 64 <= 160 * 1024, "LDS, with the kernel's static arrays");
};

typedef short v4s_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ v4s_t lds_read_tr16(const unsigned char *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s_t *)(p));
}

// The kernel arguments, read at entry in one batch (one wait) and kept: left to
// the compiler they are read in dependent rounds where they are used, each a
// miss to host memory once the key stream has swept the L2.  The row records
// come in the same batch, one per lane, and are taken from there by readlane.
struct StreamCtx {
    uint64_t q, k, v, out, lse, part, counters;
    int64_t seq, head;
    float cs;
    int cap, Hq, Hkv, G, T, base, rem, by_unit, merge2, rows, wgs;   // rows, wgs: slabs and (by_unit) workgroups of one KV head over all rows
    int4 rec;   // lane b: row b's record
    __device__ __forceinline__ int tile0(int b) const { return __builtin_amdgcn_readlane(rec.w, b); }
    __device__ __forceinline__ int slabs(int b) const { return (b == kMaxB - 1 ? rows : tile0(b + 1)) - tile0(b); }
    __device__ __forceinline__ int wg0(int b) const { return __builtin_amdgcn_readlane(rec.z, b); }
    __device__ __forceinline__ int splits(int b) const { return (b == kMaxB - 1 ? wgs : wg0(b + 1)) - wg0(b); }
    __device__ __forceinline__ int len(int b) const { return __builtin_amdgcn_readlane(rec.x, b); }
};
__device__ __forceinline__ StreamCtx load_ctx(const StreamArgs &a) {
    StreamCtx x;
    x.rec = a.row[threadIdx.x & 63];
    x.q = ptr_bits(a.q); x.k = ptr_bits(a.k); x.v = ptr_bits(a.v); x.out = ptr_bits(a.out); x.lse = ptr_bits(a.lse);
    x.part = ptr_bits(a.part); x.counters = ptr_bits(a.counters);
    x.seq = a.seq; x.head = a.head;
    x.cs = a.scale_log2;
    x.cap = a.cap; x.Hq = a.Hq; x.Hkv = a.Hkv; x.G = a.G; x.T = a.T; x.base = a.base; x.rem = a.rem;
    x.by_unit = a.by_unit; x.merge2 = a.merge2; x.rows = a.rows; x.wgs = a.wgs;
    asm volatile("" : "+s"(x.q), "+s"(x.k), "+s"(x.v), "+s"(x.out), "+s"(x.lse), "+s"(x.part),
                 "+s"(x.counters), "+s"(x.seq), "+s"(x.head), "+s"(x.cs));
    asm volatile("" : "+s"(x.cap), "+s"(x.Hq), "+s"(x.Hkv), "+s"(x.G), "+s"(x.T), "+s"(x.base), "+s"(x.rem),
                 "+s"(x.by_unit), "+s"(x.merge2), "+s"(x.rows), "+s"(x.wgs));
    return x;
}

// The draft's window ring and new token, and per lane the ring start and the
// new-token mode of row `lane` (rec.x is then the row's memory length, rec.y
// its window length).
struct DraftCtx {
    uint64_t wk, wv, kn, vn;
    int64_t seq, head;
    int cap;
    int2 rec;
    __device__ __forceinline__ int start(int b) const { return __builtin_amdgcn_readlane(rec.x, b); }
    __device__ __forceinline__ int mode(int b) const { return __builtin_amdgcn_readlane(rec.y, b); }
};
__device__ __forceinline__ DraftCtx load_draft(const StreamArgs &a) {
    DraftCtx x;
    x.rec = a.ring[threadIdx.x & 63];
    x.wk = ptr_bits(a.wk); x.wv = ptr_bits(a.wv); x.kn = ptr_bits(a.kn); x.vn = ptr_bits(a.vn);
    x.seq = a.w_seq; x.head = a.w_head; x.cap = a.w_cap;
    asm volatile("" : "+s"(x.wk), "+s"(x.wv), "+s"(x.kn), "+s"(x.vn), "+s"(x.seq), "+s"(x.head), "+s"(x.cap));
    return x;
}

// where unit u's pieces are: np of them, the first numbered p0
struct UnitPieces {
    int p0, np;
};
__device__ __forceinline__ UnitPieces unit_pieces(const StreamCtx &a, int u) {
    const int b = u / a.Hkv, c = u - b * a.Hkv;
    if (a.by_unit) {
        const int k = a.splits(b);
        return {a.Hkv * a.wg0(b) + c * k + u, k};
    }
    const int nt = a.slabs(b), s0 = a.Hkv * a.tile0(b) + c * nt, w0 = stream_owner(s0, a.base, a.rem);
    return {w0 + u, stream_owner(s0 + nt - 1, a.base, a.rem) - w0 + 1};
}

// A piece in the workspace: [R][D] unnormalised o, [R] (max in log2 units, sum),
// padded to 16 bytes.
__host__ __device__ constexpr int piece_floats(int R, int d) { return (R * (d + 2) + 3) & ~3; }

__device__ __forceinline__ size_t out_head(const StreamCtx &a, int u, int row) {
    const int b = u / a.Hkv, c = u - b * a.Hkv, tt = row / a.G;
    return ((size_t)b * a.T + tt) * a.Hq + (size_t)c * a.G + (row - tt * a.G);
}

// Log-sum-exp merge of the nr rows of unit u from its np pieces as they lie in
// LDS, by a workgroup of 512 threads: eight lanes per row turn the pieces'
// (max, sum) into weights, then (behind a barrier) one thread per feature quad.
// Piece p's o rows are at so + p * po bytes, its (max, sum) pairs at sm + p * po.
template <int D>
struct MergeJob {
    int u, np, nr;
    unsigned char *so, *sm;
    int po;
    float *sinv;   // [nr]

    __device__ __forceinline__ void weights(const StreamCtx &a) const {
        for (int r = threadIdx.x >> 3; r < nr; r += 64) {
            const int l8 = threadIdx.x & 7;
            float M = -INFINITY, L = 0.f;
            for (int p = l8; p < np; p += 8) M = fmaxf(M, reinterpret_cast<const float2 *>(sm + p * po)[r].x);
            M = group_max<8>(M);
            const float mr = M == -INFINITY ? 0.f : M;
            for (int p = l8; p < np; p += 8) {
                float2 *v = reinterpret_cast<float2 *>(sm + p * po) + r;
                const float wt = __builtin_amdgcn_exp2f(v->x - mr);
                L = fmaf(wt, v->y, L);
                v->x = wt;
            }
            L = group_sum<8>(L);
            if (l8 == 0) {
                sinv[r] = L > 0.f ? 1.f / L : 0.f;
                if (a.lse) bits_ptr<float>(a.lse)[out_head(a, u, r)] = L > 0.f ? (M + log2f(L)) * kLn2 : -INFINITY;
            }
        }
    }
    __device__ __forceinline__ void sums(const StreamCtx &a) const {
        for (int x = threadIdx.x; x < nr * (D / 4); x += 512) {   // feature quad x % (D / 4) of row x / (D / 4)
            const int r = x / (D / 4);
            f32x4_v y = f32x4_v{0.f, 0.f, 0.f, 0.f};
            #pragma unroll 8
            for (int p = 0; p < np; ++p) {
                const f32x4_v v = *reinterpret_cast<const f32x4_v *>(so + p * po + x * 16);
                const float wt = reinterpret_cast<const float2 *>(sm + p * po)[r].x;
                #pragma unroll
                for (int e = 0; e < 4; ++e) y[e] = fmaf(wt, v[e], y[e]);
            }
            const float inv = sinv[r];
            *reinterpret_cast<uint2 *>(bits_ptr<bf16_t>(a.out) + out_head(a, u, r) * D + (x % (D / 4)) * 4) =
                make_uint2(pack_bf16x2(y[0] * inv, y[1] * inv), pack_bf16x2(y[2] * inv, y[3] * inv));
        }
    }
};

// `bytes` (a multiple of 16) of pieces straight into LDS, whole; lanes past the end read its last 16 bytes
// again.  The LDS behind is padded to 1 KB.
__device__ __forceinline__ void load_pieces(const float *src, int bytes, unsigned char *lds) {
    for (int x = (threadIdx.x >> 6) * 1024; x < bytes; x += 8192)
        lds_stream16_coherent(reinterpret_cast<const unsigned char *>(src) + min(x + (int)(threadIdx.x & 63) * 16, bytes - 16), lds + x);
}

template <int D, int NB, int KIND>
__global__ __launch_bounds__(512, 1) void stream_kernel(const StreamArgs args) {
    using C = StreamCfg<D, NB>;
    constexpr int KST = D / 32, DB = D / 16;
    constexpr bool VNAT = KIND != kStreamVT, DRAFT = KIND == kStreamDraft;
    extern __shared__ __align__(16) unsigned char smem[];
    __shared__ int s_last[2];
    MAD_TRACE_T0();
    const StreamCtx a = load_ctx(args);
    const DraftCtx ring = DRAFT ? load_draft(args) : DraftCtx{};

    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int lr = lane & 15, lg = lane >> 4;
    const int w = blockIdx.x;
    const int T = DRAFT ? 1 : a.T, G = a.G, R = T * G, Hkv = a.Hkv;

    // ---- this workgroup's run of slabs: the first one's unit (b, c) and slab t, and their number ----
    int b, c, t, left, piece = w;   // piece: this run's number within its unit's pieces, less the unit's
    if (a.by_unit) {
        b = __popcll(__ballot(Hkv * a.rec.z <= w)) - 1;   // records past the last row hold the end
        const int k = a.splits(b), rel = w - Hkv * a.wg0(b), n0 = a.slabs(b);
        // by_unit 1: neighbouring workgroups take the row's units in turn (plan_stream); one division for both
        // orders, since every line of instructions here is a miss in a short launch
        const bool turn = !DRAFT && a.by_unit == 1;
        const int m = turn ? Hkv : k, x0 = rel / m, x1 = rel - x0 * m;
        c = turn ? x1 : x0;
        const int part = turn ? x0 : x1;
        if (!DRAFT) piece = w - rel + c * k + part;
        const int lo = n0 / k, hi = n0 - lo * k;   // hi pieces of lo + 1 slabs, then of lo
        t = part * lo + min(part, hi);
        left = lo + (part < hi ? 1 : 0);
    } else {
        const int g0 = stream_first(w, a.base, a.rem);
        left = stream_first(w + 1, a.base, a.rem) - g0;
        b = __popcll(__ballot(Hkv * a.rec.w <= g0)) - 1;
        const int n0 = a.slabs(b), rel = g0 - Hkv * a.tile0(b);
        c = rel / n0;
        t = rel - c * n0;
    }

    // ---- issue side: the next slab to load is slab i_t of unit (i_b, i_c) ----
    const int wv = __builtin_amdgcn_readfirstlane(wave);
    int i_b = b, i_c = c, i_t = t, i_left = left, i_nt = 0;
    int issued = 0, q_issued = 0, q_done = 0;   // slabs; query areas filled, and copied to registers
    int i_stage = 0;                            // stage of the slab, bytes
    int64_t i_keys = 0;                         // the unit's keys from the slab on
    const bf16_t *i_k = nullptr, *i_v = nullptr;   // the slab's K and V rows (V^T: the unit's first feature)
    // draft: the unit's memory and window lengths, ring start, ring rows and new token
    int i_mlen = 0, i_wlen = 0, i_wst = 0;
    const bf16_t *i_wk = nullptr, *i_wv = nullptr;
    auto keys_of = [&](int row) {
        return DRAFT ? a.len(row) + __builtin_amdgcn_readlane(a.rec.y, row) + (ring.mode(row) != 0 ? 1 : 0) : a.len(row);
    };
    auto i_unit = [&]() {
        i_nt = a.slabs(i_b);
        if constexpr (DRAFT) {
            i_mlen = a.len(i_b);
            i_wlen = __builtin_amdgcn_readlane(a.rec.y, i_b);
            i_wst = ring.start(i_b);
            i_wk = bits_ptr<const bf16_t>(ring.wk) + i_b * ring.seq + i_c * ring.head;
            i_wv = bits_ptr<const bf16_t>(ring.wv) + i_b * ring.seq + i_c * ring.head;
        }
        i_keys = keys_of(i_b) - (int64_t)i_t * C::SLAB;
        i_k = bits_ptr<const bf16_t>(a.k) + i_b * a.seq + i_c * a.head + (int64_t)i_t * C::SLAB * D;
        i_v = bits_ptr<const bf16_t>(a.v) + i_b * a.seq + i_c * a.head + (VNAT ? (int64_t)i_t * C::SLAB * D : 0);
    };
    i_unit();
    // K and natural V: lane l of wave load inst fetches row cidx / CPR (cidx = 64 inst + l) of the
    // slab; LDS slot cidx % CPR of the row holds its chunk slot ^ swizzle(row).  A wave's load j adds
    // 1024 j to both of its addresses (an instruction offset), so its lane offset leaves that out.
    constexpr int LPW = C::IPW / 2;   // K (and V) loads per wave
    uint32_t k_off[LPW], v_off[LPW];
    #pragma unroll
    for (int j = 0; j < LPW; ++j) {
        const int cidx = (wave * LPW + j) * 64 + lane, kr = cidx / C::CPR, slot = cidx % C::CPR;
        k_off[j] = kr * C::RB + ((slot ^ k_swz<D>(kr)) << 4) - 1024 * j;
        if constexpr (VNAT) {
            v_off[j] = kr * C::RB + ((slot ^ v_swz<D>(kr)) << 4) - 1024 * j;
        } else {   // V^T: a run of SLAB keys of feature cidx / VCH (from j = 1 on at least 1024 bytes on: cap >= SLAB where used)
            const int f = cidx / C::VCH, vs = cidx % C::VCH;
            v_off[j] = (uint32_t)f * (uint32_t)a.cap * 2 + ((vs ^ (f & 7)) << 4) - 1024 * j;
        }
    }
    static_assert(LPW == 2, "lds_stream16_x2");
    // Every byte is read once, hence the non-temporal hint, but for V^T runs that are not whole 128-byte
    // lines: the next slab's run takes the rest of this one's lines from L2 (8 KV heads, d 128, 32773 keys, 4
    // sequences, cap 32776: 110 -> 89 us; with whole lines, cap 32832, 86.4 us cached and 84.2 so).
    const bool v_nt = VNAT || (((a.cap | a.head | a.seq) % 64 == 0) && a.v % 128 == 0);
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane(lds_addr(smem)) + wv * LPW * 1024;
    // the first slab of a unit (or of the run) needs a free query area
    auto can_issue = [&]() {
        return i_left > 0 && ((i_t > 0 && issued > 0) || q_issued - q_done < C::QSLOTS);
    };
    auto issue = [&]() {
        if (i_t == 0 || issued == 0) {
            // the unit's query rows, 1 KB per wave load; lanes past them fetch the last chunk again
            unsigned char *qa = smem + C::OFF_Q + (C::QSLOTS == 2 ? (q_issued & 1) * C::QBYTES : 0);
            const bf16_t *qb = bits_ptr<const bf16_t>(a.q) + ((size_t)i_b * T * a.Hq + (size_t)i_c * G) * D;
            for (int p = wv; p * 1024 < R * C::RB; p += C::NWV) {
                const int ch = min(p * 64 + lane, R * C::CPR - 1), r = ch / C::CPR, tt = r / G;
                lds_stream16(qb + ((size_t)tt * a.Hq + (r - tt * G)) * D + (ch % C::CPR) * 8, qa + p * 1024);
            }
            ++q_issued;
        }
        // a slab whose rows all exist in one place (draft: in the memory, or in the ring without a
        // wrap) has one base and fixed lane offsets
        const bf16_t *k0 = i_k, *v0 = VNAT ? i_v : i_v + (int64_t)i_t * C::SLAB;
        bool one = i_keys >= C::SLAB && (VNAT || a.cap <= (int)(0xffffffffu / (2 * D)));   // (32-bit lane offsets)
        if constexpr (DRAFT) {
            const int kb = i_t * C::SLAB;
            one = kb + C::SLAB <= i_mlen;
            if (!one && kb >= i_mlen && kb + C::SLAB <= i_mlen + i_wlen) {
                int r0 = i_wst + (kb - i_mlen);
                if (r0 >= ring.cap) r0 -= ring.cap;
                one = r0 + C::SLAB <= ring.cap;
                k0 = i_wk + (size_t)r0 * D;
                v0 = i_wv + (size_t)r0 * D;
            }
        }
        if (one) {
            lds_stream16_x2<true>(k0, k_off[0], k_off[1], lds0 + i_stage);
            if (v_nt) lds_stream16_x2<true>(v0, v_off[0], v_off[1], lds0 + i_stage + C::KBYTES);
            else lds_stream16_x2<false>(v0, v_off[0], v_off[1], lds0 + i_stage + C::KBYTES);
        } else if constexpr (DRAFT) {
            // row by row: memory, ring, the new token; rows past the end repeat the last one (masked),
            // those of an empty row read the queries (never used)
            unsigned char *st = smem + i_stage;
            const int n = keys_of(i_b);
            #pragma unroll
            for (int j = 0; j < LPW; ++j) {
                const int inst = wv * LPW + j;
                const int cidx = inst * 64 + lane, kr = cidx / C::CPR, slot = cidx % C::CPR;
                const int key = min(i_t * C::SLAB + kr, n - 1), i = key - i_mlen;
                int r = i_wst + i;
                if (r >= ring.cap) r -= ring.cap;
                const size_t nrow = ((size_t)i_b * Hkv + i_c) * D;
                const bf16_t *kp = i < 0 ? i_k + (int64_t)(key - i_t * C::SLAB) * D
                                 : i < i_wlen ? i_wk + (size_t)r * D : bits_ptr<const bf16_t>(ring.kn) + nrow;
                const bf16_t *vp = i < 0 ? i_v + (int64_t)(key - i_t * C::SLAB) * D
                                 : i < i_wlen ? i_wv + (size_t)r * D : bits_ptr<const bf16_t>(ring.vn) + nrow;
                if (n == 0) kp = vp = bits_ptr<const bf16_t>(a.q);
                lds_stream16_nt(kp + (slot ^ k_swz<D>(kr)) * 8, st + inst * 1024);
                lds_stream16_nt(vp + (slot ^ v_swz<D>(kr)) * 8, st + C::KBYTES + inst * 1024);
            }
        } else {
            unsigned char *st = smem + i_stage;
            const int keys = (int)min(i_keys, (int64_t)C::SLAB);
            #pragma unroll
            for (int j = 0; j < LPW; ++j) {
                const int inst = wv * LPW + j;
                const int cidx = inst * 64 + lane;
                const int kr = cidx / C::CPR, slot = cidx % C::CPR;
                const int key = min(kr, keys - 1);   // rows past len: a valid row, masked
                lds_stream16_nt(i_k + key * D + (slot ^ k_swz<D>(kr)) * 8, st + inst * 1024);
                if constexpr (VNAT) {
                    lds_stream16_nt(i_v + key * D + (slot ^ v_swz<D>(kr)) * 8, st + C::KBYTES + inst * 1024);
                } else {
                    // V^T: feature cidx / VCH, LDS slot holds key chunk slot ^ (f & 7)
                    const int f = cidx / C::VCH, vs = cidx % C::VCH;
                    int kc = i_t * C::SLAB + ((vs ^ (f & 7)) << 3);
                    if (kc + 8 > a.cap) kc = a.cap - 8;      // chunks past the cache: any valid chunk (zeroed when used)
                    lds_stream16_nt(i_v + (size_t)f * a.cap + kc, st + C::KBYTES + inst * 1024);
                }
            }
        }
        ++issued;
        --i_left;
        i_stage = (i_stage + C::STAGE) & (C::NST * C::STAGE - 1);
        i_keys -= C::SLAB;
        i_k += C::SLAB * D;
        if (VNAT) i_v += C::SLAB * D;
        if (++i_t == i_nt && i_left > 0) {
            i_t = 0;
            if (++i_c == Hkv) {
                i_c = 0;
                ++i_b;
            }
            i_unit();
        }
    };

    // ---- compute side: row block rbw, key group kg of every slab ----
    const int rbw = wave % NB, kg = wave / NB, row = rbw * 16 + lr;
    const bool active = kg < C::KS;
    const int row_t = min(row, R - 1) / G;   // this row's query index t
    bf16x8_v qf[KST];
    int len = 0, lim = 0, nt = 0;
    f32x4_v o[DB];
    float m_run = -INFINITY, l_run = 0.f;
    const float cs = a.cs;

    auto start_unit = [&]() {
        nt = a.slabs(b);
        len = keys_of(b);
        lim = len - T + row_t;
        const unsigned char *qa = smem + C::OFF_Q + (C::QSLOTS == 2 ? (q_done & 1) * C::QBYTES : 0) + min(row, R - 1) * C::RB;
        #pragma unroll
        for (int ks = 0; ks < KST; ++ks) qf[ks] = *reinterpret_cast<const bf16x8_v *>(qa + ks * 64 + lg * 16);
        m_run = -INFINITY;
        l_run = 0.f;
        #pragma unroll
        for (int db = 0; db < DB; ++db) o[db] = f32x4_v{0.f, 0.f, 0.f, 0.f};
    };

    // 32 keys of the slab, from key 32 kh of it
    auto compute = [&](const unsigned char *st, int kb, int kh) {
        // A row m of block blk is key 32 kh + 8(m/4) + 4 blk + m%4 of the slab, so
        // accumulator element e&3 of block e>>2 is key 32 kh + 8 lg + e
        // Every operand of the step is read at once, so V's LDS latency runs behind the scores and the softmax.
        bf16x8_v kf[2][KST], vf[DB];
        #pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
            const int kr = 32 * kh + 8 * (lr >> 2) + 4 * blk + (lr & 3);
            #pragma unroll
            for (int ks = 0; ks < KST; ++ks)
                kf[blk][ks] = *reinterpret_cast<const bf16x8_v *>(st + kr * C::RB + (((4 * ks + lg) ^ k_swz<D>(kr)) << 4));
        }
        const unsigned char *sv8 = st + C::KBYTES;
        if constexpr (VNAT) {
            // A = V^T rows (features db*16 + lr), keys 32 kh + 8 lg .. +7, from
            // the transposing reads of key rows 32 kh + 8 lg + {0..3} and {4..7}
            // (rows past len hold the clamped row len - 1, weighted 0)
            const int r0 = 32 * kh + 8 * lg + (lr >> 2), r1 = r0 + 4, tr_byte = 8 * (lr & 3);
            #pragma unroll
            for (int db = 0; db < DB; ++db) {
                const int byte = db * 32 + tr_byte, chunk = byte >> 4, half = byte & 8;
                const v4s_t lo = lds_read_tr16(sv8 + r0 * C::RB + ((chunk ^ v_swz<D>(r0)) << 4) + half);
                const v4s_t hi = lds_read_tr16(sv8 + r1 * C::RB + ((chunk ^ v_swz<D>(r1)) << 4) + half);
                vf[db] = __builtin_bit_cast(bf16x8_v, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
            }
        } else {
            #pragma unroll
            for (int db = 0; db < DB; ++db) {
                const int f = db * 16 + lr;
                vf[db] = *reinterpret_cast<const bf16x8_v *>(sv8 + f * C::VROW + (((4 * kh + lg) ^ (f & 7)) << 4));
            }
            if (kb + C::SLAB > len) {   // the unit's last slab: values of keys past len may be anything, zero them
                u32x4_v keep;
                #pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int kk = kb + 32 * kh + 8 * lg + 2 * e;
                    keep[e] = kk >= len ? 0u : kk + 1 >= len ? 0x0000ffffu : 0xffffffffu;
                }
                #pragma unroll
                for (int db = 0; db < DB; ++db) vf[db] = __builtin_bit_cast(bf16x8_v, __builtin_bit_cast(u32x4_v, vf[db]) & keep);
            }
        }
        f32x4_v sacc[2];
        #pragma unroll
        for (int blk = 0; blk < 2; ++blk) {
            sacc[blk] = f32x4_v{0.f, 0.f, 0.f, 0.f};
            #pragma unroll
            for (int ks = 0; ks < KST; ++ks)
                sacc[blk] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[blk][ks], qf[ks], sacc[blk], 0, 0, 0);
        }
        float sv[8];
        float mt = -INFINITY;
        const int kg0 = kb + 32 * kh + 8 * lg;
        if (__all(kb + C::SLAB - 1 <= lim)) {
            #pragma unroll
            for (int j = 0; j < 8; ++j) {
                sv[j] = sacc[j >> 2][j & 3];
                mt = fmaxf(mt, sv[j]);
            }
        } else {
            #pragma unroll
            for (int j = 0; j < 8; ++j) {
                sv[j] = kg0 + j <= lim ? sacc[j >> 2][j & 3] : -INFINITY;
                mt = fmaxf(mt, sv[j]);
            }
        }
        mt = max_over_row_lanes(mt);
        const float mn = fmaxf(m_run, mt);
        const bool same = mn == m_run;
        const float ms = (mn == -INFINITY) ? 0.f : mn * cs;
        const float alpha = same ? 1.f : __builtin_amdgcn_exp2f(fmaf(m_run, cs, -ms));
        m_run = mn;
        float ps = 0.f;
        uint32_t pk[4];
        #pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(sv[2 * e], cs, -ms));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(sv[2 * e + 1], cs, -ms));
            ps += p0 + p1;
            pk[e] = cvt_pk_bf16(p0, p1);
        }
        const bf16x8_v pf = __builtin_bit_cast(bf16x8_v, u32x4_v{pk[0], pk[1], pk[2], pk[3]});
        l_run = fmaf(l_run, alpha, ps);
        if (!__all(same)) {
            #pragma unroll
            for (int db = 0; db < DB; ++db) o[db] *= alpha;
        }
        #pragma unroll
        for (int db = 0; db < DB; ++db) o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[db], pf, o[db], 0, 0, 0);
    };

    // ---- end of a unit's run in this workgroup: the key groups' results go to
    // the stage just read (the next load into it is issued behind the loop's
    // next barrier), chunks swizzled by row, and every thread merges whole
    // 16-byte chunks: either the unit's result or its piece for the merge.
    // Written straight from the accumulators (16 rows, 32 bytes of each, a
    // wave store) with unswizzled exchange rows a flush stalled the stream for
    // 2.6 us at 48 rows, d 128; so 1.6 us. ----
    int pu0 = -1, pu1 = -1;   // units of which this run holds a piece: begun by an earlier workgroup, begun here
    float *lse = bits_ptr<float>(a.lse);
    auto flush = [&](unsigned char *st, bool from0) {
        const bool whole = from0 && t == nt;   // every slab of the unit ran here
        const int u = b * Hkv + c;
        if (!from0) pu0 = u;
        else if (!whole) pu1 = u;
        constexpr int DP = D / C::XPASS, QP = DP / 4;                 // features, chunks of a row per pass
        float2 *xml = reinterpret_cast<float2 *>(smem + C::OFF_ML);   // [KS][RP]
        const float lt = sum_over_row_lanes(l_run);
        if constexpr (DRAFT) {
            // the unit's last slab holds the new token: append it to the window ring from here
            // (its row is outside every window of the launch)
            if (t == nt && ring.mode(b) == 2 && tid < 2 * C::CPR) {
                const int kr = len - 1 - (nt - 1) * C::SLAB, ch = tid % C::CPR;
                const bool is_v = tid >= C::CPR;
                const uint4 x = *reinterpret_cast<const uint4 *>(st + (is_v ? C::KBYTES : 0) + kr * C::RB +
                                                                 ((ch ^ (is_v ? v_swz<D>(kr) : k_swz<D>(kr))) << 4));
                int r = ring.start(b) + __builtin_amdgcn_readlane(a.rec.y, b);
                if (r >= ring.cap) r -= ring.cap;
                bf16_t *dst = bits_ptr<bf16_t>(is_v ? ring.wv : ring.wk) + b * ring.seq + c * ring.head + (size_t)r * D;
                reinterpret_cast<uint4 *>(dst)[ch] = x;
            }
        }
        #pragma unroll
        for (int ps = 0; ps < C::XPASS; ++ps) {
            __syncthreads();   // every wave is done with the stage
            if (active) {
                #pragma unroll
                for (int db = 0; db < DP / 16; ++db)
                    *reinterpret_cast<f32x4_v *>(st + ((kg * C::RP + row) * QP + ((db * 4 + lg) ^ (row & (QP - 1) & 15))) * 16) =
                        o[ps * (DP / 16) + db];
                if (ps == 0 && lg == 0) xml[kg * C::RP + row] = make_float2(m_run == -INFINITY ? -INFINITY : m_run * cs, lt);
            }
            __syncthreads();
            for (int x = tid; x < R * QP; x += 512) {
                const int r = x / QP, ch = x % QP;
                float m[C::KS], M = -INFINITY, L = 0.f;
                f32x4_v y = f32x4_v{0.f, 0.f, 0.f, 0.f};
                #pragma unroll
                for (int k = 0; k < C::KS; ++k) {
                    m[k] = xml[k * C::RP + r].x;
                    M = fmaxf(M, m[k]);
                }
                #pragma unroll
                for (int k = 0; k < C::KS; ++k) {
                    const float wt = M == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[k] - M);
                    const f32x4_v v = *reinterpret_cast<const f32x4_v *>(st + ((k * C::RP + r) * QP + (ch ^ (r & (QP - 1) & 15))) * 16);
                    L = fmaf(wt, xml[k * C::RP + r].y, L);
                    #pragma unroll
                    for (int e = 0; e < 4; ++e) y[e] = fmaf(wt, v[e], y[e]);
                }
                if (whole) {
                    const int tt = r / G;
                    const size_t head = ((size_t)b * T + tt) * a.Hq + (size_t)c * G + (r - tt * G);
                    const float inv = L > 0.f ? 1.f / L : 0.f;
                    uint2 pk = make_uint2(pack_bf16x2(y[0] * inv, y[1] * inv), pack_bf16x2(y[2] * inv, y[3] * inv));
                    if (L == 0.f) pk = make_uint2(0u, 0u);   // no key at all: whatever rows stood in
                    *reinterpret_cast<uint2 *>(bits_ptr<bf16_t>(a.out) + head * D + ps * DP + ch * 4) = pk;
                    if (lse && ps == 0 && ch == 0) lse[head] = L > 0.f ? (M + log2f(L)) * kLn2 : -INFINITY;
                } else {
                    // runs and units both advance in slab order, so piece + u numbers the pieces one after the other
                    float *pp = bits_ptr<float>(a.part) + (size_t)(piece + u) * piece_floats(R, D);
                    store_agent4(pp + r * D + ps * DP + ch * 4, y);
                    if (ps == 0 && ch == 0) store_agent2(pp + R * D + 2 * r, M, L);
                }
            }
        }
    };

    while (issued < C::NST - 1 && can_issue()) issue();
    bool first = true;   // the run's first unit
    int c_stage = 0;
    for (int i = 0; i < left; ++i) {
        if (issued <= i) {   // the slab waited for a query area, which every wave has read by now
            __syncthreads();
            issue();
        }
        wait_vm(C::IPW * (issued - 1 - i));   // slab i has landed (this wave's part; newer query loads only make it stricter)
        __syncthreads();                      // ... every wave's part; stage (i-1) % NST is free
        while (issued < i + C::NST && can_issue()) issue();
        if (t == 0 || i == 0) {
            start_unit();
            ++q_done;
        }
        unsigned char *st = smem + c_stage;
        c_stage = (c_stage + C::STAGE) & (C::NST * C::STAGE - 1);
        if (active) {
            #pragma unroll
            for (int h = 0; h < C::KPG / 32; ++h) compute(st, t * C::SLAB, kg * (C::KPG / 32) + h);
        }
        ++t;
        if (t == nt || i == left - 1) {
            flush(st, !first || i + 1 == t);
            first = false;
            if (t == nt) {
                t = 0;
                if (++c == Hkv) {
                    c = 0;
                    ++b;
                }
            }
        }
    }
    MAD_TRACE_SAVE_T0(mad_trace_verify);
    MAD_TRACE(mad_trace_verify, 1);
    if ((pu0 < 0 && pu1 < 0) || a.merge2) return;

    // ---- arrivals; the last workgroup at a unit merges its pieces, both of its units' (where it is
    // last at both) behind one round trip ----
    const UnitPieces up0 = unit_pieces(a, max(pu0, 0)), up1 = unit_pieces(a, max(pu1, 0));
    wait_vm_stores();
    __syncthreads();
    MAD_TRACE(mad_trace_verify, 2);
    if (tid == 0 || tid == 64) {
        const int u = tid == 0 ? pu0 : pu1;
        int last = 0;
        if (u >= 0) {
            unsigned *cnt = bits_ptr<unsigned>(a.counters) + (size_t)u * kCounterStride;
            last = arrive(cnt) == (unsigned)((tid == 0 ? up0.np : up1.np) - 1);
            if (last) reset_counter(cnt);
        }
        s_last[tid >> 6] = last;
    }
    __syncthreads();
    MAD_TRACE(mad_trace_verify, 3);
    const int pf = piece_floats(R, D);
    const float *part = bits_ptr<const float>(a.part);
    const int last = (s_last[0] ? 1 : 0) + (s_last[1] ? 2 : 0);
    if (last == 0) return;
    const int bytes0 = (last & 1) ? up0.np * pf * 4 : 0, bytes1 = (last & 2) ? up1.np * pf * 4 : 0;
    const int at1 = (bytes0 + 1023) & ~1023;
    static_assert(kMergeBytes <= C::OFF_Q, "the pieces lie in the ring");
    __shared__ float sinv[2 * MAD_MAX_VERIFY_ROWS];
    auto merge = [&](bool first_unit, bool second_unit, int at) {
        if (first_unit) load_pieces(part + (size_t)up0.p0 * pf, bytes0, smem);
        if (second_unit) load_pieces(part + (size_t)up1.p0 * pf, bytes1, smem + at);
        const MergeJob<D> j0 = {pu0, up0.np, R, smem, smem + R * D * 4, pf * 4, sinv};
        const MergeJob<D> j1 = {pu1, up1.np, R, smem + at, smem + at + R * D * 4, pf * 4, sinv + R};
        wait_vm(0);
        __syncthreads();
        if (first_unit) j0.weights(a);
        if (second_unit) j1.weights(a);
        __syncthreads();
        if (first_unit) j0.sums(a);
        if (second_unit) j1.sums(a);
    };
    if (at1 + bytes1 <= kMergeBytes) {
        merge(last & 1, last & 2, at1);
    } else {   // one after the other (each fits: plan_stream)
        merge(true, false, 0);
        __syncthreads();
        merge(false, true, 0);
    }
    MAD_TRACE(mad_trace_verify, 4);
}

// The merge as a launch of its own, one workgroup per unit and query row: NG
// groups of D/4 threads, a feature quad each, take every NG-th piece.  A thread
// issues the loads of up to U pieces with their (max, sum) at once and folds
// them on its own, so the chain is one round trip, an exponential per piece
// and one exchange between the groups.
template <int D>
__global__ __launch_bounds__(256) void stream_merge_kernel(const StreamArgs args) {
    constexpr int FQ = D / 4, NG = 256 / FQ;
    __shared__ f32x4_v s_y[NG][FQ];
    __shared__ float2 s_ml[NG];
    const StreamCtx a = load_ctx(args);
    const int u = blockIdx.x, r = blockIdx.y, R = a.T * a.G;
    const UnitPieces up = unit_pieces(a, u);
    if (up.np == 1) return;   // finished by its workgroup
    const int fq = threadIdx.x % FQ, grp = threadIdx.x / FQ, pf = piece_floats(R, D);
    const float *po = bits_ptr<const float>(a.part) + (size_t)up.p0 * pf + r * D + fq * 4;
    const float *pm = bits_ptr<const float>(a.part) + (size_t)up.p0 * pf + R * D + r * 2;
    float M = -INFINITY, L = 0.f;
    f32x4_v y = f32x4_v{0.f, 0.f, 0.f, 0.f};
    auto fold = [&](int p0, auto n_const) {
        constexpr int U = decltype(n_const)::value;
        f32x4_v v[U];
        float2 ml[U];
        #pragma unroll
        for (int k = 0; k < U; ++k) {   // past the unit's pieces: the last one again, not used
            const size_t at = (size_t)min(p0 + k * NG, up.np - 1) * pf;
            ml[k] = *reinterpret_cast<const float2 *>(pm + at);
            v[k] = *reinterpret_cast<const f32x4_v *>(po + at);
        }
        float mn = M;
        #pragma unroll
        for (int k = 0; k < U; ++k) mn = fmaxf(mn, ml[k].x);
        const float mr = mn == -INFINITY ? 0.f : mn, c = __builtin_amdgcn_exp2f(M - mr);
        L *= c;
        y *= c;
        #pragma unroll
        for (int k = 0; k < U; ++k) {
            const bool in = p0 + k * NG < up.np;   // (a weight of 0 would make NaN of an infinite value)
            const float wt = in ? __builtin_amdgcn_exp2f(ml[k].x - mr) : 0.f;
            L = fmaf(wt, ml[k].y, L);
            #pragma unroll
            for (int e = 0; e < 4; ++e) y[e] = fmaf(wt, in ? v[k][e] : 0.f, y[e]);
        }
        M = mn;
    };
    if (up.np <= NG) {
        fold(grp, std::integral_constant<int, 1>());
    } else if (up.np <= 4 * NG) {
        fold(grp, std::integral_constant<int, 4>());
    } else {
        for (int p = grp; p < up.np; p += 8 * NG) fold(p, std::integral_constant<int, 8>());
    }
    s_y[grp][fq] = y;
    if (fq == 0) s_ml[grp] = make_float2(M, L);
    __syncthreads();
    if (threadIdx.x >= FQ) return;
    float w[NG];
    M = s_ml[0].x;
    #pragma unroll
    for (int k = 1; k < NG; ++k) M = fmaxf(M, s_ml[k].x);
    const float mr = M == -INFINITY ? 0.f : M;
    L = 0.f;
    y = f32x4_v{0.f, 0.f, 0.f, 0.f};
    #pragma unroll
    for (int k = 0; k < NG; ++k) {
        w[k] = __builtin_amdgcn_exp2f(s_ml[k].x - mr);
        L = fmaf(w[k], s_ml[k].y, L);
        #pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = fmaf(w[k], s_y[k][fq][e], y[e]);
    }
    const float inv = L > 0.f ? 1.f / L : 0.f;
    const size_t head = out_head(a, u, r);
    *reinterpret_cast<uint2 *>(bits_ptr<bf16_t>(a.out) + head * D + fq * 4) =
        make_uint2(pack_bf16x2(y[0] * inv, y[1] * inv), pack_bf16x2(y[2] * inv, y[3] * inv));
    if (a.lse && fq == 0) bits_ptr<float>(a.lse)[head] = L > 0.f ? (M + log2f(L)) * kLn2 : -INFINITY;
}

// ------------------------------------------------------------------ host ----

// One workgroup per CU (its ring fills most of the LDS); fewer when there are
// fewer slabs.  Two ways to deal the slabs, by the longest share they give:
//   by unit   unit (b, c) is cut into k_b even pieces, k_b as the row's length
//             asks: no workgroup crosses a unit, every unit has few pieces;
//   runs      equal contiguous runs over all units in unit order, for ragged
//             batches whose pieces would come out uneven.
// Neighbouring workgroups are on different XCDs.  With a multiple of 8 KV heads,
// taking the row's units in turn keeps a unit's pieces (its query rows, its
// partials) on one, which counts where the pieces are large and the runs short:
// from 32 query rows and up to 16 slabs (64/8 heads, d 128, 5 queries, 1 sequence: 2000 keys
// 11.1 -> 9.8 us, 8000 keys 15.4 -> 14.9; 4 of 512 keys 11.8 -> 10.8), from 17 rows and up to 3 slabs
// (32/8 heads, 4088 keys 10.9 -> 10.3, 4100 keys 11.5 -> 11.2).  Elsewhere the pieces of one unit side by
// side do better (8/8 heads, 4 sequences of 2048 keys 12.8 us against 13.6; 64/8 heads, 32773 keys, runs
// of 17, 30.3 against 31.0; 32/8, 4 sequences, runs of 65, 83.6 against 90), except over V^T of
// long units, whose runs lie all over the unit's 2 MB and more (32/8 heads, d 128, 16384 keys: 1 sequence 20.5 us
// side by side, 18.2 in turn, 4 52.6 and 48.1; 8192 keys 15.1 and 14.1; but 4 of 4096 17.2 and 17.7).
// A run that crosses into the next unit stalls once (the flush, 1.6 us at 48
// rows, d 128) and units get one piece more, so by unit is taken up to 2 slabs
// and 1/16 above the even share: the draft's 16 sequences of 700 .. 1500 keys
// took 15.4 us in runs of 4 or 5 slabs, 13.4 by unit with 6; 4 sequences of 32773 keys (513 slabs a unit) took
// 88.7 us in runs, 87.1 by unit; 16 of 600 .. 12000 keys 74 us in runs (100 with
// splits of one length).  By unit also serves launches with more units than workgroups can
// count (a unit each: no pieces, no counters).
void plan_stream(StreamArgs &a, int B, int Hkv, int d, const int *n_keys) {
    const int slab = stream_slab(d);
    int64_t rows = 0;
    int nt[kMaxB], nt_max = 1;
    for (int b = 0; b < B; ++b) {
        nt[b] = n_keys[b] > 0 ? (n_keys[b] - 1) / slab + 1 : 1;
        a.row[b].x = n_keys[b];
        a.row[b].w = (int)rows;
        rows += nt[b];
        nt_max = nt[b] > nt_max ? nt[b] : nt_max;
    }
    for (int b = B; b < kMaxB; ++b) a.row[b].w = (int)rows;
    a.rows = (int)rows;
    const int64_t total = rows * Hkv;
    a.B = B;
    a.Hkv = Hkv;
    a.merge2 = 0;
    const bool whole = (int64_t)B * Hkv > kCounterLines || total > 0x3fffffff;   // a unit each
    a.n_wg = total < kStreamWGs ? (int)total : kStreamWGs;
    a.base = whole ? 1 : (int)(total / a.n_wg);
    a.rem = whole ? 0 : (int)(total % a.n_wg);
    int np_max = 1;
    const int even = a.base + (a.rem > 0 ? 1 : 0);
    a.by_unit = 0;
    for (int share = whole ? nt_max : even; whole || share <= even + 2 + even / 16; share += 1 + even / 64) {
        int wgs = 0;
        np_max = 1;
        for (int b = 0; b < B; ++b) {
            const int k = (nt[b] - 1) / share + 1;
            a.row[b].z = wgs;
            wgs += k;
            np_max = k > np_max ? k : np_max;
        }
        if (!whole && wgs * Hkv > kStreamWGs) continue;
        for (int b = B; b < kMaxB; ++b) a.row[b].z = wgs;
        const bool long_vt = a.kind == kStreamVT && nt_max >= 128;
        a.by_unit = Hkv % 8 == 0 && (long_vt || share <= (a.T * a.G >= 32 ? 16 : a.T * a.G > 16 ? 3 : 0)) ? 1 : 2;
        a.wgs = wgs;
        a.n_wg = wgs * Hkv;
        break;
    }
    if (!a.by_unit) {
        np_max = (nt_max - 1) / a.base + 2;
        np_max = np_max > a.n_wg ? a.n_wg : np_max;
    }
    // A unit's pieces are merged by the last workgroup at it, or by a second launch, which takes 1 - 2 us of the
    // host's time and of the GPU's, more with many units, but spreads over the CUs what one workgroup does serially.  Calls issued one
    // by one / in a graph replay (us; 32/8 heads, d 128, 5 queries unless given), in the launch -> in two:
    //   up to 48 KB of pieces: 256 keys, 42 KB, 8.6 -> 9.4 / 9.5 -> 8.6; 2000 keys T 1 G 1, 32 pieces of one row,
    //     8.6 -> 9.5 / 9.65 -> 8.6 (a longer chain in the launch, but the host has one to issue);
    //   above: 1000 keys, 166 KB, 13.4 -> 8.2 in a graph; 4100 keys 17.9 -> 11.2; 32773 keys 29.5 -> 26.9; 4 of 512
    //     keys, 83 KB, 10.5 -> 8.8 / 11.7 -> 9.4;
    //   many units, up to the LDS: 64 sequences of 512 keys, 32/2 heads, T 4, 2 pieces of 33 KB, 17.2 -> 22.5 /
    //     18.4 -> 23.4; 16 of 512 keys at d 64, 4 of 17 KB, 9.7 -> 11.4 / 10.5 -> 11.0.
    const int64_t bytes = (int64_t)np_max * piece_floats(a.T * a.G, d) * 4;
    const int units = B * Hkv;
    const bool in_launch = bytes <= kMergeInLaunch || (units >= 64 && bytes <= kMergeBytes) ||
                           (units >= 32 && np_max <= 4 && bytes <= 72 << 10);
    a.merge2 = np_max > 1 && !in_launch ? 1 : 0;
}

// the pieces of a launch's units: at most one per workgroup and unit
size_t stream_part_bytes(int units, int rows, int d) {
    return align256(((size_t)units + kStreamWGs) * piece_floats(rows, d) * 4);
}

size_t verify_ws_bytes(int B, int Hq, int Hkv, int d, int T) {
    const size_t bf = kCounterRegionBytes + stream_part_bytes(B * Hkv, T * (Hq / Hkv), d);
    // fp32 verify runs the decode kernel once per sequence, its T query rows as the rows
    const size_t f32 = decode_split_bytes(T, Hq, Hkv, d);
    return bf > f32 ? bf : f32;
}

template <int D, int NB>
static hipError_t launch_nb(const StreamArgs &a, hipStream_t st) {
    using C = StreamCfg<D, NB>;
    const dim3 grid((unsigned)a.n_wg), block(64 * C::NWV);
    if (a.kind == kStreamRows)
        hipLaunchKernelGGL((stream_kernel<D, NB, kStreamRows>), grid, block, C::SMEM, st, a);
    else if (a.kind == kStreamVT)
        hipLaunchKernelGGL((stream_kernel<D, NB, kStreamVT>), grid, block, C::SMEM, st, a);
    else if constexpr (NB == 1)
        hipLaunchKernelGGL((stream_kernel<D, NB, kStreamDraft>), grid, block, C::SMEM, st, a);
    return hipGetLastError();
}

template <int D>
static hipError_t launch_d(const StreamArgs &a, hipStream_t st) {
    const int nb = (a.T * a.G + 15) / 16;
    if (a.kind == kStreamDraft && nb != 1) return hipErrorInvalidValue;
    switch (nb) {
        case 1: return launch_nb<D, 1>(a, st);
        case 2: return launch_nb<D, 2>(a, st);
        case 3: return launch_nb<D, 3>(a, st);
        case 4: return launch_nb<D, 4>(a, st);
    }
    return hipErrorInvalidValue;
}

template <int D>
static hipError_t launch_merge(const StreamArgs &a, hipStream_t st) {
    hipLaunchKernelGGL((stream_merge_kernel<D>), dim3((unsigned)(a.B * a.Hkv), (unsigned)(a.T * a.G)), dim3(256), 0, st, a);
    return hipGetLastError();
}

hipError_t launch_stream(const StreamArgs &a, int d, hipStream_t st) {
    if (d != 64 && d != 128) return hipErrorInvalidValue;
    const hipError_t e = d == 64 ? launch_d<64>(a, st) : launch_d<128>(a, st);
    if (e != hipSuccess || a.merge2 == 0) return e;
    return d == 64 ? launch_merge<64>(a, st) : launch_merge<128>(a, st);
}

}  // namespace mad
