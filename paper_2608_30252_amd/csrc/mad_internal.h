// mad_internal.h -- kernel argument blocks and launchers shared between the
// C-ABI layer (mad_api.hip) and the kernels.  Not installed; not part of the ABI.
#pragma once
#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include "mad.h"

namespace mad {

constexpr int kMaxB = MAD_MAX_BATCH;

// ---------------------------------------------------------------- decode ----
// The split count aims at one 4-wave or two 8-wave workgroups per CU; splits
// are whole super-tiles (see plan_decode).
constexpr int kDecodeCUs = 256;        // compute units of the device the split plan is sized for
constexpr int kDecodeWideKeys = 65536;      // 8-wave workgroups: launches holding at least this many keys
constexpr int kDecodeMaxSplits = 256;
// Every workspace starts with a fixed counter region that holds nothing but
// arrival counters (one per 256-byte line) and that every kernel leaves at
// zero.  Its layout therefore never overlaps the partial results of a call
// with other shapes.  Split partials follow it.
constexpr size_t kCounterRegionBytes = (size_t)1 << 20;
constexpr int kCounterStride = 64;   // unsigned ints per counter line
constexpr int kCounterLines = (int)(kCounterRegionBytes / (kCounterStride * 4));

struct DecodeArgs {
    const void *q;
    void *out;
    float *lse;
    const void *mk, *mv;  // memory segment (sinks, slots): linear
    int64_t m_seq, m_head;
    void *wk, *wv;        // local window: ring
    int64_t w_seq, w_head;
    const void *kn, *vn;  // current token K/V [B][Hkv][D] or null
    float *part;          // split partials, one block of part_stride floats per unit
    int64_t part_stride;
    unsigned *counters;   // counter region: unit u on line u
    float scale_log2;     // softmax scale * log2(e)
    int Hq, Hkv, units, n_splits, chunk, w_cap;
    int nsub;             // wave groups per workgroup (1 or 2)
    int fold;             // 1: the last split runs to the end of the row (keys past n_splits * chunk)
    // per row, one 16-byte record read by a single scalar load: memory length,
    // window length, ring start, new-token mode (0 none, 1 attend, 2 attend and append)
    int4 seq[kMaxB];
};

struct DecodePlan {
    int units, n_splits, chunk, n_max, nsub;
    int fold;   // 1: the last split also takes the few keys past n_splits * chunk
};

bool decode_streams(int B, int Hkv, int G, int d, int dtype, const int *n_keys);
DecodePlan plan_decode(int B, int Hkv, int G, int d, int dtype, const int *n_keys);
int decode_max_splits(int d, int G);
size_t decode_part_stride(int d, int G);
size_t decode_split_bytes(int B, int Hq, int Hkv, int d);
size_t decode_ws_bytes(int B, int Hq, int Hkv, int d);
hipError_t launch_decode(const DecodeArgs &a, int dtype, int d, int G, hipStream_t st);

// ---------------------------------------------------------------- update ----
struct UpdateArgs {
    const void *x, *w;    // [R][D] slot rows, [2*Hkv*d][D] mirrored projections
    void *mk, *mv;        // memory segment to append to
    int64_t m_seq, m_head;
    double log2_base;     // log2 of the RoPE base
    int R, n_new, D, Hkv, d;
    int mlen[kMaxB];
    int pos[MAD_MAX_UPDATE_ROWS];
    unsigned char fire[kMaxB];
};

hipError_t launch_update(const UpdateArgs &a, int dtype, hipStream_t st);
constexpr int kUpdateGemvRows = 8;   // bf16 updates of at most this many rows take the weight stream
bool update_uses_gemv(int R, int D, int dtype);

// ---------------------------------------------------------------- stream ----
// bf16 attention over long key streams (stream.hip)
constexpr int kStreamWGs = 256;   // workgroups of a launch: one per CU
__host__ __device__ constexpr int stream_slab(int d) { return d == 128 ? 64 : 128; }   // keys per slab (32 KB of K + V)

constexpr int kMergeBytes = 128 << 10;      // LDS for the pieces of a unit that a workgroup merges in the launch
constexpr int kMergeInLaunch = 48 << 10;    // such pieces where the units are few (plan_stream)

// verify over a cache of K and V rows; over K rows and V^T (one run of cap keys per feature);
// the draft's decode: memory rows, window ring, new token (T = 1)
enum { kStreamRows = 0, kStreamVT = 1, kStreamDraft = 2 };

struct StreamArgs {
    const void *q, *k, *v;    // draft: k and v are the memory rows
    void *out;
    float *lse;
    int64_t seq, head;        // element strides of sequences and KV heads (K and V alike)
    float *part;              // the units' pieces
    unsigned *counters;       // counter region: unit u on line u
    float scale_log2;
    int cap, Hq, Hkv, G, T, kind;
    int n_wg, base, rem;      // workgroup w runs base (+ 1 for w < rem) consecutive slabs
    int by_unit;              // 1, 2: instead, the workgroups of a row's units split each unit evenly (1: the units in turn)
    int B, merge2;            // merge2: the pieces are merged by a second launch
    int rows, wgs;            // slabs, and by_unit workgroups, of one KV head over all rows
    // per row: keys, -, workgroups (by_unit) and slabs of the rows before it (one KV head); past the last row: the end
    int4 row[kMaxB];          // (draft: memory rows, window rows, ...)
    // draft: the window ring and the new token; per row the ring start and the new-token mode
    void *wk, *wv;
    const void *kn, *vn;
    int64_t w_seq, w_head;
    int w_cap;
    int2 ring[kMaxB];
};

// the first slab of workgroup w's run, and the workgroup whose run holds slab x
__host__ __device__ inline int stream_first(int w, int base, int rem) {
    return w * base + (w < rem ? w : rem);
}
__host__ __device__ inline int stream_owner(int x, int base, int rem) {
    const int big = rem * (base + 1);
    return x < big ? x / (base + 1) : rem + (x - big) / base;
}
void plan_stream(StreamArgs &a, int B, int Hkv, int d, const int *n_keys);
hipError_t launch_stream(const StreamArgs &a, int d, hipStream_t st);
size_t verify_ws_bytes(int B, int Hq, int Hkv, int d, int T);
size_t stream_part_bytes(int units, int rows, int d);

// ----------------------------------------------------------------- layer ----
constexpr int kMaxLinRows = MAD_MAX_LAYER_ROWS;

struct LinearArgs {
    const void *x, *w, *gamma, *res;
    void *out, *xn, *q, *k, *v;
    float eps;
    double log2_base;
    int R, D, N, Hq, Hkv, head_dim, kv_from_row0;
    int pos[kMaxLinRows];
};

hipError_t launch_linear(const LinearArgs &a, int mode, hipStream_t st);

// --------------------------------------------------------------- prefill ----
struct PrefillArgs {
    const void *q_raw, *q_slot;
    void *o_raw, *o_slot;
    float *lse_raw, *lse_slot;
    const void *mk, *mv;  // memory segment: sinks, then slots
    int64_t m_seq, m_head;
    const void *rk, *rv;  // the prefix's raw K/V, position x in row x
    int64_t r_seq, r_head;
    float scale_log2;
    int q_cap, slot_cap, Hq, Hkv, units, nrb, nsb;
    int S, W, r, u;
    int P[kMaxB], Mtot[kMaxB];
};

int prefill_tokens_per_block(int d, int G);
hipError_t launch_prefill(const PrefillArgs &a, int d, int G, hipStream_t st);

// ---------------------------------------------------------------- accept ----
constexpr int kAcceptChunk = 8192;   // vocabulary entries per workgroup, greedy rule
constexpr int kStochChunk = 2048;    // ... stochastic rule
constexpr int kAcceptMaxT = 256;     // rows per sequence of the greedy rule (one workgroup applies it)
static_assert((size_t)kMaxB * kCounterStride * 4 + (size_t)kMaxB * kAcceptMaxT * 8 <= kCounterRegionBytes,
              "greedy-accept counters and row keys fit the counter region");

struct AcceptArgs {
    const void *logits;
    const int32_t *draft;      // [B][T-1] device
    int32_t *n_accept, *next_tok;
    uint64_t *row_best;        // [rows] row argmax keys, in the counter region after line B-1 (zero between calls)
    unsigned *counters;        // line b: arrivals of sequence b's workgroups
    int B, T, V, n_chunks;
    int vec16;                 // rows 16-byte aligned and V a multiple of 16 / element size
};

size_t accept_ws_bytes(int B, int T, int V);
hipError_t launch_accept(const AcceptArgs &a, int dtype, hipStream_t st);

struct StochArgs {
    const float *p, *q, *u;    // [B][T][V], [B][T-1][V], [B][T]
    const int32_t *draft;      // [B][T-1]
    int32_t *n_accept, *next_tok;
    double *sums;              // [B][n_chunks][2]: chunk sums of the draw's r and of p_a
    unsigned *counters;        // line b: arrivals of sequence b's chunks
    int B, T, V, n_chunks;
    int vec16;                 // rows of p and q 16-byte aligned (V % 4 == 0, aligned bases)
};
size_t stoch_ws_bytes(int B, int V);
hipError_t launch_stoch(const StochArgs &a, hipStream_t st);

// ws layout helpers: counters first (256-byte aligned), then partials.
inline size_t align256(size_t x) { return (x + 255) & ~(size_t)255; }

}  // namespace mad
