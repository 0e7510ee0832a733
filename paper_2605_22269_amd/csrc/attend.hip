// Attention of new tokens over the retrieved context at one layer (Sec. 3.5, Eq. 9): queries
// W_Q X against keys [R_k, W_K X] and values [R_v, W_V X], where R are the kept rows of the
// frames chosen by the retrieval -- read in place from the store, no gathered copy -- and X the
// caller's own ("local") rows.
//
// attend_kernel: one workgroup of four waves per (question, KV head, tile of 16 queries, share of the rows).  A query of
// the tile is a (token, head of the KV group) pair, so a key / value row is read once for all the heads that share it.
// Nothing crosses the waves until the end: a wave walks blocks of its own, with running statistics of its own, and the
// four results join in LDS.  The shares of a tile whose rows are split are merged by the last of its workgroups to finish; a
// prefill's, whose records are in the caller's workspace, which has no counts, by attend_combine_kernel.
// Everything is summed in a fixed order: the result does not depend on timing.
//
// The prefill of new tokens (Sec. 3.2: they attend to the past cache and to themselves) is the same
// computation with many query tokens, and yields Eq. 1 -- the attention each new token receives --
// on the way: bf16 rows of 64 or 128 features take the kernels further down; for the others attend_kernel (or the merge) also
// writes every query's reference and normaliser; prefill_colsum_kernel recomputes the scores against the new tokens' keys, turns
// them into softmax weights with those and adds them over shares of the queries; prefill_signal_kernel adds the shares and
// KV heads in order and divides by Hq * n_q.  Scratch for it comes from the caller (a workspace argument).
#include <climits>
#include <type_traits>

#include "mukv_internal.h"

namespace mukv {

namespace {

constexpr int kAttQ = 16, kAttWaves = 4; // queries and waves per workgroup of attend_kernel
constexpr int kTileQ = 8;    // queries a row of column sums stands for in the workspace's size
constexpr int kColKeys = 64; // new tokens per workgroup of prefill_colsum_kernel
constexpr int kThreads = 256;

struct AttendArgs {
    const void *q;            // [B][n_q][Hq][D]
    const int32_t *frame_idx; // [B][k_frame] or null
    const void *k_local, *v_local; // [n_local_total][Hkv][D] or null
    const int32_t *local_offsets;  // [B+1] or null
    const void *store_k, *store_v; // the layer's slabs: [Hkv][store_cap][D]
    float *part;                   // [B][n_q*Hq][n_split][D+2]
    int64_t store_cap;
    int n_q, Hq, Hkv, G, k_frame, kappa, n_frames, n_split, n_qtiles, causal;
    float scale_log2e;
    // for prefill_colsum_kernel: a query's pair (what its weights' exponents subtract, 1 / sum of the weights, 0 if there are none)
    // is at part + pair_stride * query, where its first record was if its rows were split; 0: no pairs wanted
    int pair_stride;
};

typedef __attribute__((ext_vector_type(4))) unsigned int raw16; // 16 bytes as they come from memory
template <typename T>
__device__ __forceinline__ raw16 load16(const T *p) {
    return *reinterpret_cast<const raw16 *>(p);
}

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) int i32x4;
typedef __attribute__((ext_vector_type(2))) unsigned int u32x2;
typedef __attribute__((ext_vector_type(4))) short i16x4;
typedef __attribute__((ext_vector_type(8))) short i16x8;
// two floats as bf16, x below y: the conversion instruction rounds to nearest even and keeps NaN a NaN
__device__ __forceinline__ uint32_t bf16_pair(float x, float y) {
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{x, y}, bf16x2));
}
__device__ __forceinline__ void store_out(uint16_t *p, float x) { *p = (uint16_t)bf16_pair(x, 0.f); }
__device__ __forceinline__ void store_out(float *p, float x) { *p = x; }
// ds_read_b64_tr_b16, the LDS transpose read of 16-bit elements: every lane names 8 bytes; within each block
// of 16 lanes, result[t] of lane i is element i % 4 of the 8 bytes named by lane 4 * t + i / 4 of the block,
// t = 0..3 (lane layout checked by an in-bounds probe on the device).
__device__ __forceinline__ i16x4 lds_read_tr16(const unsigned char *p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((i16x4 __attribute__((address_space(3))) *)(p));
}

// Slot of 16-byte piece x of staged row `row`: x ^ row_swizzle.  The transpose reads of half a wave take two neighbouring
// pieces of eight neighbouring rows: 256 bytes over all banks.
template <int D>
__device__ __forceinline__ int row_swizzle(int row) {
    return ((row / (128 / D)) & (D / 16 - 1)) << 1;
}

// Shapes whose prefill is attend_kernel and prefill_colsum_kernel.  The others' kernels carry nothing of the pairs between the two
// (one bf16 question of 28 heads of 128, a call: 9.43 us with a pair worked out and dropped, 9.33 without).
template <typename T, int D>
constexpr bool column_sums() {
    return sizeof(T) == 4 || D < 64;
}

// attend_kernel and prefill_colsum_kernel, fp32 rows and bf16 rows of 16: the queries are brought down before the product by a
// power of two, exactly, to where a score that is finite once scaled by log2(e) / sqrt(D) does not overflow before.
template <typename T, int D>
constexpr float query_factor() {
    return sizeof(T) == 2 && D > 16 ? 1.f : D <= 32 ? 0.25f : 0.125f; // (D = 16 .. 128: the scale is 0.361, 0.255, 0.180, 0.128)
}
template <typename T, int D>
__device__ __forceinline__ raw16 brought_down(raw16 x) {
    constexpr float f = query_factor<T, D>();
    if constexpr (f != 1.f)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if constexpr (sizeof(T) == 4)
                x[e] = __float_as_uint(__uint_as_float(x[e]) * f);
            else
                x[e] = __float_as_uint(__uint_as_float(x[e] << 16) * f) >> 16 | (__float_as_uint(__uint_as_float(x[e] & 0xFFFF0000u) * f) & 0xFFFF0000u);
        }
    return x;
}

// x * s - y with the product rounded, as the maximum y was.
__device__ __forceinline__ float scaled_apart(float x, float s, float y) {
#pragma clang fp contract(off)
    const float p = x * s;
    return p - y;
}

// 2^(x s - ref), ref a whole number.  The difference itself would be rounded at its own size, so the whole number nearest to
// x s goes to the weight's exponent, exactly, and at most a half through the exponential.
__device__ __forceinline__ float weight_of(float x, float s, float ref) {
    const float n = fmaxf(rintf(x * s), ref - 256.f); // (a masked score is -inf, its weight 0)
    return __builtin_amdgcn_ldexpf(__builtin_amdgcn_exp2f(fmaf(x, s, -n)), (int)(n - ref));
}

constexpr float kLargeRef = 16777216.f; // whole numbers up to here have no gaps
// The same for references of any size.
__device__ __forceinline__ float weight_of_any(float x, float s, float ref) {
    return fabsf(ref) > kLargeRef ? __builtin_amdgcn_exp2f(scaled_apart(x, s, ref)) : weight_of(x, s, ref);
}

// Two floats that another workgroup of the launch reads: written through to, and read from, the memory that all XCDs share.
__device__ __forceinline__ void store_far(float *p, float x, float y) {
    __hip_atomic_store(reinterpret_cast<uint64_t *>(p), __builtin_bit_cast(uint64_t, f32x2{x, y}), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ f32x2 load_far(const float *p) {
    return __builtin_bit_cast(f32x2, __hip_atomic_load(reinterpret_cast<const uint64_t *>(p), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
}
// Before the context's records: arrivals of a tile's workgroups, [question][tile][KV head], zero between launches.
__device__ __forceinline__ int *arrivals_of(float *part) { return reinterpret_cast<int *>(part) - kAttendMaxTiles; }
// The last of n workgroups to get here, all of whose store_far's are then there to be read, by every thread.  The arrival that makes
// n sets the count back to zero in the same step, so none is lost between the two.
__device__ __forceinline__ bool last_to_arrive(int *count, int n, int *s_last) {
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); // this wave's stores are in the shared memory
    __syncthreads();                                 // every wave's are
    if (threadIdx.x == 0)
        *s_last = __builtin_amdgcn_atomic_inc32(reinterpret_cast<uint32_t *>(count), (uint32_t)(n - 1), __ATOMIC_RELAXED, "agent") == (uint32_t)(n - 1);
    __syncthreads();
    return *s_last != 0;
}
__global__ __launch_bounds__(kAttendMaxTiles) void clear_arrivals_kernel(float *part) { arrivals_of(part)[threadIdx.x] = 0; }

// Where row `code` of [retrieved rows, local rows] lives: >= 0 a row of the store's slab, < 0 local row ~code.
__device__ __forceinline__ const unsigned char *row_at(const unsigned char *store, const unsigned char *local, int code,
                                                       unsigned store_stride, unsigned local_stride) {
    const bool in_store = code >= 0;
    const uint64_t off = (uint64_t)(unsigned)(in_store ? code : ~code) * (in_store ? store_stride : local_stride);
    return (in_store ? store : local) + off;
}

// The rows of a tile are [kept rows of the listed frames, local rows], in blocks of 32 (bf16) or 16 (fp32), dealt to the
// waves in turn.  A wave's block:
//   rows     a lane works out where one row lives; the others fetch that by lane permutes.  Keys and values go straight to
//            registers, 8 KB each, the next block's requested as soon as this one's are used up.
//   scores   S^T = K Q^T (16x16x32 bf16, 16x16x4 fp32): a lane holds ONE query (lane % 16) and the rows 4 (lane / 16) + r
//            of every 16, so a query's statistics are in-lane work and two exchanges between the rows of lanes.  (The
//            reduction may walk the features in any order: a lane takes 16-byte pieces lane / 16 + 4 k of both.)
//   values   O^T += V^T P^T: the weights are the B operand as they stand in the lane.  bf16: pairs hi + lo (two products,
//            nothing of the fp32 weight is lost), the value rows pass through LDS the wave has to itself and the transpose
//            read hands every lane the 8 rows of one feature.  fp32: step r takes rows 4 (lane / 16) + r, whose features
//            the lanes of a row load in pieces of up to 16 bytes; a piece's elements belong to different output tiles, so
//            no transpose is needed.  Sums are joined pair by pair and the exponentials' arguments kept small (weight_of):
//            one token, 28 heads of 128 over 30 / 81 / 832 rows, distance from 64 bits 1.17 / 1.35 / 1.59e-7; with a block's
//            16 rows one after another and rounded differences 1.28 / 1.45 / 1.68e-7, on the vector ALU 1.21 / 1.36 / 1.66e-7
//            (64 questions a call: 33 us, the former 29, the latter 60).
// What bounds it: many questions, the rate at which the rows arrive (64 questions over 768 + 40 rows, 7B head layout, graph
// replay: 16.4 us a call = 6.4 TB/s of rows, half of them read by several questions; a workgroup that took its rows through
// tables and barriers shared by the waves, with a merge launch: 25.4); few, the chain launch -> frame list -> rows -> merge:
// a compute unit alone draws its rows at 40 GB/s, so the rows of one question are split over workgroups (attend_split).
// Eight waves a workgroup are no faster (16.4; 9.8 against 9.6 for one question).
// MERGE: the rows are shared and the last of a tile's workgroups to finish merges them (one question, 7B head layout, 768 + 32
// rows: 9.3 us a call in four shares with attend_combine_kernel after them, 8.0 without, 7.5 in seven).
template <typename T, int D, bool MERGE>
__global__ __launch_bounds__(64 * kAttWaves) __attribute__((amdgpu_waves_per_eu(2, 2))) void attend_kernel(
    AttendArgs a, T *__restrict__ out) {
    constexpr int W = kAttWaves;
    constexpr bool kBf16 = sizeof(T) == 2;
    constexpr int kRowB = D * (int)sizeof(T), kPieces = kRowB / 16;
    constexpr int kRows = kBf16 ? 32 : 16;  // rows of a block
    constexpr int kTiles = kRows / 16;      // 16-row tiles of the scores
    constexpr int KK = kBf16 ? (D + 31) / 32 : D / 16; // 16-byte pieces of a key row (and of a query) per lane
    constexpr int NF = D / 16;                         // 16-feature tiles of the output
    // bf16: value pieces per lane, each load of the wave kRowsPerLoad whole rows.  fp32: per 4-row step D / 16 floats
    constexpr int kRowsPerLoad = 64 / kPieces, NV = kBf16 ? kRows / kRowsPerLoad : 4;
    constexpr int kVW = kBf16 ? 4 : (D >= 64 ? 4 : D / 16), kVH = kBf16 ? 1 : (D == 128 ? 2 : 1); // dwords per load, loads per row
    typedef __attribute__((ext_vector_type(kVW))) unsigned int raw_v;
    // per wave: staged value rows (bf16), at the end its outputs [16 queries][D]
    __shared__ __align__(1024) unsigned char s_buf[W][64 * D];
    __shared__ int s_frame[kMaxGatherK]; // the question's frames; -1: names no frame of the cache
    __shared__ float s_m[W][kAttQ], s_l[W][kAttQ];
    constexpr bool kQueryLds = !kBf16 && D == 128; // fp32, 128 features: the queries' operands wait in LDS
    __shared__ raw16 s_q[kQueryLds ? KK : 1][kQueryLds ? 64 : 1];
    const int sp = blockIdx.x, g = blockIdx.y % a.Hkv, qt = blockIdx.y / a.Hkv, b = blockIdx.z;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, lr = lane & 15, lg = lane >> 4;
    const int n_queries = a.n_q * a.G; // of this KV head: (token, head in group), token-major
    const float scale = a.scale_log2e * (1.f / query_factor<T, D>());
    for (int i = tid; i < a.k_frame; i += 64 * W) {
        const int f = a.frame_idx[(int64_t)b * a.k_frame + i];
        s_frame[i] = (f >= 0 && f < a.n_frames) ? f : -1;
    }
    // the lane's query as a matrix operand: 16-byte pieces lg, lg + 4, ... of its row
    const int my_q = qt * kAttQ + lr;
    const bool q_ok = my_q < n_queries;
    const int my_tok = q_ok ? my_q / a.G : 0;
    const int64_t my_row = ((int64_t)b * a.n_q + my_tok) * a.Hq + g * a.G + (q_ok ? my_q - my_tok * a.G : 0);
    raw16 qb[kQueryLds ? 1 : KK];
    const bool has_piece = kPieces >= 4 || lg < kPieces; // (rows of 32 bytes have two pieces)
    const int my_piece = kPieces >= 4 ? lg : lg & (kPieces - 1);
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        if (kQueryLds && wave != 0) break; // the same in all waves
        raw16 x = load16(static_cast<const T *>(a.q) + my_row * D + (my_piece + 4 * kk) * (16 / (int)sizeof(T)));
        x = q_ok && has_piece ? brought_down<T, D>(x) : raw16{0u, 0u, 0u, 0u};
        if constexpr (kQueryLds)
            s_q[kk][lane] = x;
        else
            qb[kk] = x;
    }
    const int n_ret = a.k_frame * a.kappa;
    int l0 = 0, n_loc = 0;
    if (a.local_offsets) {
        l0 = a.local_offsets[b];
        n_loc = a.local_offsets[b + 1] - l0;
        if (n_loc < 0) n_loc = 0;
    }
    // rows up to the last one that a query of the tile sees (retrieved rows: every query)
    const int first_tok = qt * kAttQ / a.G;
    const int last_tok = (qt * kAttQ + kAttQ - 1 < n_queries ? qt * kAttQ + kAttQ - 1 : n_queries - 1) / a.G;
    int n_rows = n_ret + n_loc;
    if (a.causal && n_loc - a.n_q + last_tok + 1 < n_loc) n_rows = n_ret + (n_loc - a.n_q + last_tok + 1 > 0 ? n_loc - a.n_q + last_tok + 1 : 0);
    // the workgroup's blocks of rows, dealt to its waves
    const int n_blk = (n_rows + kRows - 1) / kRows, per = (n_blk + a.n_split - 1) / a.n_split;
    const int b_lo = sp * per, b_hi = b_lo + per < n_blk ? b_lo + per : n_blk;
    const unsigned char *sk = static_cast<const unsigned char *>(a.store_k) + (int64_t)g * a.store_cap * kRowB;
    const unsigned char *sv = static_cast<const unsigned char *>(a.store_v) + (int64_t)g * a.store_cap * kRowB;
    const unsigned char *lk = static_cast<const unsigned char *>(a.k_local) + g * kRowB;
    const unsigned char *lv = static_cast<const unsigned char *>(a.v_local) + g * kRowB;
    const unsigned local_stride = (unsigned)a.Hkv * kRowB;
    __syncthreads(); // the frame list is there

    // Where row lane % kRows of a block lives, and the first token that sees it (INT_MAX: it lives nowhere).  Loads are
    // unconditional: a row that lives nowhere, or past the last, reads the slab's first row.  What was read instead of a value
    // row becomes zeros (its weights are zero, but zero times anything must stay zero).
    auto find = [&](int blk, int *code, int *ft) __attribute__((always_inline)) {
        const int r = blk < b_hi ? blk * kRows + (lane & (kRows - 1)) : INT_MAX;
        *code = 0;
        *ft = INT_MAX;
        if (r < n_ret) {
            const int slot = (int)((unsigned)r / (unsigned)a.kappa), f = s_frame[slot];
            if (f >= 0) {
                *code = f * a.kappa + (r - slot * a.kappa);
                *ft = 0;
            }
        } else if (r < n_rows) {
            const int j = r - n_ret;
            *code = ~(l0 + j);
            *ft = a.causal ? j - (n_loc - a.n_q) : 0; // token i sees local row j iff j <= n_loc - n_q + i
        }
    };
    auto value_row = [&](int u) { return kBf16 ? u * kRowsPerLoad + lane / kPieces : 4 * lg + u; }; // of the lane's load u
    raw16 kx[kTiles][KK];
    raw_v vx[NV][kVH];
    auto request_keys = [&](int code) __attribute__((always_inline)) {
#pragma unroll
        for (int t = 0; t < kTiles; ++t) {
            const unsigned char *p = row_at(sk, lk, __shfl(code, 16 * t + lr), kRowB, local_stride) + 16 * my_piece;
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) kx[t][kk] = *reinterpret_cast<const raw16 *>(p + 64 * kk);
        }
    };
    auto request_values = [&](int code) __attribute__((always_inline)) {
#pragma unroll
        for (int u = 0; u < NV; ++u) {
            const unsigned char *p = row_at(sv, lv, __shfl(code, value_row(u)), kRowB, local_stride) + (kBf16 ? lane % kPieces : lr) * 4 * kVW;
#pragma unroll
            for (int h = 0; h < kVH; ++h) vx[u][h] = *reinterpret_cast<const raw_v *>(p + 256 * h);
        }
    };

    float m_run = -INFINITY, l_run = 0.f; // of query lr; l_run: over the rows this lane holds
    f32x4 acc[NF]; // of query lr.  bf16: tile f, features 16 f + 4 lg + r.  fp32: tile (h, e), features 64 h + kVW (4 lg + r) + e
#pragma unroll
    for (int f = 0; f < NF; ++f) acc[f] = f32x4{0.f, 0.f, 0.f, 0.f};
    unsigned char *const buf = s_buf[wave];
    int code, ft; // of the block in hand
    // One block; the next one's keys and values are requested as soon as the registers of this one's are free.
    auto step = [&](auto more, int next) __attribute__((always_inline)) {
        // ---- scores S^T = K Q^T: query lr, rows 16 t + 4 lg + r ----
        f32x4 sc[kTiles];
        if constexpr (kQueryLds) asm volatile("" ::: "memory"); // (the queries are read again, not held)
        if constexpr (kBf16) {
#pragma unroll
            for (int t = 0; t < kTiles; ++t) {
                sc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
                for (int kk = 0; kk < KK; ++kk) {
                    if (!has_piece) kx[t][kk] = raw16{0u, 0u, 0u, 0u};
                    sc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, kx[t][kk]),
                                                                    __builtin_bit_cast(bf16x8, qb[kk]), sc[t], 0, 0, 0);
                }
            }
        } else { // sums of four terms each, joined pair by pair: one sum of D terms is 9.6e-7 from fp64 over 800 rows of 128
                 // features, of which the scores' share is most; this way 2.6e-7
            f32x4 part[KK];
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                f32x4 c[4];
                const raw16 qk = kQueryLds ? s_q[kk][lane] : qb[kQueryLds ? 0 : kk];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    c[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(kx[0][kk][e]), __uint_as_float(qk[e]),
                                                                f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                part[kk] = (c[0] + c[1]) + (c[2] + c[3]);
            }
#pragma unroll
            for (int n = KK; n > 1; n /= 2)
#pragma unroll
                for (int i = 0; i < n / 2; ++i) part[i] = part[2 * i] + part[2 * i + 1];
            sc[0] = part[0];
        }
        int code_next = 0, ft_next = 0;
        if constexpr (more.value) {
            __builtin_amdgcn_sched_barrier(0);
            find(next, &code_next, &ft_next);
            request_keys(code_next);
            __builtin_amdgcn_sched_barrier(0);
        }
        const bool late = __builtin_amdgcn_ballot_w64(ft > first_tok) != 0; // somebody does not see some row
        if (late) {
#pragma unroll
            for (int t = 0; t < kTiles; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    const int from = __shfl(ft, 16 * t + 4 * lg + r);
                    sc[t][r] = my_tok >= from ? sc[t][r] : -INFINITY;
                }
        }
        // ---- statistics and weights, all of query lr (a NaN score is in no maximum and makes the sum one).  What the
        // exponents subtract is a whole number, so that bringing sums from one to another multiplies by a power of two ----
        float mx = fmaxf(fmaxf(sc[0][0], sc[0][1]), fmaxf(sc[0][2], sc[0][3]));
        if constexpr (kTiles == 2) mx = fmaxf(mx, fmaxf(fmaxf(sc[1][0], sc[1][1]), fmaxf(sc[1][2], sc[1][3])));
        mx = ceilf(xrow_max(mx) * scale);
        if (__builtin_amdgcn_ballot_w64(mx > m_run) != 0) { // a maximum moved: bring what was summed to it
            const float m_new = fmaxf(m_run, mx);
            const float corr = m_run == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l_run *= corr;
#pragma unroll
            for (int f = 0; f < NF; ++f) acc[f] *= corr;
        }
        const float ref = m_run == -INFINITY ? 0.f : m_run;
        float p[4 * kTiles];
        if (__builtin_amdgcn_ballot_w64(fabsf(ref) > kLargeRef) != 0) { // somebody's is so large that its rounding shows
#pragma unroll
            for (int t = 0; t < kTiles; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if constexpr (kBf16)
                        p[4 * t + r] = __builtin_amdgcn_exp2f(fabsf(ref) > kLargeRef ? scaled_apart(sc[t][r], scale, ref) : fmaf(sc[t][r], scale, -ref));
                    else
                        p[4 * t + r] = weight_of_any(sc[t][r], scale, ref);
        } else {
#pragma unroll
            for (int t = 0; t < kTiles; ++t)
#pragma unroll
                for (int r = 0; r < 4; ++r) // (bf16 payloads: the output's own rounding is four orders above the difference's)
                    p[4 * t + r] = kBf16 ? __builtin_amdgcn_exp2f(fmaf(sc[t][r], scale, -ref)) : weight_of(sc[t][r], scale, ref);
        }
        float sum = (p[0] + p[1]) + (p[2] + p[3]);
        if constexpr (kTiles == 2) sum += (p[4] + p[5]) + (p[6] + p[7]);
        l_run += sum;
        if (late) { // what was read instead of a value row
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                const bool nowhere = __shfl(ft, value_row(u)) == INT_MAX;
#pragma unroll
                for (int h = 0; h < kVH; ++h)
#pragma unroll
                    for (int e = 0; e < kVW; ++e) vx[u][h][e] = nowhere ? 0u : vx[u][h][e];
            }
        }
        // ---- O^T += V^T P^T: the weights are the B operand as they stand in the lane ----
        if constexpr (kBf16) {
            raw16 hi, lo;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                hi[e] = bf16_pair(p[2 * e], p[2 * e + 1]);
                lo[e] = bf16_pair(p[2 * e] - __uint_as_float(hi[e] << 16), p[2 * e + 1] - __uint_as_float(hi[e] & 0xFFFF0000u));
            }
#pragma unroll
            for (int u = 0; u < NV; ++u) {
                const int row = value_row(u);
                *reinterpret_cast<raw_v *>(buf + row * kRowB + 16 * ((lane % kPieces) ^ row_swizzle<D>(row))) = vx[u][0];
            }
            if constexpr (more.value) request_values(code_next);
            asm volatile("" ::: "memory"); // a wave's LDS accesses keep their order; no other wave reads these rows
            const int q4 = lr >> 2, piece = (lane & 3) >> 1, sub = 8 * (lane & 1);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                const int r0 = 4 * lg + q4, r1 = r0 + 16;
                const i16x4 v0 = lds_read_tr16(buf + r0 * kRowB + 16 * ((2 * f + piece) ^ row_swizzle<D>(r0)) + sub);
                const i16x4 v1 = lds_read_tr16(buf + r1 * kRowB + 16 * ((2 * f + piece) ^ row_swizzle<D>(r1)) + sub);
                const bf16x8 av = __builtin_bit_cast(bf16x8, i16x8{v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]});
                acc[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, hi), acc[f], 0, 0, 0);
                acc[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, __builtin_bit_cast(bf16x8, lo), acc[f], 0, 0, 0);
            }
            asm volatile("" ::: "memory"); // the next block's rows take their place
        } else {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int h = 0; h < kVH; ++h) // (four rows at a time, joined pair by pair, then one addition to what was summed before)
#pragma unroll
                for (int e = 0; e < kVW; ++e) {
                    f32x4 d[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        d[u] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(vx[u][h][e]), p[u], f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                    acc[kVW * h + e] += (d[0] + d[1]) + (d[2] + d[3]);
                }
            if constexpr (more.value) {
                __builtin_amdgcn_sched_barrier(0);
                request_values(code_next);
            }
        }
        code = code_next;
        ft = ft_next;
    };
    if (b_lo + wave < b_hi) {
        int blk = b_lo + wave;
        find(blk, &code, &ft);
        request_keys(code);
        request_values(code);
        // the last block apart: a branch around the loads would make every wait in the loop one for all of them
        for (; blk + W < b_hi; blk += W) step(std::true_type{}, blk + W);
        step(std::false_type{}, 0);
    }
    // ---- the waves' results join in LDS ----
    const float l_sum = xrow_sum(l_run);
    if (lg == 0) {
        // (maxima leave NaN scores out: where there was nothing else the sum is still to be looked at)
        s_m[wave][lr] = m_run == -INFINITY && l_sum != 0.f ? 0.f : m_run;
        s_l[wave][lr] = l_sum;
    }
    constexpr int kQuads = D / 4; // 4-feature pieces of an output row, piece c of query n at c ^ (n % kQuads)
    f32x4(*const s_o)[kQuads] = reinterpret_cast<f32x4(*)[kQuads]>(buf);
#pragma unroll
    for (int f = 0; f < NF; ++f) {
        if constexpr (kBf16) {
            s_o[lr][(4 * f + lg) ^ (lr & (kQuads - 1))] = acc[f];
        } else if constexpr (kVW == 4) { // register r of the four tiles of h: features 64 h + 16 lg + 4 r ..
            const int h = f / 4, r = f % 4;
            s_o[lr][(16 * h + 4 * lg + r) ^ (lr & (kQuads - 1))] =
                f32x4{acc[4 * h][r], acc[4 * h + 1][r], acc[4 * h + 2][r], acc[4 * h + 3][r]};
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int d = kVW * (4 * lg + r) + f;
                s_o[lr][(d / 4) ^ (lr & (kQuads - 1))][d % 4] = acc[f][r];
            }
        }
    }
    __syncthreads();
    const int n_q_here = n_queries - qt * kAttQ < kAttQ ? n_queries - qt * kAttQ : kAttQ;
    for (int i = tid; i < n_q_here * kQuads; i += 64 * W) {
        const int n = i / kQuads, c = i - n * kQuads, qq = qt * kAttQ + n, tok = qq / a.G;
        float m = -INFINITY;
#pragma unroll
        for (int w = 0; w < W; ++w) m = fmaxf(m, s_m[w][n]);
        float l = 0.f;
        f32x4 o = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int w = 0; w < W; ++w) {
            const float lw = s_l[w][n];
            if (lw != 0.f) { // a wave none of whose rows the query sees has nothing to add (a NaN has)
                const float x = __builtin_amdgcn_exp2f(s_m[w][n] - m);
                l = fmaf(lw, x, l);
                const f32x4 ow = reinterpret_cast<const f32x4(*)[kQuads]>(s_buf[w])[n][c ^ (n & (kQuads - 1))];
#pragma unroll
                for (int e = 0; e < 4; ++e) o[e] = fmaf(ow[e], x, o[e]);
            }
        }
        const int64_t row = ((int64_t)b * a.n_q + tok) * a.Hq + g * a.G + (qq - tok * a.G);
        if (MERGE || a.n_split > 1) { // the split's record: [0] maximum, [1] normaliser, [2..] unnormalised output
            float *rec = a.part + (row * a.n_split + sp) * (D + 2);
            if constexpr (MERGE) {
                if (c == 0) store_far(rec, m, l);
                store_far(rec + 2 + 4 * c, o[0], o[1]);
                store_far(rec + 4 + 4 * c, o[2], o[3]);
            } else {
                if (c == 0) {
                    rec[0] = m;
                    rec[1] = l;
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) rec[2 + 4 * c + e] = o[e];
            }
        } else {
            const float den = l != 0.f ? l : 1.f;
            if constexpr (kBf16)
                *reinterpret_cast<u32x2 *>(out + row * D + 4 * c) = u32x2{bf16_pair(o[0] / den, o[1] / den), bf16_pair(o[2] / den, o[3] / den)};
            else
                *reinterpret_cast<f32x4 *>(out + row * D + 4 * c) = o / den;
            if (column_sums<T, D>() && a.pair_stride && c == 0)
                *reinterpret_cast<f32x2 *>(a.part + row * a.pair_stride) = l != 0.f ? f32x2{m, 1.f / l} : f32x2{0.f, 0.f};
        }
    }
    if constexpr (MERGE) {
        // ---- the shares' records: the last workgroup of the tile to get here does what attend_combine_kernel does ----
        __shared__ int s_last;
        if (!last_to_arrive(arrivals_of(a.part) + ((int)blockIdx.z * (int)gridDim.y + (int)blockIdx.y), a.n_split, &s_last)) return;
        for (int i = tid; i < n_q_here * kQuads; i += 64 * W) {
            const int n = i / kQuads, c = i - n * kQuads, qq = qt * kAttQ + n, tok = qq / a.G;
            const int64_t row = ((int64_t)b * a.n_q + tok) * a.Hq + g * a.G + (qq - tok * a.G);
            const float *rec = a.part + row * a.n_split * (D + 2);
            f32x2 st[kAttendMaxSplit], x0[kAttendMaxSplit], x1[kAttendMaxSplit]; // all requested before any is used
#pragma unroll
            for (int s = 0; s < kAttendMaxSplit; ++s) {
                if (s >= a.n_split) break;
                st[s] = load_far(rec + s * (D + 2));
                x0[s] = load_far(rec + s * (D + 2) + 2 + 4 * c);
                x1[s] = load_far(rec + s * (D + 2) + 4 + 4 * c);
            }
            float m = -INFINITY;
#pragma unroll
            for (int s = 0; s < kAttendMaxSplit; ++s)
                if (s < a.n_split) m = fmaxf(m, st[s][0]);
            float l = 0.f;
            f32x4 o = {0.f, 0.f, 0.f, 0.f};
            if (m > -INFINITY) {
#pragma unroll
                for (int s = 0; s < kAttendMaxSplit; ++s) {
                    if (s >= a.n_split) break;
                    const float x = st[s][0] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(st[s][0] - m);
                    l = fmaf(st[s][1], x, l);
                    o = f32x4{fmaf(x0[s][0], x, o[0]), fmaf(x0[s][1], x, o[1]), fmaf(x1[s][0], x, o[2]), fmaf(x1[s][1], x, o[3])};
                }
            }
            const bool seen = l != 0.f; // nobody's share holds a row that the query sees: zeros
            o = seen ? o / l : f32x4{0.f, 0.f, 0.f, 0.f};
            if constexpr (kBf16)
                *reinterpret_cast<u32x2 *>(out + row * D + 4 * c) = u32x2{bf16_pair(o[0], o[1]), bf16_pair(o[2], o[3])};
            else
                *reinterpret_cast<f32x4 *>(out + row * D + 4 * c) = o;
        }
    }
}

// out[b][i][h][:] = sum_s o_s 2^(m_s - m) / sum_s z_s 2^(m_s - m), m = max_s m_s; zero if no split saw a key, which
// is a denominator of exactly zero (a NaN or +inf score makes it a NaN, and the output with it)
// lse (may be null): log2 of the query's softmax denominator, in the scores' log2 units; +inf for a
// query that sees no key, so that every weight computed from it is zero.
// Part: const float *__restrict__, or float *: then the query's pair takes the place of its first record's start (see AttendArgs).
template <typename T, int D, typename Part>
__global__ void attend_combine_kernel(Part part, int n_split, T *__restrict__ out, float *__restrict__ lse) {
    constexpr bool kPairs = std::is_same<Part, float *>::value;
    const int64_t row = blockIdx.x;
    Part p = part + row * n_split * (D + 2);
    f32x2 pair = {0.f, 0.f};
    for (int d = threadIdx.x; d < D; d += blockDim.x) {
        // every record's maximum, normaliser and this thread's element requested before any is used
        float ms[kAttendMaxSplit], zz[kAttendMaxSplit], oo[kAttendMaxSplit];
#pragma unroll
        for (int s = 0; s < kAttendMaxSplit; ++s) {
            const float *ps = p + (s < n_split ? s : 0) * (D + 2);
            ms[s] = ps[0];
            zz[s] = ps[1];
            oo[s] = ps[2 + d];
        }
        float m = -INFINITY;
#pragma unroll
        for (int s = 0; s < kAttendMaxSplit; ++s)
            if (s < n_split) m = fmaxf(m, ms[s]);
        float zs = 0.f, os = 0.f;
        if (m > -INFINITY) {
#pragma unroll
            for (int s = 0; s < kAttendMaxSplit; ++s) {
                if (s >= n_split) break;
                const float w = ms[s] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(ms[s] - m);
                zs = fmaf(zz[s], w, zs);
                os = fmaf(oo[s], w, os);
            }
        }
        store_out(out + row * D + d, zs != 0.f ? os / zs : 0.f);
        if (lse && d == 0) lse[row] = zs != 0.f ? m + __builtin_amdgcn_logf(zs) : INFINITY;
        if (kPairs && zs != 0.f) pair = f32x2{m, 1.f / zs};
    }
    if constexpr (kPairs) {
        __syncthreads(); // the record has been read
        if (threadIdx.x == 0) *reinterpret_cast<f32x2 *>(p) = pair;
    }
}

// Softmax weights on the new tokens (the last n_q local rows of the question), added over a share of the queries, for the
// shapes of attend_kernel.  Grid (64 new tokens x share, KV head, question).  A wave keeps the keys of 16 tokens as the B
// operand in registers and its share's queries stream past, 16 at a time and requested one tile ahead, so S = Q K^T leaves a
// lane one key and four queries: no LDS, no barrier, and the sum over the queries is a running one until the end.  What bounds
// it is a tile's chain, query -> scores -> weights, with few waves to hide it, and uneven shares under the mask: 600 tokens over
// 768 rows, fp32, 44 us at 30 TFLOP/s, the matrix pipes busy a quarter of the time.  (With eight queries in LDS and a thread per
// key on the vector ALU, a layer call of fp32, 28 heads of 128 took: 32 tokens over 192 rows 28.6 us, now 19.7, 600 over 768 220, now 206; bf16
// rows of 32 features, 400 tokens 46, now 20.)
// colpart [B][Hkv][n_qs][n_q].
template <typename T, int D>
__global__ __launch_bounds__(kThreads) void prefill_colsum_kernel(AttendArgs a, float *__restrict__ colpart, int n_qs, int tiles_per) {
    constexpr bool kBf16 = sizeof(T) == 2;
    constexpr int kPieces = D * (int)sizeof(T) / 16, E = 16 / (int)sizeof(T), KK = kBf16 ? (D + 31) / 32 : D / 16;
    const int kt = blockIdx.x / n_qs, qs = blockIdx.x - kt * n_qs, g = blockIdx.y, b = blockIdx.z;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63, lr = lane & 15, lg = lane >> 4;
    const int j0 = kColKeys * kt + 16 * wave; // this wave's new tokens
    if (j0 >= a.n_q) return;
    const int n_queries = a.n_q * a.G; // of this KV head: (token, head in group), token-major
    const float scale = a.scale_log2e * (1.f / query_factor<T, D>());
    const int l0 = a.local_offsets[b];
    int n_loc = a.local_offsets[b + 1] - l0;
    if (n_loc < 0) n_loc = 0;
    // the lane's new token j is local row n_loc - n_q + j; it may not exist.  Query qq sees it iff qq >= q_min.
    const int j = j0 + lr, lrow = n_loc - a.n_q + j;
    const bool ok = j < a.n_q && lrow >= 0;
    const int q_min = !ok ? INT_MAX : a.causal ? j * a.G : 0;
    const bool has_piece = kPieces >= 4 || lg < kPieces; // (rows of 32 bytes have two pieces)
    const int my_piece = kPieces >= 4 ? lg : lg & (kPieces - 1);
    const int64_t base = (int64_t)b * a.n_q * a.Hq + g * a.G;
    const T *q = static_cast<const T *>(a.q) + base * D + my_piece * E;
    const T *kp = n_loc == 0 ? q : static_cast<const T *>(a.k_local) + ((int64_t)(l0 + (ok ? lrow : 0)) * a.Hkv + g) * D + my_piece * E; // (memory that exists)
    raw16 kx[KK], qx[KK], qn[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) {
        kx[kk] = brought_down<T, D>(load16(kp + 4 * kk * E)); // (the keys instead of the queries, once: the same products)
        if (!has_piece) kx[kk] = raw16{0u, 0u, 0u, 0u};
    }
    const int n_tiles = (n_queries + 15) / 16;
    const int t_end = (qs + 1) * tiles_per < n_tiles ? (qs + 1) * tiles_per : n_tiles;
    int t = qs * tiles_per;
    if (a.causal && j0 * a.G / 16 > t) t = j0 * a.G / 16; // nobody before token j0 sees these
    f32x2 s_cur = {0.f, 0.f}, s_next = {0.f, 0.f}; // of query lr: what its exponents subtract, 1 / sum of its weights
    auto request = [&](int tile, raw16 *x, f32x2 *s) __attribute__((always_inline)) {
        const int qq = 16 * tile + lr < n_queries ? 16 * tile + lr : n_queries - 1, tok = qq / a.G; // (past the last: masked)
        const int64_t row = (int64_t)tok * a.Hq + (qq - tok * a.G);
        *s = *reinterpret_cast<const f32x2 *>(a.part + (base + row) * a.pair_stride);
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) x[kk] = load16(q + row * D + 4 * kk * E);
    };
    float sum = 0.f;
    if (t < t_end) request(t, qx, &s_cur);
    for (; t < t_end; ++t) {
        if (t + 1 < t_end) request(t + 1, qn, &s_next);
        f32x4 sc;
        if constexpr (kBf16) {
            sc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                if (!has_piece) qx[kk] = raw16{0u, 0u, 0u, 0u};
                sc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, qx[kk]), __builtin_bit_cast(bf16x8, kx[kk]), sc, 0, 0, 0);
            }
        } else { // sums of four terms, joined pair by pair, as in attend_kernel
            f32x4 part[KK];
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) {
                f32x4 c[4];
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    c[e] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(qx[kk][e]), __uint_as_float(kx[kk][e]),
                                                                f32x4{0.f, 0.f, 0.f, 0.f}, 0, 0, 0);
                part[kk] = (c[0] + c[1]) + (c[2] + c[3]);
            }
#pragma unroll
            for (int n = KK; n > 1; n /= 2)
#pragma unroll
                for (int i = 0; i < n / 2; ++i) part[i] = part[2 * i] + part[2 * i + 1];
            sc = part[0];
        }
        // reference and normaliser apart, as the attention had them: their log2 in one number would be rounded at its size
        float w[4];
        if (__builtin_amdgcn_ballot_w64(fabsf(s_cur[0]) > kLargeRef) != 0) {
#pragma unroll
            for (int r = 0; r < 4; ++r) w[r] = weight_of_any(sc[r], scale, __shfl(s_cur[0], 4 * lg + r));
        } else {
#pragma unroll
            for (int r = 0; r < 4; ++r) w[r] = __builtin_amdgcn_exp2f(fmaf(sc[r], scale, -__shfl(s_cur[0], 4 * lg + r)));
        }
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const int qq = 16 * t + 4 * lg + r;
            const float x = w[r] * __shfl(s_cur[1], 4 * lg + r);
            w[r] = qq >= q_min && qq < n_queries ? x : 0.f;
        }
        sum += (w[0] + w[1]) + (w[2] + w[3]);
        s_cur = s_next;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) qx[kk] = qn[kk];
    }
    sum = xrow_sum(sum);
    if (lg == 0 && j < a.n_q) colpart[(((int64_t)b * a.Hkv + g) * n_qs + qs) * a.n_q + j] = sum;
}

// The work of prefill_keysum_kernel (below): key tile kt takes the queries from its first token's on (all of them
// without the mask), in steps of kCQ, shared out steps_per at a time.
constexpr int kCK = 128, kCQ = 64; // keys per workgroup, queries per step
__host__ __device__ inline int keysum_shares(int kt, int n_queries, int G, int causal, int steps_per) {
    const int steps = (n_queries - (causal ? kt * kCK * G : 0) + kCQ - 1) / kCQ;
    return (steps + steps_per - 1) / steps_per;
}

// signal[b][j] = (sum over KV heads and query tiles of colpart) / (Hq * n_q), in a fixed order: 32 columns
// per workgroup, the terms of a column split into 8 contiguous runs (one per group of 32 threads, 8 loads
// in flight), the runs joined in order.
constexpr int kSigCols = 32, kSigRuns = kThreads / kSigCols;
// Of the n_per terms of a KV head a column has the first n_valid(column): steps_per 0: all of them; otherwise the shares
// of its key tile.
__global__ __launch_bounds__(kThreads) void prefill_signal_kernel(const float *__restrict__ colpart, int Hkv, int n_per, int n_q,
                                                                  float inv, float *__restrict__ signal, int G, int causal,
                                                                  int steps_per) {
    __shared__ float s_run[kSigRuns][kSigCols];
    const int b = blockIdx.y, col = threadIdx.x % kSigCols, run = threadIdx.x / kSigCols;
    const int j = blockIdx.x * kSigCols + col;
    static_assert(kCK % kSigCols == 0, "the columns of a workgroup belong to one key tile");
    const int n_valid = steps_per ? keysum_shares(blockIdx.x * kSigCols / kCK, n_q * G, G, causal, steps_per) : n_per;
    const int n_terms = Hkv * n_valid;
    const int per = (n_terms + kSigRuns - 1) / kSigRuns;
    const int t0 = run * per, t1 = t0 + per < n_terms ? t0 + per : n_terms;
    float s = 0.f;
    if (j < n_q && t0 < t1) {
        const float *p = colpart + (int64_t)b * Hkv * n_per * n_q + j;
        if (n_valid == n_per) { // every term counts: they are evenly spaced
            for (int t = t0; t < t1; t += 8) {
                float v[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) v[u] = p[(int64_t)(t + u < t1 ? t + u : t1 - 1) * n_q];
#pragma unroll
                for (int u = 0; u < 8; ++u) s += t + u < t1 ? v[u] : 0.f;
            }
        }
        int g = t0 / n_valid, i = t0 - g * n_valid; // otherwise: the run's next term
        for (int t = n_valid == n_per ? t1 : t0; t < t1; t += 8) {
            float v[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                v[u] = p[((int64_t)g * n_per + i) * n_q];
                if (t + u + 1 < t1 && ++i == n_valid) {
                    i = 0;
                    ++g;
                }
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) s += t + u < t1 ? v[u] : 0.f;
        }
    }
    s_run[run][col] = s;
    __syncthreads();
    if (run == 0 && j < n_q) {
        float tot = s_run[0][col];
#pragma unroll
        for (int r = 1; r < kSigRuns; ++r) tot += s_run[r][col];
        signal[(int64_t)b * n_q + j] = tot * inv;
    }
}

// ------------------------------------------------------------------------------------------
// The prefill on the matrix cores (bf16 rows of 64 or 128 features): both products of the attention are
// dense contractions here, queries -- (token, head of the KV group) pairs -- against every row.
// One workgroup of four waves per (128 queries, KV head, question), a wave owns 32 queries from the scores
// to the output, so nothing crosses the waves but the staged rows:
//   rows     in steps of 64, keys and values double-buffered in LDS by the direct global -> LDS load (no
//            registers hold a row in flight); a step's loads are issued one step ahead, one barrier per step.
//            A row's 16-byte pieces are stored at piece ^ f(row) -- the permutation sits in the lanes' source
//            addresses -- so that the 16-byte operand reads of the keys (f = row) and the transpose reads of
//            the values (f spreads the 4 rows of a 4 x 16 tile over the banks) are free of conflicts.
//   scores   S^T = K Q^T with v_mfma_f32_32x32x16_bf16, the keys as the A operand from LDS, the queries as the
//            B operand in registers: a lane holds ONE query (lane % 32) and the rows 8 (j / 4) + 4 (lane / 32) +
//            j % 4 of every 32, so a query's statistics are in-lane work and one exchange between the halves.
//   values   O^T += V^T P^T: the weights are the B operand as they stand in the lane -- the order in which the
//            product walks the rows is free, so the A operand (LDS transpose reads of the values) takes them in
//            the order the lane holds them: reduction slots 8 h + i of a 16-row step are rows 4 h + i (i < 4) and
//            8 + 4 h + i - 4.  No weight passes through LDS.
// The exponent subtracts the running maximum itself: the largest weight is then 1, which bf16 holds exactly (a
// reference that lags behind it by up to 2^8 saves most of the rescaling, but where one row dominates its weight gets
// a rounding error: 2.2e-3 from an fp64 evaluation against 1.7e-3).  The output is rescaled only in steps where a
// maximum of the wave's queries moved.  (Rows of 64 features: the weights are bf16 pairs hi + lo, as in the kernels
// that take the other shapes, so nothing of the fp32 weight is lost.)  Only steps with a row that some query of the tile may not see look at the mask.
// ------------------------------------------------------------------------------------------
// The direct global -> LDS load: 16 bytes per lane from the lane's address to dst + 16 * lane (dst is the same in all
// lanes).  The instruction has no destination register, only addresses, which are read when it issues.  It is not the
// builtin because the compiler makes every later LDS read wait for that one, which would end the overlap of a step's
// loads with the step before: here rows_landed() and a barrier stand between a load and the first read of its rows.
__device__ __forceinline__ void load_to_lds(const unsigned char *src, unsigned char *dst) {
    const unsigned base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)dst;
    unsigned saved; // m0, which carries the LDS address, is left as it was
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %2, off\n\ts_mov_b32 m0, %0"
                 : "=&s"(saved)
                 : "s"(base), "v"(src)
                 : "memory");
}
__device__ __forceinline__ void load4_to_lds(const float *src, float *dst) { // 4 bytes per lane
    const unsigned base = (unsigned)(uintptr_t)(__attribute__((address_space(3))) float *)dst;
    unsigned saved;
    asm volatile("s_mov_b32 %0, m0\n\ts_mov_b32 m0, %1\n\ts_nop 0\n\tglobal_load_lds_dword %2, off\n\ts_mov_b32 m0, %0"
                 : "=&s"(saved)
                 : "s"(base), "v"(src)
                 : "memory");
}
__device__ __forceinline__ void rows_landed() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }
// over the two lanes lane % 32 and lane % 32 + 32, result in both
__device__ __forceinline__ float half_max(float v) {
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return fmaxf(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float half_sum(float v) {
    auto b = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

constexpr int kFK = 64, kFQ = 128; // rows per step, queries per workgroup
// Most new tokens of which an unsplit attention kernel sums Eq. 1 itself (a multiple of 64).  The key sums' launch costs
// more than the tile's own last steps while these are one or two (7B head layout, no past, us a call, here / in a launch
// of its own: 32 tokens 8.6 / 11.9, 64: 9.1 / 12.4, 128: 11.6 / 14.5); with more, the last tile's chain is the launch's
// (196 tokens: 18.6 / 17.5).
constexpr int kFusedSums = 128;
constexpr float kHidden = -1e30f, kFloor = -1e20f; // score of a row a query may not see; least running maximum

// Slot of 16-byte piece `piece` of staged row `row` in a row of D * 2 bytes.
template <int D>
__device__ __forceinline__ int key_slot(int piece, int row) {
    // 16 lanes read one piece of 16 neighbouring rows: 256 B over all banks
    return D == 128 ? piece ^ (row & 15) : piece ^ ((row >> 1) & 7);
}
template <int D>
__device__ __forceinline__ int val_slot(int piece, int row) {
    // half a wave reads 4 pieces of 4 neighbouring rows (4-aligned both)
    return D == 128 ? piece ^ (((row & 3) << 2) | ((row >> 2) & 3)) : piece ^ (((row >> 1) & 1) << 2);
}

// Workgroup -> (tile, combination of KV head and question).  Workgroup id runs on XCD id % 8; the rows of a
// combination are read by all of its tiles, so where the counts allow it a combination stays on as few XCDs
// as there are for it (its rows then sit in those L2 caches).  The last tiles, under the causal mask the heavy ones,
// start first.  Returns false for the padding workgroups.
__device__ __forceinline__ bool tile_of(unsigned id, int n_tiles, int combos, int *tile, int *combo) {
    const unsigned xcd = id & 7, slot = id >> 3;
    int rank;
    if (8 % combos == 0) {
        const int per = 8 / combos;
        *combo = xcd / per;
        rank = slot * per + xcd % per;
    } else if (combos % 8 == 0) {
        const unsigned m = combos / 8;
        *combo = (slot % m) * 8 + xcd;
        rank = slot / m;
    } else {
        *combo = id % combos;
        rank = id / combos;
    }
    *tile = n_tiles - 1 - rank;
    return rank < n_tiles;
}
// Workgroups of two fours per combination: a tile each, and where there are more tiles than compute units as many as those.
__host__ __device__ __forceinline__ int pairs_grid(int n_tiles, int combos) {
    const int places = 256 / combos;
    return n_tiles <= places ? n_tiles : places;
}
unsigned tile_grid(int n_tiles, int combos) {
    if (8 % combos == 0) {
        const int per = 8 / combos;
        return (unsigned)((n_tiles + per - 1) / per) * 8u;
    }
    return (unsigned)((int64_t)n_tiles * combos);
}

// What bounds it: the latency of a wave's chain scores -> statistics -> weights -> values, with two waves per SIMD to
// hide it (254 registers, 80 KB of LDS): a 64-row step of a workgroup alone on its compute unit takes 2850 cycles for
// 1024 of matrix work (64-query tiles of 16x16x32 products whose weights cross the waves through LDS: 1568 new tokens over 768
// rows, 7B head layout, 186 us with the column sums, which are 23 us in the kernel below; 4000 tokens 269 us for the whole call
// against 673).
// FOURS = 2: eight waves, of which four take the even steps and four the odd ones, with rows and tables of their own (158 KB of
// LDS, one workgroup per compute unit), and join at the end: a tile's chain is half as long, which is what counts where there
// are no more tiles than compute units (600 tokens over 768 rows 44.4 -> 39.4 us a call).  Where there are somewhat
// more the smallest tiles take a four each, two to a workgroup, at the larger one's barriers: under the mask every compute unit then
// has about the same to do (1568 tokens, 344 tiles, 79.7 -> 72.5 us a call, 54 of them here, its matrix pipes busy 40 % of the time).
// flash_split says where.  Also built and slower, measured with four waves and 1568 tokens at 60-64 us a launch: the next block's
// scores interleaved instruction by instruction with this block's weights and values (66 us), 64 queries per wave (85 us: the
// accumulators pass 256 registers and are moved in and out of the accumulation registers).
// SPLIT: a short prefill has too few tiles to fill the chip, so its rows are shared by n_split workgroups per
// tile; the split's (maximum, normaliser, unnormalised output) go to the records attend_combine_kernel merges
// (aux = records).  Otherwise the output is final here, and so are the log-sum-exps: they go to aux for the key sums'
// launch, or (SUMS, few new tokens) Eq. 1 is summed right here, over the tile's queries, and goes to aux
// [B][Hkv][n_tiles][n_q].
template <int D, int FOURS, bool SPLIT, bool SUMS>
__global__ __launch_bounds__(256 * FOURS) __attribute__((amdgpu_waves_per_eu(D == 128 || FOURS == 2 ? 2 : 3, D == 128 || FOURS == 2 ? 2 : 3))) void prefill_flash_kernel(
    AttendArgs a, uint16_t *__restrict__ out, int n_tiles, int combos, float *__restrict__ aux, int n_split) {
    using T = uint16_t;
    constexpr int kRowB = D * 2, kPieces = kRowB / 16, kRowsPerLoad = 64 / kPieces; // rows one load of a wave brings
    constexpr int kLoads = kFK / 4 / kRowsPerLoad;                                   // such loads per wave and step
    constexpr int KK = D / 16, NF = D / 32; // 16-feature steps of the scores, 32-feature blocks of the output
    constexpr bool kPairs = D == 64;        // weights as bf16 pairs hi + lo
    // every four waves have staged rows and tables of their own
    __shared__ __align__(1024) unsigned char s_kk[FOURS][2][kFK * kRowB];
    __shared__ __align__(1024) unsigned char s_vv[FOURS][2][kFK * kRowB];
    constexpr int kRing = 8;                                    // steps whose row tables are held
    __shared__ ulonglong2 s_addrs[FOURS][kRing][kFK];           // addresses of the row's key and value
    __shared__ __align__(16) int s_fts[FOURS][kRing][kFK];      // first token that sees the row
    __shared__ int s_maskeds[FOURS][kRing];                     // some query of the tile may not see some row of the step
    __shared__ int s_frame[kMaxGatherK]; // the question's frames; -1: names no frame of the cache
    static_assert(!(SPLIT && SUMS) && !(FOURS == 2 && (SPLIT || SUMS)), "the sums want final statistics, the two fours have no shares");
    __shared__ __align__(16) float s_lse[SUMS ? kFQ : 1];
    const int tid = threadIdx.x, lane = tid & 63, lq = lane & 31, half = lane >> 5;
    const int four = FOURS == 2 ? __builtin_amdgcn_readfirstlane(tid >> 8) : 0, wave = __builtin_amdgcn_readfirstlane(tid >> 6) & 3;
    const int n_wgs = FOURS == 2 ? pairs_grid(n_tiles, combos) : SPLIT ? n_tiles * n_split : n_tiles; // per combination
    int tile_id, combo;
    if (!tile_of(blockIdx.x, n_wgs, combos, &tile_id, &combo)) return;
    // two fours: the first workgroups take a tile together, the others one each (the smallest with the largest that is left)
    const int n_pairs = FOURS == 2 ? n_tiles - n_wgs : 0, left = n_pairs - 1 - tile_id;
    const bool joint = FOURS == 2 && left < 0;
    const int qt_most = FOURS == 2 ? (joint ? tile_id + n_pairs : 2 * n_pairs - 1 - left) : 0; // the tile with the most steps here
    const int qt = FOURS == 2 ? (joint || four == 0 ? qt_most : left) : SPLIT ? tile_id / n_split : tile_id, sp = SPLIT ? tile_id % n_split : 0;
    const int g = combo % a.Hkv, b = combo / a.Hkv;
    auto &s_k = s_kk[four], &s_v = s_vv[four];
    auto &s_addr = s_addrs[four];
    auto &s_ft = s_fts[four];
    auto &s_masked = s_maskeds[four];
    const int n_queries = a.n_q * a.G;
    const T *q = static_cast<const T *>(a.q);
    for (int i = tid; i < a.k_frame; i += 256 * FOURS) {
        const int f = a.frame_idx[(int64_t)b * a.k_frame + i];
        s_frame[i] = (f >= 0 && f < a.n_frames) ? f : -1;
    }
    // the wave's 32 queries as a matrix operand (row / column lane % 32, 8 features from 8 * half of every 16)
    bf16x8 qb[KK];
    const int my_q = qt * kFQ + 32 * wave + lq;
    const bool q_ok = my_q < n_queries;
    const int my_tok = q_ok ? my_q / a.G : INT_MIN; // nothing is visible to a query that does not exist
    const int64_t my_row = ((int64_t)b * a.n_q + (q_ok ? my_tok : 0)) * a.Hq + g * a.G + (q_ok ? my_q - my_tok * a.G : 0);
    {
        const T *qp = q + my_row * D + 8 * half;
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) {
            raw16 u = load16(qp + 16 * kk);
            if (!q_ok) u = raw16{0u, 0u, 0u, 0u};
            qb[kk] = __builtin_bit_cast(bf16x8, u);
        }
    }
    const int n_ret = a.k_frame * a.kappa;
    const int l0 = __builtin_amdgcn_readfirstlane(a.local_offsets[b]); // the same in all lanes: scalar registers
    int n_loc = __builtin_amdgcn_readfirstlane(a.local_offsets[b + 1]) - l0;
    if (n_loc < 0) n_loc = 0;
    const int total = n_ret + n_loc;
    const unsigned char *sk = static_cast<const unsigned char *>(a.store_k) + (int64_t)g * a.store_cap * kRowB;
    const unsigned char *sv = static_cast<const unsigned char *>(a.store_v) + (int64_t)g * a.store_cap * kRowB;
    const unsigned char *lk = static_cast<const unsigned char *>(a.k_local) + g * kRowB;
    const unsigned char *lv = static_cast<const unsigned char *>(a.v_local) + g * kRowB;
    const unsigned local_stride = (unsigned)a.Hkv * kRowB;
    const int first_tok = (qt * kFQ) / a.G;
    const int last_q = (qt * kFQ + kFQ - 1 < n_queries ? qt * kFQ + kFQ - 1 : n_queries - 1) / a.G;

    // with the causal mask the rows after a tile's last token are seen by none of its queries
    auto seen_by = [&](int last_tok) {
        if (!a.causal) return total;
        // local rows up to the tile's last token; the retrieved rows are seen by every token, also by
        // tokens that have no local row of their own (fewer local rows than new tokens)
        int ns = n_ret + n_loc - a.n_q + last_tok + 1;
        if (ns < n_ret) ns = n_ret;
        return ns < total ? ns : total;
    };
    // (two fours on one tile: an odd step out is joined by one whose rows nobody of the tile sees)
    auto steps_of = [&](int rows) { return joint ? (rows + 2 * kFK - 1) / (2 * kFK) : (rows + kFK - 1) / kFK; };
    const int n_seen = seen_by(last_q);

    // Row r of [retrieved rows, local rows]: where its key and value live and the first token that sees it, worked
    // out by the lanes of one wave, four steps at a time (one per wave).  A row that lives nowhere, or past the last that a query
    // of the tile sees, is seen by nobody and reads a row that exists; its weight is zero, but zero times a NaN is not, so that row is one
    // that every query sees anyway (the first retrieved one; without any, the first local one, which is seen by all that
    // see something; with neither, the slab's first row, and nobody sees anything).
    int first_frame = a.k_frame > 0 ? __builtin_amdgcn_readfirstlane(a.frame_idx[(int64_t)b * a.k_frame]) : -1;
    if (first_frame >= a.n_frames) first_frame = -1;
    auto find_first_frame = [&]() { // where the list does not start with one: the same in all lanes
        for (int i0 = 0; i0 < a.k_frame && first_frame < 0; i0 += 64) {
            const int f = i0 + lane < a.k_frame ? s_frame[i0 + lane] : -1;
            const uint64_t some = __builtin_amdgcn_ballot_w64(f >= 0);
            if (some) first_frame = __builtin_amdgcn_readlane(f, __builtin_ctzll(some));
        }
    };
    const unsigned char *pad_k = sk, *pad_v = sv;
    auto find_pad = [&]() {
        if (first_frame < 0) find_first_frame();
        if (first_frame < 0 && n_loc == 0) return;
        const uint64_t off = first_frame < 0 ? (uint64_t)(unsigned)l0 * local_stride : (uint64_t)(unsigned)(first_frame * a.kappa) * kRowB;
        pad_k = (first_frame < 0 ? lk : sk) + off;
        pad_v = (first_frame < 0 ? lv : sv) + off;
    };
    auto tabulate = [&](int t) {
        const int slot = t & (kRing - 1), r = (joint ? 2 * t + four : t) * kFK + lane;
        const unsigned char *rk = pad_k, *rv = pad_v;
        int ft = INT_MAX;
        if (r < n_ret) {
            const int e = (int)((unsigned)r / (unsigned)a.kappa);
            const int f = s_frame[e];
            if (f >= 0) {
                const uint64_t off = (uint64_t)(unsigned)(f * a.kappa + (r - e * a.kappa)) * kRowB;
                rk = sk + off;
                rv = sv + off;
                ft = 0;
            }
        } else if (r < n_seen) {
            const int j = r - n_ret;
            const uint64_t off = (uint64_t)(unsigned)(l0 + j) * local_stride;
            rk = lk + off;
            rv = lv + off;
            ft = a.causal ? j - (n_loc - a.n_q) : 0;
        }
        s_addr[slot][lane] = ulonglong2{(uint64_t)(uintptr_t)rk, (uint64_t)(uintptr_t)rv};
        s_ft[slot][lane] = ft;
        const bool any = __builtin_amdgcn_ballot_w64(ft > first_tok) != 0;
        if (lane == 0) s_masked[slot] = any;
    };
    // A wave brings rows 16 wave .. 16 wave + 15 of the step, kRowsPerLoad at a time.
    const int ld_row = 16 * wave + lane / kPieces, ld_piece = lane % kPieces;
    unsigned kswz[kLoads], vswz[kLoads];
#pragma unroll
    for (int u = 0; u < kLoads; ++u) {
        kswz[u] = 16 * key_slot<D>(ld_piece, ld_row + u * kRowsPerLoad);
        vswz[u] = 16 * val_slot<D>(ld_piece, ld_row + u * kRowsPerLoad);
    }
    auto look_up = [&](int t, ulonglong2(&ad)[kLoads]) {
#pragma unroll
        for (int u = 0; u < kLoads; ++u) ad[u] = s_addr[t & (kRing - 1)][ld_row + u * kRowsPerLoad];
    };
    auto request = [&](int u, const ulonglong2(&ad)[kLoads], unsigned char *dk, unsigned char *dv) __attribute__((always_inline)) {
        const int lds = (16 * wave + u * kRowsPerLoad) * kRowB; // the wave's 1024 bytes, lane order
        load_to_lds(reinterpret_cast<const unsigned char *>(ad[u].x + kswz[u]), dk + lds);
        load_to_lds(reinterpret_cast<const unsigned char *>(ad[u].y + vswz[u]), dv + lds);
    };
    // this lane's offsets in a staged buffer: key operand of 16-feature step kk (rows lq, lq + 32 share the slot)
    int koff[KK];
#pragma unroll
    for (int kk = 0; kk < KK; ++kk) koff[kk] = lq * kRowB + 16 * key_slot<D>(2 * kk + half, lq);

    const bool idle = qt * kFQ + 32 * wave >= n_queries; // a wave without queries (its operand reads alone slow the others)
    float m_run = kFloor, l_run = 0.f; // of query lq; l_run: over the rows this lane holds
    f32x16 o[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int j = 0; j < 16; ++j) o[f][j] = 0.f;

    const int n_steps_all = steps_of(n_seen);
    // this workgroup's steps: all of them, or its share of them
    const int per_split = SPLIT ? (n_steps_all + n_split - 1) / n_split : n_steps_all;
    const int t_lo = SPLIT ? sp * per_split : 0;
    const int n_steps = t_lo + per_split < n_steps_all ? t_lo + per_split : n_steps_all;
    __syncthreads(); // the frame list is there
    find_pad();
    tabulate(t_lo + wave);
    tabulate(t_lo + wave + 4);
    __syncthreads();
    if (t_lo < n_steps) {
        ulonglong2 ad[kLoads];
        look_up(t_lo, ad);
#pragma unroll
        for (int u = 0; u < kLoads; ++u) request(u, ad, s_k[0], s_v[0]);
    }
    // One step: the rows in ck / cv are used while those of step t + 1 are on their way into nk / nv.
    auto step = [&](int t, const unsigned char *ck, const unsigned char *cv, unsigned char *nk,
                    unsigned char *nv) __attribute__((always_inline)) {
        ulonglong2 ad[kLoads];
        look_up(t + 1, ad);
        const int masked = s_masked[t & (kRing - 1)];
        rows_landed();   // this wave's rows of step t are in LDS
        __syncthreads(); // everybody's are; every wave is done with step t-1
        const bool more = t + 1 < n_steps; // its loads are issued between the groups of matrix instructions
        // tables of the steps before t are free: four new ones every four steps
        if (((t - t_lo) & 3) == 0 && t > t_lo && t + 4 < n_steps) tabulate(t + 4 + wave);
        if (SUMS && idle) { // brings its rows and leaves the LDS to the others
            if (more) {
#pragma unroll
                for (int u = 0; u < kLoads; ++u) request(u, ad, nk, nv);
            }
            return;
        }
        // Operands are requested one group of matrix instructions ahead (the barriers keep the compiler's order to it):
        // 16 features of both blocks of 32 rows.
        f32x16 sc[2];
#pragma unroll
        for (int j = 0; j < 16; ++j) sc[0][j] = sc[1][j] = 0.f;
        bf16x8 ak[2][2][2];
        auto load_k = [&](int grp) {
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
                    ak[grp & 1][i][kb] = *reinterpret_cast<const bf16x8 *>(ck + koff[2 * grp + i] + 32 * kRowB * kb);
        };
        load_k(0);
#pragma unroll
        for (int grp = 0; grp < KK / 2; ++grp) {
            if (grp + 1 < KK / 2) load_k(grp + 1);
            if (grp < kLoads && more) request(grp, ad, nk, nv);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
                    sc[kb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ak[grp & 1][i][kb], qb[2 * grp + i], sc[kb], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        }
        bf16x8 av[2][NF]; // value operands of 16 rows, also one group ahead
        auto load_v = [&](int grp) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                // rows 4 half + (lane % 16) / 4 and 8 later, 4 features per lane
                const int row = 16 * grp + 4 * half + ((lane & 15) >> 2);
                const int piece = 4 * f + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1), sub = 8 * (lane & 1);
                const i16x4 lo = lds_read_tr16(cv + row * kRowB + 16 * val_slot<D>(piece, row) + sub);
                const i16x4 hi = lds_read_tr16(cv + (row + 8) * kRowB + 16 * val_slot<D>(piece, row + 8) + sub);
                av[grp & 1][f] = __builtin_bit_cast(bf16x8, i16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
            }
        };
        load_v(0);
        // Scores stay unscaled (the factor to log2 units sits in the exponent's multiply-add); a row a query
        // may not see scores kHidden, and the running maximum never drops below kFloor: exp2 of the difference is an
        // exact zero for hidden rows, and a query that has seen nothing yet sums zeros.
        if (__builtin_amdgcn_readfirstlane(masked)) {
#pragma unroll
            for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const i32x4 ft = *reinterpret_cast<const i32x4 *>(&s_ft[t & (kRing - 1)][32 * kb + 8 * jj + 4 * half]);
#pragma unroll
                    for (int r = 0; r < 4; ++r) sc[kb][4 * jj + r] = my_tok >= ft[r] ? sc[kb][4 * jj + r] : kHidden;
                }
        }
        float m4[4];
#pragma unroll
        for (int c = 0; c < 4; ++c) m4[c] = fmaxf(sc[0][c], sc[1][c]);
#pragma unroll
        for (int j = 4; j < 16; ++j) m4[j & 3] = fmaxf(fmaxf(m4[j & 3], sc[0][j]), sc[1][j]);
        const float mx = half_max(fmaxf(fmaxf(m4[0], m4[1]), fmaxf(m4[2], m4[3]))) * a.scale_log2e;
        if (__builtin_amdgcn_ballot_w64(mx > m_run) != 0) { // a maximum moved: bring what was summed to it
            const float m_new = fmaxf(m_run, mx);
            const float corr = __builtin_amdgcn_exp2f(m_run - m_new);
            m_run = m_new;
            l_run *= corr;
#pragma unroll
            for (int f = 0; f < NF; ++f)
#pragma unroll
                for (int j = 0; j < 16; ++j) o[f][j] *= corr;
        }
        bf16x8 pw[2], pl[2];
        auto weights = [&](int grp) { // of 16 rows
            float p[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) p[e] = __builtin_amdgcn_exp2f(fmaf(sc[grp >> 1][8 * (grp & 1) + e], a.scale_log2e, -m_run));
            l_run += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
            raw16 u;
#pragma unroll
            for (int e = 0; e < 4; ++e) u[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{p[2 * e], p[2 * e + 1]}, bf16x2));
            pw[grp & 1] = __builtin_bit_cast(bf16x8, u);
            if constexpr (kPairs) {
                raw16 w;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    w[e] = __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2{p[2 * e] - __uint_as_float(u[e] << 16),
                                                                                      p[2 * e + 1] - __uint_as_float(u[e] & 0xFFFF0000u)}, bf16x2));
                pl[grp & 1] = __builtin_bit_cast(bf16x8, w);
            }
        };
        weights(0);
#pragma unroll
        for (int grp = 0; grp < 4; ++grp) {
            if (grp < 3) load_v(grp + 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int f = 0; f < NF; ++f)
            {
                o[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[grp & 1][f], pw[grp & 1], o[f], 0, 0, 0);
                if constexpr (kPairs) o[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[grp & 1][f], pl[grp & 1], o[f], 0, 0, 0);
            }
            if (grp < 3) weights(grp + 1);
            __builtin_amdgcn_sched_barrier(0);
        }
    };
    for (int t = t_lo; t < n_steps; t += 2) {
        step(t, s_k[0], s_v[0], s_k[1], s_v[1]);
        if (t + 1 < n_steps) step(t + 1, s_k[1], s_v[1], s_k[0], s_v[0]);
    }
    if (FOURS == 2 && !joint && four == 1) { // its tile is the smaller one: the other four's barriers
        const int last = (qt_most * kFQ + kFQ - 1 < n_queries ? qt_most * kFQ + kFQ - 1 : n_queries - 1) / a.G;
        for (int t = n_steps; t < steps_of(seen_by(last)); ++t) __syncthreads();
    }
    float l_sum = half_sum(l_run);
    // Two waves of the same queries join: each hands the other the output blocks it does not finish itself, four floats a lane at
    // [piece][lane], where the staged rows were; the ones it finishes are then its first.
    constexpr int kJoint = NF / 2;
    if (FOURS == 2 && joint) {
        __shared__ float s_stat[2][2][kFQ];
        static_assert(kJoint * 16 * 64 * sizeof(float) <= sizeof(s_kk[0]) / 4, "a wave's quarter of its four's keys");
        f32x4 *const box = reinterpret_cast<f32x4 *>(s_kk[four]) + wave * (kJoint * 4 * 64);
        __syncthreads(); // every wave is done with the keys
#pragma unroll
        for (int f = 0; f < kJoint; ++f)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                f32x4 x;
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    x[r] = four == 0 ? o[kJoint + f][4 * c + r] : o[f][4 * c + r];
                    o[f][4 * c + r] = four == 0 ? o[f][4 * c + r] : o[kJoint + f][4 * c + r];
                }
                box[(4 * f + c) * 64 + lane] = x;
            }
        if (half == 0) {
            s_stat[0][four][32 * wave + lq] = m_run;
            s_stat[1][four][32 * wave + lq] = l_sum;
        }
        __syncthreads();
        const f32x4 *const other = reinterpret_cast<const f32x4 *>(s_kk[FOURS == 2 ? 1 - four : 0]) + wave * (kJoint * 4 * 64);
        const float m2 = s_stat[0][1 - four][32 * wave + lq], l2 = s_stat[1][1 - four][32 * wave + lq];
        const float m = fmaxf(m_run, m2); // (sums of nothing have the least maximum, and a factor of zero)
        const float c1 = __builtin_amdgcn_exp2f(m_run - m), c2 = __builtin_amdgcn_exp2f(m2 - m);
        l_sum = four == 0 ? fmaf(l2, c2, l_sum * c1) : fmaf(l_sum, c1, l2 * c2); // the same bits in both
        m_run = m;
#pragma unroll
        for (int f = 0; f < kJoint; ++f)
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const f32x4 x = other[(4 * f + c) * 64 + lane];
#pragma unroll
                for (int r = 0; r < 4; ++r) o[f][4 * c + r] = fmaf(x[r], c2, o[f][4 * c + r] * c1);
            }
    }
    const bool seen = l_sum != 0.f; // a query that saw nothing leaves zeros, whatever its hidden rows held; NaN stays NaN
    // feature 32 f + 8 jj + 4 half + r of the query is in register 4 jj + r of block f
    if constexpr (SPLIT) { // the split's record: [0] maximum, [1] normaliser, [2..] unnormalised output
        if (!q_ok) return;
        float *rec = aux + (my_row * n_split + sp) * (D + 2);
        if (half == 0) {
            rec[0] = m_run;
            rec[1] = l_sum;
        }
#pragma unroll
        for (int f = 0; f < NF; ++f)
#pragma unroll
            for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                for (int r = 0; r < 4; ++r) rec[2 + 32 * f + 8 * jj + 4 * half + r] = seen ? o[f][4 * jj + r] : 0.f;
    } else {
        // Eq. 1 of the tile: the wave's queries (now the A operand: S = Q K^T) against the new tokens' keys, 64 at a time.
        // New token j is local row n_loc - n_q + j; it may not exist.  The last two steps' keys are still in LDS, which are
        // all there are for up to 64 new tokens; others come from memory (the L2 cache).
        const int j_end = a.causal && last_q + 1 < a.n_q ? last_q + 1 : a.n_q; // later tokens get nothing from here
        const int r_new0 = n_ret + n_loc - a.n_q;
        bf16x8 kb[SUMS ? 2 : 1][KK];
        int q_min[2]; // queries of the KV head before this one do not see the lane's key
        auto load_keys = [&](int j0) {
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int j = j0 + 32 * i + lq, lrow = n_loc - a.n_q + j;
                const bool ok = j < a.n_q && lrow >= 0;
                q_min[i] = !ok ? n_queries : (a.causal ? j * a.G : 0);
                if ((r_new0 + j0 > 0 ? r_new0 + j0 : 0) >= (n_steps - 2) * kFK) { // (masked keys: whatever is there)
                    const int row = (r_new0 + j) & (2 * kFK - 1);
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk)
                        kb[i][kk] = *reinterpret_cast<const bf16x8 *>(s_k[0] + row * kRowB + 16 * key_slot<D>(2 * kk + half, row));
                } else {
                    const T *kp = static_cast<const T *>(a.k_local) + ((int64_t)(l0 + (ok ? lrow : 0)) * a.Hkv + g) * D + 8 * half;
                    if (n_loc == 0) kp = q + 8 * half; // memory that exists
#pragma unroll
                    for (int kk = 0; kk < KK; ++kk) kb[i][kk] = __builtin_bit_cast(bf16x8, load16(kp + 16 * kk));
                }
            }
        };
        if constexpr (SUMS) {
            if (!idle) load_keys(0);
        }
        const float inv = 1.0f / l_sum, lse = seen ? m_run + __builtin_amdgcn_logf(l_sum) : INFINITY;
        {
            // a lane holds features 8 jj + 4 half .. + 3: the halves swap, so that it stores 16 bytes in a row (in 8-byte
            // stores twice as many lines are opened twice as often: 32 tokens without a past 9.9 us a call, now 8.8)
            uint16_t *op = out + my_row * D + 8 * half + (joint ? 32 * kJoint * four : 0);
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                if (FOURS == 2 && joint && f >= kJoint) break; // the other wave's
#pragma unroll
                for (int jj = 0; jj < 4; jj += 2) {
                    raw16 w;
#pragma unroll
                    for (int e = 0; e < 2; ++e) {
                        uint32_t pk[2];
#pragma unroll
                        for (int u = 0; u < 2; ++u)
                            pk[u] = bf16_pair(o[f][4 * (jj + u) + 2 * e] * inv, o[f][4 * (jj + u) + 2 * e + 1] * inv);
                        auto sw = __builtin_amdgcn_permlane32_swap(pk[0], pk[1], false, false);
                        w[e] = sw[0];
                        w[2 + e] = sw[1];
                    }
                    if (!seen) w = raw16{0u, 0u, 0u, 0u};
                    if (q_ok) *reinterpret_cast<raw16 *>(op + 32 * f + 8 * jj) = w;
                }
            }
            if (!SUMS && q_ok && half == 0 && !(joint && four == 1)) aux[my_row] = lse;
        }
        if constexpr (SUMS) {
            float(*s_col)[kFusedSums] = reinterpret_cast<float(*)[kFusedSums]>(s_vv); // per wave, where the values were
            static_assert(4 * kFusedSums * sizeof(float) <= sizeof(s_vv), "a sum per wave and new token");
            const int qq0 = qt * kFQ + 32 * wave;
            if (half == 0) s_lse[32 * wave + lq] = lse; // read by this wave only
            __syncthreads();                            // every wave is done with the values
            f32x4 l4[4];
#pragma unroll
            for (int jj = 0; jj < 4; ++jj) l4[jj] = *reinterpret_cast<const f32x4 *>(&s_lse[32 * wave + 8 * jj + 4 * half]);
            if (idle) {
                for (int j = lane; j < kFusedSums; j += 64) s_col[wave][j] = 0.f;
            }
            for (int j0 = idle ? j_end : 0; j0 < j_end; j0 += 64) {
                f32x16 sc[2];
#pragma unroll
                for (int e = 0; e < 16; ++e) sc[0][e] = sc[1][e] = 0.f;
#pragma unroll
                for (int kk = 0; kk < KK; ++kk)
#pragma unroll
                    for (int i = 0; i < 2; ++i) sc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qb[kk], kb[i][kk], sc[i], 0, 0, 0);
                const unsigned q_lo[2] = {(unsigned)q_min[0], (unsigned)q_min[1]};
                if (j0 + 64 < j_end) load_keys(j0 + 64);
#pragma unroll
                for (int i = 0; i < 2; ++i) {
                    if (j0 + 32 * i >= j_end) break;
                    float part = 0.f;
#pragma unroll
                    for (int jj = 0; jj < 4; ++jj)
#pragma unroll
                        for (int r = 0; r < 4; ++r) {
                            const unsigned qq = qq0 + 8 * jj + 4 * half + r;
                            const float x = fmaf(sc[i][4 * jj + r], a.scale_log2e, -l4[jj][r]);
                            part += __builtin_amdgcn_exp2f(qq - q_lo[i] < n_queries - q_lo[i] ? x : -INFINITY); // q_lo <= qq < n_queries
                        }
                    part = half_sum(part);
                    if (half == 0) s_col[wave][j0 + 32 * i + lq] = part;
                }
            }
            __syncthreads();
            float *dst = aux + (((int64_t)b * a.Hkv + g) * n_tiles + qt) * a.n_q;
            for (int j = tid; j < a.n_q; j += 256)
                dst[j] = j < j_end ? (s_col[0][j] + s_col[1][j]) + (s_col[2][j] + s_col[3][j]) : 0.f;
        }
    }
}

// ------------------------------------------------------------------------------------------
// Eq. 1 for the matrix-core prefill: softmax weights on the new tokens, from the final log-sum-exps, added over
// queries and heads.  One workgroup per (128 new tokens, KV head, question, share of the queries): a wave keeps
// the keys of 64 tokens as the B operand in registers (two waves share them, each with 32 of a step's 64 queries) and the
// queries stream past it through LDS, so that S = Q K^T leaves a lane two keys and 16 queries and the sum over the
// queries is a running sum per lane and key, written once at the end.  (The same sums inside the attention kernel, walked
// by query tile, need a reduction over the waves and a store per 64 keys: 2400 cycles a step against 1000.  Few tokens pay
// that and save the launch: see kFusedSums.)
// colpart [B][Hkv][n_qs][n_q], of which a key tile fills as many rows as it has shares; they are added in a fixed order by
// prefill_signal_kernel.
// ------------------------------------------------------------------------------------------
template <int D>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3))) void prefill_keysum_kernel(
    AttendArgs a, const float *__restrict__ lse, float *__restrict__ colpart, int n_units, int combos, int n_qs, int steps_per) {
    using T = uint16_t;
    constexpr int kRowB = D * 2, kPieces = kRowB / 16, kRowsPerLoad = 64 / kPieces, kLoads = kCQ / 4 / kRowsPerLoad, KK = D / 16;
    __shared__ __align__(1024) unsigned char s_q[2][kCQ * kRowB];
    __shared__ __align__(16) float s_lse[2][kCQ];
    __shared__ float s_sum[kCK];
    int unit, combo;
    if (!tile_of(blockIdx.x, n_units, combos, &unit, &combo)) return;
    // the unit's key tile and its share of that tile's queries; here the first tiles are the heavy ones, so they start
    // first (8 questions of 1568 tokens, 64 heads, a whole tile a workgroup: 643 us a call, 625 this way round)
    int kt = 0, qs = n_units - 1 - unit;
    for (int n; qs >= (n = keysum_shares(kt, a.n_q * a.G, a.G, a.causal, steps_per)); ++kt) qs -= n;
    const int g = combo % a.Hkv, b = combo / a.Hkv;
    const int tid = threadIdx.x, wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63, lq = lane & 31, half = lane >> 5;
    const int n_queries = a.n_q * a.G;
    const int l0 = __builtin_amdgcn_readfirstlane(a.local_offsets[b]);
    int n_loc = __builtin_amdgcn_readfirstlane(a.local_offsets[b + 1]) - l0;
    if (n_loc < 0) n_loc = 0;
    const int kw = wave & 1, qpart = wave >> 1; // the wave's 64 keys, its 32 queries of every step
    // new token j is local row n_loc - n_q + j; it may not exist.  Query qq sees it iff qq >= q_min.
    int q_min[2];
    int64_t krow[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int j = kt * kCK + 64 * kw + 32 * i + lq, lrow = n_loc - a.n_q + j;
        const bool ok = j < a.n_q && lrow >= 0;
        q_min[i] = !ok ? INT_MAX : (a.causal ? j * a.G : 0);
        krow[i] = (int64_t)(l0 + (ok ? lrow : 0)) * a.Hkv + g;
    }
    // the steps of this key tile start at its first token's queries; this workgroup takes steps_per of them
    const int q0 = (a.causal ? kt * kCK * a.G : 0) + qs * steps_per * kCQ;
    int n_steps = q0 < n_queries ? (n_queries - q0 + kCQ - 1) / kCQ : 0;
    if (n_steps > steps_per) n_steps = steps_per;
    float sum[2] = {0.f, 0.f};
    if (n_steps > 0) {
        bf16x8 kb[2][KK];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const T *kp = static_cast<const T *>(a.k_local) + krow[i] * D + 8 * half;
            if (n_loc == 0) kp = static_cast<const T *>(a.q) + 8 * half; // memory that exists; the weights are masked
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) kb[i][kk] = __builtin_bit_cast(bf16x8, load16(kp + 16 * kk));
        }
        // query qq = (token qq / G, head qq % G of the group) is row (b n_q + token) Hq + g G + head of q and lse;
        // a lane walks its rows 64 queries at a time (past the last query: the last row, masked)
        const int row_last = (a.n_q - 1) * a.Hq + a.G - 1;
        const int dt = kCQ / a.G, dh = kCQ - dt * a.G;
        auto row_of = [&](int qq, int *h) {
            const int t = qq / a.G;
            *h = qq - t * a.G;
            return t * a.Hq + *h;
        };
        auto advance = [&](int &row, int &h) {
            row += dt * a.Hq + dh;
            h += dh;
            if (h >= a.G) {
                h -= a.G;
                row += a.Hq - a.G;
            }
        };
        const int64_t base = (int64_t)b * a.n_q * a.Hq + g * a.G;
        const unsigned char *qbase = static_cast<const unsigned char *>(a.q) + base * kRowB;
        const float *lbase = lse + base;
        const int ld_row = 16 * wave + lane / kPieces, ld_piece = lane % kPieces;
        int row[kLoads], hd[kLoads], lrow_q, lhd;
#pragma unroll
        for (int u = 0; u < kLoads; ++u) row[u] = row_of(q0 + ld_row + u * kRowsPerLoad, &hd[u]);
        lrow_q = row_of(q0 + lane, &lhd);
        auto request = [&](unsigned char *dq, float *dl) __attribute__((always_inline)) {
#pragma unroll
            for (int u = 0; u < kLoads; ++u) {
                const int r = row[u] < row_last ? row[u] : row_last;
                load_to_lds(qbase + (int64_t)r * kRowB + 16 * key_slot<D>(ld_piece, ld_row + u * kRowsPerLoad),
                            dq + (16 * wave + u * kRowsPerLoad) * kRowB);
                advance(row[u], hd[u]);
            }
            if (wave == 0) {
                load4_to_lds(lbase + (lrow_q < row_last ? lrow_q : row_last), dl);
                advance(lrow_q, lhd);
            }
        };
        int qoff[KK];
#pragma unroll
        for (int kk = 0; kk < KK; ++kk) qoff[kk] = (32 * qpart + lq) * kRowB + 16 * key_slot<D>(2 * kk + half, lq);
        float part[2][2] = {{0.f, 0.f}, {0.f, 0.f}};
        auto step = [&](int t, const unsigned char *cq, const float *cl, unsigned char *nq, float *nl) __attribute__((always_inline)) {
            rows_landed();
            __syncthreads();
            if (t + 1 < n_steps) request(nq, nl);
            f32x16 sc[2];
#pragma unroll
            for (int e = 0; e < 16; ++e) sc[0][e] = sc[1][e] = 0.f;
            bf16x8 aq[KK];
#pragma unroll
            for (int kk = 0; kk < KK; ++kk) aq[kk] = *reinterpret_cast<const bf16x8 *>(cq + qoff[kk]);
#pragma unroll
            for (int kk = 0; kk < KK; ++kk)
#pragma unroll
                for (int i = 0; i < 2; ++i) sc[i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(aq[kk], kb[i][kk], sc[i], 0, 0, 0);
            const int qq0 = q0 + t * kCQ + 32 * qpart;
            const bool masked = __builtin_amdgcn_ballot_w64(q_min[0] > qq0 || q_min[1] > qq0) != 0 || qq0 + 32 > n_queries;
            auto add = [&](auto with_mask) __attribute__((always_inline)) {
#pragma unroll
                for (int jj = 0; jj < 4; ++jj) {
                    const f32x4 l4 = *reinterpret_cast<const f32x4 *>(cl + 32 * qpart + 8 * jj + 4 * half);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const int qq = qq0 + 8 * jj + 4 * half + r;
#pragma unroll
                        for (int i = 0; i < 2; ++i) {
                            float x = fmaf(sc[i][4 * jj + r], a.scale_log2e, -l4[r]);
                            if constexpr (with_mask.value) x = qq >= q_min[i] && qq < n_queries ? x : -INFINITY;
                            part[i][r & 1] += __builtin_amdgcn_exp2f(x);
                        }
                    }
                }
            };
            if (masked)
                add(std::true_type{});
            else
                add(std::false_type{});
        };
        request(s_q[0], s_lse[0]);
        for (int t = 0; t < n_steps; t += 2) {
            step(t, s_q[0], s_lse[0], s_q[1], s_lse[1]);
            if (t + 1 < n_steps) step(t + 1, s_q[1], s_lse[1], s_q[0], s_lse[0]);
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) sum[i] = half_sum(part[i][0] + part[i][1]);
    }
    // the two waves that share the keys
    if (qpart == 1 && half == 0) {
        s_sum[64 * kw + lq] = sum[0];
        s_sum[64 * kw + 32 + lq] = sum[1];
    }
    __syncthreads();
    if (qpart == 0 && half == 0) {
        float *dst = colpart + (((int64_t)b * a.Hkv + g) * n_qs + qs) * a.n_q;
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int jl = 64 * kw + 32 * i + lq, j = kt * kCK + jl;
            if (j < a.n_q) dst[j] = sum[i] + s_sum[jl];
        }
    }
}

struct PrefillOut { // all null for the plain attention call
    float *lse, *colpart, *signal; // (lse: matrix-core prefill)
};

template <typename T, int D>
hipError_t launch_typed(const AttendArgs &a, int B, void *out, const PrefillOut &po, hipStream_t st) {
    const dim3 grid(a.n_split, a.Hkv * ((a.n_q * a.G + kAttQ - 1) / kAttQ), B);
    const bool merge = a.n_split > 1 && !po.signal; // a prefill's records are in the caller's workspace, which has no counts
    if (merge)
        hipLaunchKernelGGL((attend_kernel<T, D, true>), grid, dim3(64 * kAttWaves), 0, st, a, static_cast<T *>(out));
    else
        hipLaunchKernelGGL((attend_kernel<T, D, false>), grid, dim3(64 * kAttWaves), 0, st, a, static_cast<T *>(out));
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    if constexpr (column_sums<T, D>())
        if (a.n_split > 1 && !merge) {
            float *const no_lse = nullptr;
            hipLaunchKernelGGL((attend_combine_kernel<T, D, float *>), dim3((unsigned)(B * a.n_q * a.Hq)), dim3(D < 64 ? 64 : D), 0, st, a.part,
                               a.n_split, static_cast<T *>(out), no_lse);
        }
    if constexpr (!column_sums<T, D>()) return hipGetLastError(); // their prefill is the matrix-core one
    if ((e = hipGetLastError()) != hipSuccess || !po.signal) return e;
    // Shares of the queries, no more rows than the workspace has room for.  Under the causal mask the shares are uneven, so
    // where a tile is long work (fp32 rows of 64 features and more) there are up to 16 workgroups per compute unit, otherwise
    // four.  us a layer call with one / four / sixteen: fp32, 28 heads of 128, 196 tokens 42.5 / 41.8 / 41.2, 600 over 768 rows
    // 260 / 208 / 207, 32 heads of 64, 600 tokens 106 / 87 / 80; rows of 16, 300 tokens 17.3 / 16.0 / 16.9; bf16 rows of 32,
    // 400 tokens 25.4 / 20.1 / 20.6.
    constexpr int kWgs = sizeof(T) == 4 && D >= 64 ? 4096 : 1024;
    const int n_kt = (a.n_q + kColKeys - 1) / kColKeys, n_tiles = (a.n_q * a.G + 15) / 16;
    const int64_t wgs = (int64_t)n_kt * a.Hkv * B;
    int n_qs = wgs < kWgs ? (int)((kWgs + wgs - 1) / wgs) : 1;
    n_qs = n_qs < n_tiles ? n_qs : n_tiles;
    const int tiles_per = (n_tiles + n_qs - 1) / n_qs;
    n_qs = (n_tiles + tiles_per - 1) / tiles_per;
    if constexpr (column_sums<T, D>())
        hipLaunchKernelGGL((prefill_colsum_kernel<T, D>), dim3(n_kt * n_qs, a.Hkv, B), dim3(kThreads), 0, st, a, po.colpart, n_qs,
                           tiles_per);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(prefill_signal_kernel, dim3((a.n_q + kSigCols - 1) / kSigCols, B), dim3(kThreads), 0, st, po.colpart,
                       a.Hkv, n_qs, a.n_q, 1.0f / ((float)a.Hq * (float)a.n_q), po.signal, a.G, a.causal, 0);
    return hipGetLastError();
}

template <typename T>
hipError_t launch_by_dim(const AttendArgs &a, int D, int B, void *out, const PrefillOut &po, hipStream_t st) {
    switch (D) {
    case 16: return launch_typed<T, 16>(a, B, out, po, st);
    case 32: return launch_typed<T, 32>(a, B, out, po, st);
    case 64: return launch_typed<T, 64>(a, B, out, po, st);
    case 128: return launch_typed<T, 128>(a, B, out, po, st);
    default: return hipErrorInvalidValue;
    }
}

// Steps a workgroup of prefill_keysum_kernel takes: one, where that is at most a workgroup per compute unit (7B head
// layout, 128 tokens over 768 rows, 56 workgroups: 27.1 us a call against 28.0 with two steps; 600 tokens, 760
// workgroups: 49.3 against 47.5); otherwise as few as leave all workgroups resident at once (three per compute unit: one
// more round of them costs as much as the first), at least two.
int keysum_plan(int n_q, int G, int combos, int causal, int *n_units) {
    const int tiles = (n_q + kCK - 1) / kCK, all = (n_q * G + kCQ - 1) / kCQ;
    for (int per = 1;; per += (per + 15) / 16) {
        int n = 0;
        for (int kt = 0; kt < tiles; ++kt) n += keysum_shares(kt, n_q * G, G, causal, per);
        if ((int64_t)n * combos <= (per == 1 ? 256 : 3 * 256) || per >= all) {
            *n_units = n;
            return per;
        }
    }
}

// Rows of colpart per KV head, whichever way the mask is set.
int keysum_rows(int n_q, int G, int combos) {
    int rows = 0;
    for (int causal = 0; causal < 2; ++causal) {
        int n_units;
        const int n = keysum_shares(0, n_q * G, G, causal, keysum_plan(n_q, G, combos, causal, &n_units));
        if (n > rows) rows = n;
    }
    return rows;
}

template <int D>
hipError_t launch_flash(const AttendArgs &a, int n_fs, bool two_fours, int B, void *out, const PrefillOut &po, hipStream_t st) {
    const int n_tiles = (int)(((int64_t)a.n_q * a.G + kFQ - 1) / kFQ), combos = a.Hkv * B;
    uint16_t *o16 = static_cast<uint16_t *>(out);
    const unsigned grid = tile_grid(n_tiles * n_fs, combos);
    hipError_t e;
    const float inv = 1.0f / ((float)a.Hq * (float)a.n_q);
    const dim3 sig_grid((a.n_q + kSigCols - 1) / kSigCols, B);
    if (n_fs == 1 && !two_fours && a.n_q <= kFusedSums) { // two launches (see kFusedSums)
        hipLaunchKernelGGL((prefill_flash_kernel<D, 1, false, true>), dim3(grid), dim3(256), 0, st, a, o16, n_tiles, combos, po.colpart, 1);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL(prefill_signal_kernel, sig_grid, dim3(kThreads), 0, st, po.colpart, a.Hkv, n_tiles, a.n_q, inv, po.signal,
                           a.G, a.causal, 0);
        return hipGetLastError();
    }
    if (two_fours) {
        hipLaunchKernelGGL((prefill_flash_kernel<D, 2, false, false>), dim3(tile_grid(pairs_grid(n_tiles, combos), combos)), dim3(512), 0, st, a, o16, n_tiles, combos, po.lse, 1);
    } else if (n_fs == 1) {
        hipLaunchKernelGGL((prefill_flash_kernel<D, 1, false, false>), dim3(grid), dim3(256), 0, st, a, o16, n_tiles, combos, po.lse, 1);
    } else { // rows shared by n_fs workgroups per tile, merged
        hipLaunchKernelGGL((prefill_flash_kernel<D, 1, true, false>), dim3(grid), dim3(256), 0, st, a, o16, n_tiles, combos, a.part, n_fs);
        if ((e = hipGetLastError()) != hipSuccess) return e;
        hipLaunchKernelGGL((attend_combine_kernel<uint16_t, D, const float *__restrict__>), dim3((unsigned)(B * a.n_q * a.Hq)), dim3(D), 0, st, a.part,
                           n_fs, o16, po.lse);
    }
    if ((e = hipGetLastError()) != hipSuccess) return e;
    int n_units;
    const int steps_per = keysum_plan(a.n_q, a.G, combos, a.causal, &n_units);
    const int n_qs = keysum_shares(0, a.n_q * a.G, a.G, a.causal, steps_per);
    hipLaunchKernelGGL((prefill_keysum_kernel<D>), dim3(tile_grid(n_units, combos)), dim3(256), 0, st, a, po.lse, po.colpart,
                       n_units, combos, n_qs, steps_per);
    if ((e = hipGetLastError()) != hipSuccess) return e;
    hipLaunchKernelGGL(prefill_signal_kernel, sig_grid, dim3(kThreads), 0, st, po.colpart, a.Hkv, n_qs, a.n_q, inv, po.signal, a.G,
                       a.causal, steps_per);
    return hipGetLastError();
}

// Split records per query that the workspace of a prefill without the matrix-core kernels counts.
int record_splits(int B, int Hkv, int n_qtiles, int k_frame) {
    int64_t n_split = (3 * 256 + (int64_t)B * Hkv * n_qtiles - 1) / ((int64_t)B * Hkv * n_qtiles);
    if (n_split > kAttendMaxSplit) n_split = kAttendMaxSplit;
    if (n_split > k_frame) n_split = k_frame;
    if (n_split < 1) n_split = 1;
    const int per = k_frame > 0 ? (int)((k_frame + n_split - 1) / n_split) : 0;
    if (k_frame > 0) n_split = (k_frame + per - 1) / per;
    return (int)n_split;
}

// Workgroups that share the rows of one tile of attend_kernel, at most one per compute unit.
// A call whose last workgroup merges: as many as cost the least by what the parts were measured to take (us) -- a wave's block while
// the chip is nearly empty 0.7 to 1.6 by type and features, the merge 1.6 and 0.2 or 0.3 a share, and what the records of a full
// chip add, 0.7.  Over 6357 calls (bf16 and fp32, 16 to 128 features, six head layouts, 1 to 64 questions of 1 to 16 tokens, 80 to
// 3900 rows), each timed with every number of shares, the one taken is 0.4 % from the best in the mean; where it is more than 4 %
// (173 calls, nearly all fp32) the local rows, which are not known here, give some waves one block more.  us a call (graph replay), shares 1 / 2 /
// 4 / 8, the one taken with *: 7B head layout, one question over 416 rows 8.3 / 8.1 / 7.4* / 7.4, 800 rows 11.5 / 9.9 / 8.4 / 7.9 and
// in seven 7.8*; 4 questions over 800 rows 11.5 / 10.4 / 8.8 / 8.9, seven 8.8*; 32 questions of one KV head of 128 over 320 rows 8.0*
// / 9.6 / 9.4 / -; 8 KV heads of 32, 8 questions over 416 rows 6.1* / 7.0 / 6.9 / -; fp32, 7B head layout, one question over 224 rows
// 13.5 / 11.2 / 9.6* / 9.6, 416 rows 19.8 / 15.5 / 11.6 / 10.2, seven 10.0*.
// A prefill, whose records a launch of 3.5 us merges: where a wave has more than five blocks, into shares of six or more (800 rows
// with that launch, 1 / 2 / 4 / 8: 11.8 / 11.2 / 9.6 / 9.6).
// (The local rows are known on the device only; n_q of them at least are there or do not matter.)
int attend_split(const Ctx &c, int n_q, int B, int k_frame, bool prefill) {
    const int rows = c.esz == 2 ? 32 : 16, D = c.cfg.head_dim; // rows of a block
    const int64_t wgs = ((int64_t)n_q * c.group + kAttQ - 1) / kAttQ * c.cfg.n_kv_heads * B;
    const int64_t blocks = ((int64_t)k_frame * c.kappa + n_q + rows - 1) / rows;
    int64_t most = 256 / wgs;
    if (most > kAttendMaxSplit) most = kAttendMaxSplit;
    if (prefill) {
        if (blocks <= 5 * kAttWaves) return 1;
        if (most > blocks / 6) most = blocks / 6;
        return most < 1 ? 1 : (int)most;
    }
    const float block = c.esz == 2 ? (D > 64 ? 1.1f : D > 32 ? 1.0f : 0.7f) : (D > 64 ? 1.6f : D > 32 ? 1.4f : 0.9f);
    const float share = (D > 32 ? 0.3f : 0.2f) + 0.7f / 256.f * (float)wgs;
    int best = 1;
    float least = 0.f;
    for (int n = 1; n <= most; ++n) {
        const float cost = block * (float)((blocks + kAttWaves * n - 1) / (kAttWaves * n)) + (n > 1 ? 1.6f + share * (float)n : 0.f);
        if (n == 1 || cost < least) {
            best = n;
            least = cost;
        }
    }
    return best;
}

} // namespace

static bool flash_shape(const Ctx &c) { return c.cfg.dtype == MUKV_BF16 && (c.cfg.head_dim == 64 || c.cfg.head_dim == 128); }

// The workspace a caller provides, in bytes.  Part of the interface: callers keep buffers of this size, and
// mukv_prefill_attend_static takes the calls for which it fits.  Split records (at least one a query, whose start holds the
// query's pair for prefill_colsum_kernel), log-sum-exps (counted for every shape, written by the matrix-core prefill), and
// column sums per 64 queries (bf16 rows of 128 features) or 8 queries (all others); the matrix-core prefill stays within it.
int64_t prefill_workspace_bytes(const Ctx &c, int n_q, int B, int k_frame) {
    const int64_t n_queries = (int64_t)n_q * c.group, combos = (int64_t)c.cfg.n_kv_heads * B, rows = (int64_t)B * n_q * c.cfg.n_q_heads;
    const int k = k_frame > 0 ? k_frame : 0;
    int64_t n_split, tiles; // (as they were when the figure became part of the interface: more tiles than there are now)
    if (c.cfg.dtype == MUKV_BF16 && c.cfg.head_dim == 128) {
        tiles = (n_queries + 63) / 64;
        const int64_t steps = ((int64_t)k * c.kappa + n_q + 31) / 32;
        n_split = (768 + tiles * combos - 1) / (tiles * combos);
        if (n_split > kAttendMaxSplit) n_split = kAttendMaxSplit;
        if (n_split > steps / 4) n_split = steps / 4;
        if (tiles * combos >= 384 || n_split <= 1) n_split = 0; // one launch: no records
    } else {
        tiles = (n_queries + kTileQ - 1) / kTileQ;
        n_split = record_splits(B, c.cfg.n_kv_heads, (int)tiles, k);
    }
    return (rows * n_split * (c.cfg.head_dim + 2) + rows + combos * tiles * n_q) * (int64_t)sizeof(float);
}

// How the matrix-core prefill goes about its tiles, of three ways; returns the workgroups that share the rows of one (1: none do).
// Shares: where the tiles alone leave most of the chip idle; two workgroups per compute unit are wanted, at least two steps each, and
// no more than leave the records, log-sum-exps and column sums within the workspace.
// Two fours of waves that take a tile's steps in turn and join in LDS: no records, no merge, one workgroup per compute unit and half
// the chain.  One four a workgroup: what is left, and up to kFusedSums tokens the kernel that sums Eq. 1 itself.
// Shares or two fours, by what was measured (us): a pair of the two fours' steps 1.65 (rows of 64 features 1.35); a share's step
// 1.1 (0.85), the merge 1.6 and a record's number written and read again 2.8 ps (4.2).  Of 1562 calls that could go either way (1 to
// 1568 tokens, five head layouts, one and two questions, up to 1536 rows before them, with the mask and without) ten take a way more
// than 2 % slower than the other, 6 % at most.  us a call, 7B head layout over 768 rows, shares / two fours, the one taken with *:
// 1 token 18.1* / 23.7, 64 23.7* / 25.9, 128 28.2 / 26.9*, 196 35.2 / 29.3*, 600 48.4 / 39.4*; 1 token over 384 rows 16.6* / 18.3,
// 17 over 1536 22.8* / 36.3.
// Two fours or one, unshared, no more tiles than compute units: the join and the second four's tables cost what few steps give back
// (one four / two: 7B head layout, no past, 150 tokens, 3 steps, 16.5* / 18.2, 196, 4 steps, 17.6* / 18.3; 64 / 8 heads, 400, 7 steps,
// 26.2* / 26.8, 512, 8 steps, 30.0 / 29.7*; 28 / 4 heads of 64, two questions of 300, 5 steps, 17.6* / 18.0, one of 300 over 96 rows,
// 7 steps, 19.4 / 18.9*).
// More tiles than compute units, two fours with the smallest tiles in pairs: that evens out what the mask makes uneven, so only with
// it (1300 tokens over 768 rows, 7B head layout, without the mask 90.4* / 96.6), up to 7 / 4 tiles a unit.  With rows of 128 features
// two fours on a unit are slower at even tiles than two workgroups, so there the fewer tiles a unit, the more rows before the new
// ones are (28 / 4 heads, 1568 tokens over 768 rows, 1.34 tiles a unit, 79.7 / 72.5*; two questions of 1000, 1.72, without a past
// 50.2 / 48.6*, over 768 rows 70.7* / 71.8; 64 / 8 heads, 600 tokens, 1.19, over 768 rows 52.5 / 51.3*, over 1536 73.0* / 74.8; two
// questions of 300, 1.19, over 192 rows 31.0 / 30.1*, over 768 45.8* / 46.9; rows of 64 features, 64 / 8 heads, 600 tokens over 768
// rows 43.8 / 41.6*, over 1536 63.6 / 61.0*).
static int flash_split(const Ctx &c, int n_q, int B, int k_frame, bool causal, bool *two_fours) {
    const int64_t tiles = ((int64_t)n_q * c.group + kFQ - 1) / kFQ;
    const int combos = c.cfg.n_kv_heads * B, places = 256 / combos;
    const int64_t wgs = tiles * combos, past = (int64_t)(k_frame > 0 ? k_frame : 0) * c.kappa;
    const int64_t steps = (past + n_q + kFK - 1) / kFK;
    const bool wide = c.cfg.head_dim == 128;
    if (tiles <= places)
        *two_fours = n_q > kFusedSums && steps >= (wide ? 8 : 6);
    else
        *two_fours = n_q > kFusedSums && steps >= 6 && causal && 4 * tiles <= 7 * places &&
                     (!wide || 5 * past * places <= (15 * places - 7 * tiles) * n_q);
    if (wgs >= 192) return 1;
    int64_t n = (512 + wgs - 1) / wgs;
    if (n > kAttendMaxSplit) n = kAttendMaxSplit;
    if (n > steps / 2) n = steps / 2;
    const int64_t rows = (int64_t)B * n_q * c.cfg.n_q_heads;
    const int64_t rest = rows + (int64_t)combos * n_q * keysum_rows(n_q, c.group, combos);
    while (n > 1 && (rows * n * (c.cfg.head_dim + 2) + rest) * (int64_t)sizeof(float) > prefill_workspace_bytes(c, n_q, B, k_frame)) --n;
    if (n <= 1) return 1;
    const float share = (float)((steps + n - 1) / n), pairs = (float)((steps + 1) / 2), numbers = 1e-6f * (float)(rows * n * (c.cfg.head_dim + 2));
    *two_fours = wide ? 1.65f * pairs <= 1.6f + 1.1f * share + 2.8f * numbers : 1.35f * pairs <= 1.6f + 0.85f * share + 4.2f * numbers;
    return *two_fours ? 1 : (int)n;
}

// workspace == null: the plain attention call, records in the context's scratch, no signal.
hipError_t launch_attend(Ctx &c, int layer, const void *q, int n_q, const int32_t *frame_idx, int k_frame,
                         const void *k_local, const void *v_local, const int32_t *local_offsets, int B, int causal,
                         void *out, float *signal, float *workspace, hipStream_t st) {
    AttendArgs a;
    a.q = q;
    a.frame_idx = k_frame > 0 ? frame_idx : nullptr;
    a.k_local = k_local;
    a.v_local = v_local;
    a.local_offsets = local_offsets;
    const int64_t slab = (int64_t)c.store_cap * c.cfg.head_dim * c.esz; // bytes of one (layer, head) slab
    a.store_k = static_cast<const unsigned char *>(c.store_k) + (int64_t)layer * c.cfg.n_kv_heads * slab;
    a.store_v = static_cast<const unsigned char *>(c.store_v) + (int64_t)layer * c.cfg.n_kv_heads * slab;
    a.part = c.attend_part + kAttendMaxTiles;
    a.store_cap = c.store_cap;
    a.n_q = n_q;
    a.Hq = c.cfg.n_q_heads;
    a.Hkv = c.cfg.n_kv_heads;
    a.G = c.group;
    a.k_frame = k_frame > 0 ? k_frame : 0;
    a.kappa = c.kappa;
    a.n_frames = (int)c.n_frames;
    a.n_qtiles = (n_q * c.group + kTileQ - 1) / kTileQ;
    a.causal = causal;
    a.scale_log2e = 1.4426950408889634f / sqrtf((float)c.cfg.head_dim);
    a.n_split = attend_split(c, n_q, B, a.k_frame, workspace != nullptr);
    if (workspace) { // (its records are counted by the formula above)
        const int most = record_splits(B, a.Hkv, a.n_qtiles, a.k_frame);
        if (a.n_split > most) a.n_split = most;
    }
    a.pair_stride = 0;
    PrefillOut po{nullptr, nullptr, nullptr};
    bool two_fours = false;
    const int n_fs = workspace && flash_shape(c) ? flash_split(c, n_q, B, k_frame, causal != 0, &two_fours) : 0;
    if (workspace) {
        const int64_t rows = (int64_t)B * n_q * a.Hq;
        a.part = workspace;
        if (n_fs == 0) a.pair_stride = a.n_split > 1 ? a.n_split * (c.cfg.head_dim + 2) : 2; // (one record a query is counted, not written)
        po.lse = workspace + rows * (n_fs == 0 ? a.n_split : n_fs == 1 ? 0 : n_fs) * (c.cfg.head_dim + 2);
        po.colpart = po.lse + rows;
        po.signal = signal;
    }
    if (!workspace && a.n_split > 1 && c.arrivals_unsure) { // the first call that counts since the cache was emptied or replaced
        hipLaunchKernelGGL(clear_arrivals_kernel, dim3(1), dim3(kAttendMaxTiles), 0, st, a.part);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        c.arrivals_unsure = false;
    }
    if (n_fs) // the prefill on the matrix cores
        return c.cfg.head_dim == 64 ? launch_flash<64>(a, n_fs, two_fours, B, out, po, st) : launch_flash<128>(a, n_fs, two_fours, B, out, po, st);
    return c.cfg.dtype == MUKV_BF16 ? launch_by_dim<uint16_t>(a, c.cfg.head_dim, B, out, po, st)
                                    : launch_by_dim<float>(a, c.cfg.head_dim, B, out, po, st);
}

} // namespace mukv
