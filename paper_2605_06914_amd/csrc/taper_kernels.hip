// gfx950 kernels for decode-step attention over a paged KV cache with shared
// prefixes (paper §3.1: a branch attends to shared prefix ++ own tokens; all
// branches of a request are served from one set of prefix pages).
//
// Everything is computed in "transposed" form so that no operand ever has to be
// shuffled between lanes.  With 16x16x32 bf16 MFMA (A: 16 x 32, B: 32 x 16,
// C: 16 x 16; lane l supplies A[l%16][8*(l/16)..+7], B[8*(l/16)..+7][l%16] and
// receives C[4*(l/16)..+3][l%16]):
//   S^T (tokens x rows) = K (tokens x d) * Q^T (d x rows)      A = K tile, B = Q^T
//   O^T (d x rows)      = V^T (d x tokens) * P^T (tokens x rows) A = V^T,   B = P^T
// The C fragment of S^T (lane: query row l%16, tokens 4*(l/16)..+3) is, after
// exp and rounding, already the B fragment of P^T: the 32 tokens of an MFMA
// k-step are two pages, lane group l/16 holding tokens 4*(l/16)..+3 of each.  The
// pool layout (K in groups of 8 dims, V^T in groups of 4 tokens) makes the A
// fragments contiguous 16-byte / 8-byte pieces with unit stride across lanes.
//
// Softmax state per query row (one lane column): running max m in log2 units
// (scale*log2(e) folded in), running sum l, unnormalised O.  Partials of the KV
// chunks of a sequence (m, l in fp32; O / l in fp32 or, by default, in half precision with a
// per-row power-of-two scale) are combined through their (m, l) by the workgroup that delivers
// the sequence's last partial (merge_rows) or, in steps of many partials, by a launch of their own
// behind the attention launch (merge_kernel).
#include <climits>
#include <cstddef>
#include <type_traits>

#include "taper_internal.h"

namespace taper {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));

#define DEV __device__ __forceinline__

DEV f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) { return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0); }
DEV float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
DEV bf16x8 cat(bf16x4 a, bf16x4 b) { return __builtin_shufflevector(a, b, 0, 1, 2, 3, 4, 5, 6, 7); }
// KV is read exactly once per launch: stream it past the caches (measurably faster than cached loads)
template <typename T>
DEV T stream_load(const T* p) { return __builtin_nontemporal_load(p); }
// (maximum, not maxnum: v_maximum3 takes three values as they are, where maxnum first quiets each of them.  A NaN makes its row NaN either way.)
DEV float max3(float a, float b, float c) { return __builtin_elementwise_maximum(__builtin_elementwise_maximum(a, b), c); }
DEV float max8(f32x4 v, f32x4 w) {
    return max3(max3(v[0], v[1], v[2]), max3(v[3], w[0], w[1]), __builtin_elementwise_maximum(w[2], w[3]));
}

// Scores of invalid tokens of a chunk's last 32-token block -> -inf.
// sx: tokens 4*qd+i of the block's first page, sy: of its second page.
DEV void mask_tail(f32x4& sx, f32x4& sy, int qd, int n_valid) {
    const int t = n_valid - 4 * qd;  // this lane's tokens i (first page) and 16 + i (second page) are valid below t
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        if (i >= t) sx[i] = -INFINITY;
        if (16 + i >= t) sy[i] = -INFINITY;
    }
}

// A row lives in lanes n, n + 16, n + 32, n + 48.  The swap instructions exchange 32- or 16-lane halves of two
// registers without a trip through LDS (a ds_bpermute costs some 100 cycles, and each block has a chain of them).
DEV float max_lane_groups(float v) {
    unsigned u = __float_as_uint(v);
    auto p = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    u = __float_as_uint(fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1])));
    p = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return fmaxf(__uint_as_float(p[0]), __uint_as_float(p[1]));
}
DEV float sum_lane_groups(float v) {
    unsigned u = __float_as_uint(v);
    auto p = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    u = __float_as_uint(__uint_as_float(p[0]) + __uint_as_float(p[1]));
    p = __builtin_amdgcn_permlane16_swap(u, u, false, false);
    return __uint_as_float(p[0]) + __uint_as_float(p[1]);
}

// Online softmax over one 32-token block for one 16-row tile.  Every block passed
// in holds at least one valid token, so the new max is finite.  m is the row's exact running maximum: its largest
// weight is 1, which bf16 holds exactly (with a reference up to 2^8 lower, for fewer rescales, the error against 64 bits
// was 4 to 10 % larger on N(0,1) inputs and up to 20 % on wider scores, and accumulators overflowed 2^8 earlier).
// The lane groups' maxima are brought together, and the accumulators rescaled, only when some lane's is above m.
// NA tiles at a time: one branch for all of them, so that the instructions of one can fill the waits of another.
template <int DT, int NA>
DEV void softmax_block(const f32x4 (&sx)[NA], const f32x4 (&sy)[NA], float c, float (&m)[NA], float (&l)[NA], f32x4 (&O)[NA][DT], bf16x8 (&pf)[NA]) {
    float mx[NA];
    bool higher = false;
#pragma unroll
    for (int k = 0; k < NA; ++k) {
        mx[k] = max8(sx[k], sy[k]);
        higher |= mx[k] * c > m[k];
    }
    if (__any(higher)) {  // wave-uniform
#pragma unroll
        for (int k = 0; k < NA; ++k) {
            if (NA > 1 && !__any(mx[k] * c > m[k])) continue;
            const float mn = fmaxf(m[k], max_lane_groups(mx[k]) * c);
            const float alpha = fast_exp2(m[k] - mn);
            l[k] *= alpha;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) O[k][dt] *= alpha;
            m[k] = mn;
        }
    }
#pragma unroll
    for (int k = 0; k < NA; ++k) {
        f32x8 p;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            p[i] = fast_exp2(fmaf(sx[k][i], c, -m[k]));
            p[4 + i] = fast_exp2(fmaf(sy[k][i], c, -m[k]));
        }
        l[k] += ((p[0] + p[1]) + (p[2] + p[3])) + ((p[4] + p[5]) + (p[6] + p[7]));
        pf[k] = __builtin_convertvector(p, bf16x8);
    }
}

// The accumulator a block's last matrix instruction wrote must not be read by a vector instruction
// before the matrix pipeline has delivered it (four passes, 8 wait states; the hardware does not interlock, the
// compiler inserts them).  On a path that leaves the block's code through two branches
// and starts with register copies of the accumulators, the compiler was seen to leave too few: the
// last 16 dims of long private items came out wrong, in one build and not in another.  So a block
// ends with the wait states written out, fenced so that the scheduler leaves them where they are.
DEV void settle() {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_nop 11");
    __builtin_amdgcn_sched_barrier(0);
}

// Partials travel between workgroups inside one launch (to the merge launch, where a step has one, in the same way).  Workgroups may sit on
// different XCDs, whose L2s are not kept coherent for ordinary cached accesses,
// and a device-scope fence per workgroup (L2 write-back + invalidate) is far too
// slow.  So every partial word is written and read with device-scope atomic
// accesses (write-through stores, cache-bypassing loads, 8 bytes each), and the
// only ordering needed is "my stores have completed before I count myself in".
DEV void coherent_store2(float* p, float x, float y) {
    unsigned long long v = ((unsigned long long)__float_as_uint(y) << 32) | __float_as_uint(x);
    __hip_atomic_store((unsigned long long*)p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// The reader's side: 16 bytes past the caches (the sc1 bit, what a device-scope atomic load carries too),
// through a buffer descriptor with a 32-bit byte offset.  An offset at or above the descriptor's 2^31 - 1
// bytes makes the hardware return zeros without a memory access, which is how a round of merge loads
// leaves out what does not exist without a branch (the plan keeps a step's partial rows below 2^31 bytes).
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
constexpr unsigned kNoLoad = 0x80000000u;
DEV __amdgpu_buffer_rsrc_t partial_buffer(const void* base) {
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, 0x7fffffff, 0x00027000);
}
DEV u32x4 coherent_load16(__amdgpu_buffer_rsrc_t buf, unsigned byte_off) {
    return __builtin_amdgcn_raw_buffer_load_b128(buf, byte_off, 0, 16 /* sc1 */);
}
// The accumulator part of a partial row travels normalised (divided by the row's own sum, so that
// it is a weighted mean of V rows), in one of two formats (taper_partial_format):
//   PF_F32   fp32, two 8-byte accesses per four values;
//   PF_F16S  half precision after division by a power of two that brings the row's largest
//            magnitude into [0.5, 1): one 8-byte access per four values, 11 bits of mantissa
//            relative to the row's largest element beside the 8 the bf16 result keeps, and no
//            limit on the magnitude of V.  The power of two sits beside (m, l) in the row's
//            statistics record and is multiplied back in by the merge.
constexpr int PF_F16S = TAPER_PARTIAL_F16_SCALED, PF_F32 = TAPER_PARTIAL_F32;
typedef _Float16 f16x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
template <int PF>
DEV void partial_store4(void* rows, int64_t elem, f32x4 v) {
    if constexpr (PF == PF_F32) {
        float* p = (float*)rows + elem;
        coherent_store2(p, v[0], v[1]);
        coherent_store2(p + 2, v[2], v[3]);
    } else {
        const f16x4 h = __builtin_convertvector(v, f16x4);
        __hip_atomic_store((unsigned long long*)((uint16_t*)rows + elem), __builtin_bit_cast(unsigned long long, h),
                           __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}
// The elements of a partial row that one 16-byte load delivers.
template <int PF>
struct PartialVec {
    static constexpr int N = PF == PF_F32 ? 4 : 8;
    typedef float type __attribute__((ext_vector_type(N)));
    typedef __bf16 out_type __attribute__((ext_vector_type(N)));
    DEV static type unpack(u32x4 r) {
        if constexpr (PF == PF_F32) return __builtin_bit_cast(type, r);
        else return __builtin_convertvector(__builtin_bit_cast(f16x8, r), type);
    }
};
// The power of two 2^e that brings a row whose largest magnitude is `maxabs` into [0.5, 1), as
// (2^e, 2^-e); e is kept inside [-126, 126] so that both are normal numbers (an all-zero row, or one
// that holds Inf, is multiplied by some power of two all the same: it stays what it is).
DEV float2 row_scale(float maxabs) {
    int e = (int)((__float_as_uint(maxabs) >> 23) & 0xff) - 126;
    e = e < -126 ? -126 : (e > 126 ? 126 : e);
    return make_float2(__uint_as_float((unsigned)(127 + e) << 23), __uint_as_float((unsigned)(127 - e) << 23));
}
DEV float maxabs4(f32x4 v) { return fmaxf(fmaxf(fabsf(v[0]), fabsf(v[1])), fmaxf(fabsf(v[2]), fabsf(v[3]))); }
// Statistics record of a partial row: (running max in log2 units, sum) and, for PF_F16S, (row scale, unused).
template <int PF>
DEV void stats_store(float4* rec, float m, float l, float scale) {
    coherent_store2((float*)rec, m, l);
    if constexpr (PF == PF_F16S) coherent_store2((float*)rec + 2, scale, 0.f);
}
// Every earlier vector memory operation of this wave has completed, in particular its
// write-through stores of partial rows.  (A workgroup-scope release fence does not wait for
// global stores on this target, and nothing weaker than a full wait orders the stores
// before the arrival counter's increment for a reader on another compute unit.)
DEV void stores_done() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// What the end of an item needs from the plan, fetched when the item starts so that no
// dependent load is left for the end, where each one costs a loaded memory latency:
// merge_start[seq0 + b] for the item's sequences and the first kMetaWindow merge entries from
// merge_start[seq0] on (the sequences' entry lists are adjacent).
constexpr int kMetaWindow = 128;
struct MergeMeta {
    int ms[65];
    taper_merge_entry me[kMetaWindow];
};
struct MetaRegs {
    int ms;
    taper_merge_entry me;
};
// A per-lane value the compiler must not reason about: whatever is derived from it is
// computed where it is used instead of being hoisted out of the item loop, where it would
// sit in registers (or, worse, in scratch) for the whole kernel.
DEV int opaque(int v) {
    asm volatile("" : "+v"(v));
    return v;
}
// V of the invalid tokens of a chunk's last 32-token block -> 0, so that whatever bits an
// unwritten slot holds (NaN, Inf) meet their zero weight as 0 * 0.  A lane's values are tokens
// 4*qd+i of the first page (va) and of the second (vb), two per dword.  The comparisons are made
// again for every dword pair (from `opaque`) rather than kept: this runs once per chunk, in
// code that has no register to spare.
DEV unsigned keep_pair(unsigned w, int t) {  // both halves if t >= 2, the low one if t == 1, none below
    const unsigned lo = __builtin_amdgcn_ubfe(w, 0, 16);  // (no 32-bit literal: those get hoisted into registers)
    return t > 1 ? w : (t > 0 ? lo : 0u);
}
DEV bf16x4 keep_tail(bf16x4 v, int t) {  // tokens i < t of the four
    u32x2 w = __builtin_bit_cast(u32x2, v);
    w[0] = keep_pair(w[0], t);
    w[1] = keep_pair(w[1], t - 2);
    return __builtin_bit_cast(bf16x4, w);
}
template <int DT>
DEV void zero_tail(bf16x4 (&va)[DT], bf16x4 (&vb)[DT], int qd, int n_valid) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
        const int t = opaque(n_valid - 4 * qd);
        va[dt] = keep_tail(va[dt], t);
        vb[dt] = keep_tail(vb[dt], t - 16);
    }
}

// A work item by one scalar load (the compiler is not told that nothing here writes to the plan, and would use vector loads).
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(4))) int32_t* scalar_row;
DEV taper_work_item load_item(const DecodeArgs& a, const int it) {
    return __builtin_bit_cast(taper_work_item, ((const __attribute__((address_space(4))) i32x8*)a.items)[it]);
}
// What a launch's first loads need, beside a wave's start record.  It comes as two leading kernel arguments of four words, which arrive in
// registers.  (Each argument more is host time of every launch: with seven of them, calls that wait for the host took 5.4 us, with these 4.9 us.)
struct Inputs {
    const void *starts, *kv, *q;
    int n_kv_heads, n_q_heads, gqa, n_parts_shared;
    bool four_items;  // in each start record
};
static u32x4 pack_pointers(const StepArgs& a) {
    const uint64_t starts = (uint64_t)a.starts, kv = (uint64_t)a.kv;
    return {(unsigned)starts, (unsigned)(starts >> 32), (unsigned)kv, (unsigned)(kv >> 32)};
}
static u32x4 pack_queries(const StepArgs& a) {  // (gqa is at most 16: five bits, then one, then the number of shares)
    return {(unsigned)(uint64_t)a.q, (unsigned)((uint64_t)a.q >> 32), (unsigned)a.n_kv_heads, (unsigned)a.n_parts_shared << 6 | (a.start_bytes == kStartBytesFour ? 32u : 0u) | (unsigned)a.gqa};
}
DEV Inputs unpack_inputs(const u32x4 p, const u32x4 q) {
    typedef const __attribute__((address_space(1))) char* global_bytes;
    const auto pointer = [](unsigned lo, unsigned hi) { return (const void*)(global_bytes)((uint64_t)hi << 32 | lo); };
    const int gqa = q[3] & 31;
    return {pointer(p[0], p[1]), pointer(p[2], p[3]), pointer(q[0], q[1]), (int)q[2], (int)q[2] * gqa, gqa, (int)(q[3] >> 6), (q[3] & 32) != 0};
}
// A wave's start record, by scalar loads side by side.
struct Start {
    int first, end, turn, n_solo;
    taper_work_item item;
    i32x4 page, more;
};
#define CONSTANT const __attribute__((address_space(4)))
DEV Start load_start(const Inputs& in, const int part, const int wave) {
    const auto r = (CONSTANT char*)in.starts + (uint64_t)(unsigned)part * (unsigned)(in.four_items ? kStartBytesFour : kStartBytesOne);
    const i32x4 head = *(CONSTANT i32x4*)r;
    Start s;
    s.first = head[0];
    s.end = head[1];
    s.turn = head[2];
    s.n_solo = head[3];
    s.item = __builtin_bit_cast(taper_work_item, *(CONSTANT i32x8*)(r + offsetof(ShareStart, item) + (in.four_items ? wave : 0) * sizeof(taper_work_item)));
    s.page = *(CONSTANT i32x4*)(r + offsetof(ShareStart, page) + wave * sizeof(i32x4));
    s.more = *(CONSTANT i32x4*)(r + offsetof(ShareStart, more));
    // (all of it is asked for here, and the other arguments' cache lines with it, which later loads then find)
    const auto args = (CONSTANT int*)__builtin_amdgcn_kernarg_segment_ptr();
    const int line1 = args[16], line2 = args[32];
    asm volatile("" : "+s"(s.item.seq0), "+s"(s.page), "+s"(s.more) : "s"(line1), "s"(line2));
    return s;
}
// The other arguments, read from where they lie as they are needed.  (As a parameter that is used they are all loaded at the kernel's start,
// and waited for, 60 registers of them, before the start record is asked for.)
DEV const DecodeArgs& decode_args() { return *(const DecodeArgs*)((CONSTANT char*)__builtin_amdgcn_kernarg_segment_ptr() + 2 * sizeof(u32x4)); }
static_assert(alignof(DecodeArgs) <= sizeof(u32x4), "the arguments follow the leading two directly");
DEV scalar_row table_row(const DecodeArgs& a, const taper_work_item& item) {
    return (scalar_row)(a.bt + (int64_t)item.seq0 * a.bt_stride + item.page0);
}
// Pages of blocks b and b + step of a private item (past the last page: the last page).
DEV i32x4 private_pages(const DecodeArgs& a, const taper_work_item& item, const int b, const int step) {
    const scalar_row row = table_row(a, item);
    const int last = ((item.n_tokens + 15) >> 4) - 1;
    i32x4 p;
    p[0] = row[min(2 * b, last)];
    p[1] = row[min(2 * b + 1, last)];
    p[2] = row[min(2 * (b + step), last)];
    p[3] = row[min(2 * (b + step) + 1, last)];
    return p;
}

// (No branches: a lane without a value asks for one past the descriptor's end and gets zeros, so nothing is waited
// for before meta_store.)
DEV MetaRegs meta_load(const DecodeArgs& a, const taper_work_item& item, const int tid_) {
    const int tid = opaque(tid_);
    const auto starts = partial_buffer(a.merge_start), entries = partial_buffer(a.merge);
    MetaRegs r;
    r.ms = __builtin_amdgcn_raw_buffer_load_b32(starts, tid <= item.n_branch ? (item.seq0 + tid) * 4 : kNoLoad, 0, 0);
    r.me = __builtin_bit_cast(taper_merge_entry,
                              __builtin_amdgcn_raw_buffer_load_b64(
                                  entries, tid < kMetaWindow && item.merge0 + tid < a.n_merge ? (item.merge0 + tid) * 8 : kNoLoad, 0, 0));
    return r;
}
DEV void meta_store(MergeMeta& mm, const MetaRegs& r, const int n_branch, const int tid_) {
    const int tid = opaque(tid_);
    if (tid <= n_branch) mm.ms[tid] = r.ms;
    if (tid < kMetaWindow) mm.me[tid] = r.me;
}
// Log-sum-exp merge of all partials of (sequence s, kv head hk) -- its request's
// prefix chunks and its own private chunks, entries [e0, e1) of the merge map -- then
// normalisation and rounding to bf16.  Entries are taken in plan order, in rounds whose sizes follow from
// their number alone, whoever runs it, so the result does not depend on which workgroup that is.
//
// Bound by latency: the loads bypass the caches, and a trip takes 0.6 us on an idle machine and several
// times that on a saturated one.  So a round has no branch and nothing waits inside it: the entries come
// from the window in LDS, and the loads of all of them (statistics and row) are in flight together; past the
// sequence's last entry they are turned off by their offset.  (With a branch per entry the compiler waits
// for each entry's loads before it issues the next one's: 4.8 us for 8 entries on an idle machine, 2.0 this way.)
// Rounds of 8, the rest in one of 8, 4 or 2 (fp32 rows: 4 or 2): a load that is turned off still takes its turn in the
// compute unit's memory pipeline, and most sequences have two or three entries.
//
// A group of n_thr consecutive lanes (a workgroup, a wave or half a wave) merges one sequence;
// groups of one wave may work on different sequences side by side.  Lane idx of the group owns
// 16-byte columns c, c + LPR, ... (U of them) of one row; n_thr / LPR rows are merged per pass.
template <int D, int U, int PF>
DEV void merge_rows(const DecodeArgs& a, const MergeMeta& mm, const int s, const int hk, const int e0, const int e1,
                    const int idx_, const int n_thr) {
    typedef PartialVec<PF> Vec;
    typedef typename Vec::type vec;
    constexpr int LPR = D / Vec::N / U;
    constexpr int ROW_BYTES = D * 16 / Vec::N;
    const auto rows = partial_buffer(a.ws_o), stats = partial_buffer(a.ws_ml);
    const int g = a.gqa, w0 = mm.ms[0];
    const int idx = opaque(idx_);
    const int jr = idx / LPR, c0 = idx % LPR;
    for (int j0 = 0; j0 < g; j0 += n_thr / LPR) {
        const int j = j0 + jr;
        const bool okr = j < g;
        float M = -INFINITY, L = 0.f;
        vec acc[U];
#pragma unroll
        for (int u = 0; u < U; ++u) acc[u] = (vec)(0.f);
        auto round = [&](const int e, auto size) {
            constexpr int R = decltype(size)::value;
            taper_merge_entry me[R];
            if ((e + R < e1 ? e + R : e1) - w0 <= kMetaWindow) {
#pragma unroll
                for (int k = 0; k < R; ++k) me[k] = mm.me[(e + k < e1 ? e + k : e1 - 1) - w0];
            } else {
#pragma unroll
                for (int k = 0; k < R; ++k) me[k] = a.merge[e + k < e1 ? e + k : e1 - 1];
            }
            u32x4 st[R], o[R][U];
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const bool real = okr && e + k < e1;
                const unsigned row = me[k].first_row + hk * me[k].rows_per_head + j;
                st[k] = coherent_load16(stats, real ? row * 16 : kNoLoad);
#pragma unroll
                for (int u = 0; u < U; ++u) o[k][u] = coherent_load16(rows, real ? row * ROW_BYTES + 16 * (c0 + LPR * u) : kNoLoad);
            }
            float mk[R], mn = M;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                mk[k] = okr && e + k < e1 ? __uint_as_float(st[k][0]) : -INFINITY;
                mn = fmaxf(mn, mk[k]);
            }
            const float keep = fast_exp2(M - mn);  // first round: exp2(-inf) = 0
            L *= keep;
#pragma unroll
            for (int u = 0; u < U; ++u) acc[u] *= keep;
#pragma unroll
            for (int k = 0; k < R; ++k) {
                const float w = fast_exp2(mk[k] - mn) * __uint_as_float(st[k][1]);  // (the row was stored divided by its sum)
                L += w;
                const float ws = PF == PF_F16S ? w * __uint_as_float(st[k][2]) : w;
#pragma unroll
                for (int u = 0; u < U; ++u) acc[u] += ws * Vec::unpack(o[k][u]);
            }
            M = mn;
        };
        for (int e = e0; e < e1;) {
            if (PF == PF_F16S && e1 - e > 4) {
                round(e, std::integral_constant<int, PF == PF_F16S ? 8 : 2>{});
                e += 8;
            } else if (e1 - e > 2) {
                round(e, std::integral_constant<int, 4>{});
                e += 4;
            } else {
                round(e, std::integral_constant<int, 2>{});
                e += 2;
            }
        }
        if (okr) {
            const int h = hk * g + j;
            const float inv = 1.0f / L;
#pragma unroll
            for (int u = 0; u < U; ++u)
                *(typename Vec::out_type*)((__bf16*)a.out + ((int64_t)s * a.n_q_heads + h) * D + Vec::N * (c0 + LPR * u)) =
                    __builtin_convertvector(acc[u] * inv, typename Vec::out_type);
            if (a.lse && c0 == 0) a.lse[(int64_t)s * a.n_q_heads + h] = (M + __log2f(L)) * 0.6931471805599453f;
        }
    }
}

// A workgroup that has written a partial of (sequence s, kv head hk), one of n_entries,
// announces it.  Returns true to the one caller that arrives last: every other partial of
// that (s, hk) has then been written through (each writer waited for its stores before
// its increment) and the caller must merge.  The counter is left at zero for the next launch
// (by a device-scope store, like every other access to it).
DEV bool arrive_last(const DecodeArgs& a, const int s, const int hk, const int n_entries) {
    int* c = a.counters + (int64_t)s * a.n_kv_heads + hk;
    const bool last = atomicAdd(c, 1) == n_entries - 1;
    if (last) __hip_atomic_store(c, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return last;
}

// End of a shared-prefix item: every branch announces the item's partial; the branches whose set
// is now complete are merged side by side, a wave each for up to four of them, else half a wave.
// (One after the other they cost two to three memory round trips each, at the very end of a
// launch's longest workgroups.)  Called by all threads after the partial rows have been stored
// and waited for; `todo` and `n_todo` are workgroup-shared.
template <int D, int PF>
DEV void arrive_and_merge(const DecodeArgs& a, const MergeMeta& mm, int* todo, int* n_todo, const taper_work_item& item,
                          const int hk, const int tid) {
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if (wave == 0) {  // (an item has at most 64 branches)
        const bool mine = lane < item.n_branch && arrive_last(a, item.seq0 + lane, hk, mm.ms[lane + 1] - mm.ms[lane]);
        const unsigned long long mask = __ballot(mine);
        if (mine) todo[__popcll(mask & ((1ull << lane) - 1))] = lane;
        if (lane == 0) *n_todo = __popcll(mask);
    }
    __syncthreads();
    const int n = *n_todo;
    constexpr int N = PartialVec<PF>::N;
    if (n <= 4) {
        if (wave < n) {
            const int b = todo[wave];
            merge_rows<D, D / N / 8, PF>(a, mm, item.seq0 + b, hk, mm.ms[b], mm.ms[b + 1], lane, 64);
        }
    } else {
        for (int i = tid >> 5; i < n; i += 8) {
            const int b = todo[i];
            merge_rows<D, D / N / 4, PF>(a, mm, item.seq0 + b, hk, mm.ms[b], mm.ms[b + 1], tid & 31, 32);
        }
    }
}

// ---------------------------------------------------------------------------
// Private / serial kernel: one sequence's g query rows (one 16-row tile, rows
// >= g idle) against a chunk of that sequence's own pages.  No reuse across
// waves, so K/V go straight from HBM into MFMA operand registers; the four
// waves of a workgroup take alternate 32-token blocks and combine through LDS.
// ---------------------------------------------------------------------------
template <int D>
struct KVRegs {
    bf16x8 kx[D / 32], ky[D / 32];
    bf16x4 va[D / 16], vb[D / 16];
};

template <int D>
struct PrivateSmem {
    float o[4][16][D + 4];
    float2 ml[4][16];
    int last;
    int pick;      // pool item a workgroup has taken
    int todo[64];  // sequences whose last partial a run of solo items delivered
    int n_todo;
    int sink[4][64];  // see touch_block
    MergeMeta meta;
};

DEV unsigned lds_address(const void* p) { return (unsigned)(uintptr_t)(__attribute__((address_space(3))) const char*)p; }
// 64 lanes x 16 bytes: lane l's from base + off (per lane) to LDS address `lds` + 16 l; streamed past the caches.
// The compiler's hazard pass does not look inside: the statement itself keeps the one wait state from m0's write and the five that
// lie between a vector instruction's write of the base (a v_readlane of a spilled register) and the load that reads it.
// (That m0 is reserved is what the compiler would warn of at each use; nothing else in these kernels reads m0.)
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
DEV void load_to_lds(const char* base, unsigned off, unsigned lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 4\n\tglobal_load_lds_dwordx4 %0, %1 nt" ::"v"(off), "s"(base), "s"(lds) : "m0", "memory");
}
// 64 lanes x 4 bytes, to be found in the L2 later.
DEV void word_to_lds(const char* base, unsigned off, unsigned lds) {
    asm volatile("s_mov_b32 m0, %2\n\ts_nop 4\n\tglobal_load_lds_dword %0, %1" ::"v"(off), "s"(base), "s"(lds) : "m0", "memory");
}
#pragma clang diagnostic pop
// Brings a block's lines into the L2 for loads that follow when there are registers for them: a word of each 64 (32) bytes of its four tiles goes
// to a place in LDS that nobody reads.  (Loads into registers would have to be waited for, or be moved while in flight.)  The wave's later loads
// come in behind these, and it waits for some before it ends: a block is touched by the wave that goes on to compute it.
template <int D>
DEV void touch_block(const Inputs& in, const int hk, const int pid_a, const int pid_b, const void* sink) {
    constexpr int TILE_BYTES = 32 * D;
    const unsigned off = (opaque(threadIdx.x) & 63) * (TILE_BYTES / 64), lds = lds_address(sink);
    const unsigned page_bytes = in.n_kv_heads * TILE_BYTES * 2;
    // (words: a pool may start anywhere)
    const char* kvb = (const char*)((uintptr_t)in.kv & ~(uintptr_t)3) + (int64_t)hk * TILE_BYTES;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const char* k = kvb + (uint64_t)(unsigned)(i ? pid_b : pid_a) * page_bytes;
        word_to_lds(k, off, lds);
        word_to_lds(k + (int64_t)in.n_kv_heads * TILE_BYTES, off, lds);
    }
}
// What a wave has asked for of the item it does next: its queries and its first block.
template <int D>
struct Ahead {
    bf16x8 qf[D / 32];
    KVRegs<D> kv;
};
template <int D>
DEV void load_block(const Inputs& in, const int hk, const int lane, const int pid_a, const int pid_b, KVRegs<D>& r) {
    constexpr int KS = D / 32, DT = D / 16, TILE = 16 * D;
    const int n = lane & 15, qd = lane >> 4;
    const unsigned page_bytes = in.n_kv_heads * TILE * 4;
    const char* kvb = (const char*)in.kv + (int64_t)hk * TILE * 2;
    const unsigned koff = lane * 16, voff = (qd * (4 * D) + n * 4) * 2;
    const char* ka = kvb + (uint64_t)(unsigned)pid_a * page_bytes;  // (32 x 32 bits)
    const char* kb = kvb + (uint64_t)(unsigned)pid_b * page_bytes;
    const char* va = ka + (int64_t)in.n_kv_heads * TILE * 2;
    const char* vb = kb + (int64_t)in.n_kv_heads * TILE * 2;
#pragma unroll
    for (int j = 0; j < KS; ++j) {
        r.kx[j] = stream_load((const bf16x8*)(ka + koff + j * 1024));
        r.ky[j] = stream_load((const bf16x8*)(kb + koff + j * 1024));
    }
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
        r.va[dt] = stream_load((const bf16x4*)(va + voff + dt * 128));
        r.vb[dt] = stream_load((const bf16x4*)(vb + voff + dt * 128));
    }
}
// Asks for the queries and the first block (if it has one, of pages page[0] and page[1]) of an item of which the wave takes block b first.
template <int D>
DEV void begin_item(const Inputs& in, const taper_work_item& item, const i32x4 page, const int hk, const int lane, const int b, Ahead<D>& w) {
    const int n = lane & 15, qd = lane >> 4, g = in.gqa;
    // (lane columns past the last query head repeat the first; not stored)
    const __bf16* qrow = (const __bf16*)in.q + ((int64_t)item.seq0 * in.n_q_heads + hk * g + (n < g ? n : 0)) * D;
#pragma unroll
    for (int j = 0; j < D / 32; ++j) w.qf[j] = *(const bf16x8*)(qrow + 8 * (4 * j + qd));
    if (b < (item.n_tokens + 31) >> 5) load_block<D>(in, hk, lane, page[0], page[1], w.kv);
}

// One private item: a chunk of one sequence's own tokens, for kv head hk.
// SOLO: the item is run by the calling wave alone (short items: four of them proceed side by side in a workgroup, with no
// barrier and no LDS), which stores its result or its partial rows; otherwise the four waves of the workgroup share the item's
// blocks.
// Bound by HBM: 128 requests of 4096 tokens take 321 us, a bare read of the same pages 310.  The depth of the pipeline is
// not what matters then (one set of registers refilled as it is used up, two, and two with the block after next
// already asked for all measure within 0.5 %); two sets win where a wave has two blocks and the machine is idle
// (mixed batch on one kv head: 9 % slower with one set).
// The block-table row is read by scalar loads (constant address space, wave-uniform pointer), which do not wait for
// the KV loads in flight; a vector load of a page id completes in order, behind everything issued before it.
// HOLD: beside shared-prefix work (head_dim 128) a wave asks for its next block only when the one before has landed, if the
// step's shares are long (2000 tokens and more): what it asks for earlier it only waits for longer, and the shared workgroups with
// it.  Held back / not, us: 128 requests of 3 branches 471 / 474, of 17 branches 798 / 804; 16 branches of 32768 tokens 353.1 / 354.4; 8
// requests of 12 branches, 2231 tokens per share, 104 / 108; no more than 0.6 % is lost anywhere above.  In shorter shares the wait
// counts: 155 tokens per share 18.5 / 17.2, 577 31.5 / 30.4, 57 12.7 / 12.1, with 2 to 3 % the other way at others.  At
// head_dim 64 a block holds half the bytes and the wait weighs more (mixed batch 46.3 / 45.4).
// `page`: the pages of the wave's first two blocks.  `tail` is called by every wave before its last block (or where that would be).  SOLO: the item's
// queries and first block have been asked for (`w`), and `next`, called once its blocks are done with, may ask for the next item's.
// (For items of the whole workgroup that gains nothing: 512 of 600 tokens 205.9 us with it and 206.9 without.)
template <int D, bool SOLO, int PF, bool HOLD, typename Tail, typename Next>
DEV void private_item(const DecodeArgs& a, const Inputs& in, const taper_work_item item, const i32x4 page, const int hk, const int after, PrivateSmem<D>& sm,
                      Ahead<D>& w, Tail&& tail, Next&& next) {
    constexpr int KS = D / 32, DT = D / 16;
    auto& sm_o = sm.o;
    auto& sm_ml = sm.ml;
    const int lane = opaque(threadIdx.x) & 63;  // (opaque: per-lane constants are recomputed per item, not kept for the whole kernel)
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int n = lane & 15, qd = lane >> 4;
    const int g = in.gqa;
    const float c = a.scale_log2e;
    {
        const scalar_row row = table_row(a, item);
        const int n_tok = item.n_tokens;
        const int n_pages = (n_tok + 15) >> 4;
        const int n_blocks = (n_tok + 31) >> 5;
        const bool sole = item.kind >= 2;  // the sequence's whole context: no partial, no arrival, no merge
        MetaRegs mr = {};
        if (!SOLO && !sole) mr = meta_load(a, item, threadIdx.x);
        if (!SOLO) begin_item<D>(in, item, page, hk, lane, wave, w);

        bf16x8(&qf)[KS] = w.qf;
        float m1[1] = {-INFINITY}, l1[1] = {0.f};
        f32x4 O1[1][DT];
        float &m = m1[0], &l = l1[0];
        f32x4(&O)[DT] = O1[0];
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) O[dt] = (f32x4)(0.f);

        int pid_a = page[2], pid_b = page[3];  // the pages of the block loaded next
        auto fetch_ids = [&](int b) {
            const int ia = 2 * b < n_pages ? 2 * b : n_pages - 1, ib = 2 * b + 1 < n_pages ? 2 * b + 1 : n_pages - 1;
            pid_a = row[ia];
            pid_b = row[ib];
        };
        auto hold = [&] { if (HOLD && a.long_shares) asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); };
        auto compute_block = [&](int b, KVRegs<D>& r, auto last) {
            f32x4 sx[1] = {(f32x4)(0.f)}, sy[1] = {(f32x4)(0.f)};
#pragma unroll
            for (int j = 0; j < KS; ++j) {
                sx[0] = mfma16(r.kx[j], qf[j], sx[0]);
                sy[0] = mfma16(r.ky[j], qf[j], sy[0]);
            }
            const int nv = n_tok - 32 * b;
            if (last && nv < 32) mask_tail(sx[0], sy[0], qd, nv);
            bf16x8 pf[1];
            softmax_block<DT, 1>(sx, sy, c, m1, l1, O1, pf);
            if (last && nv < 32) zero_tail(r.va, r.vb, qd, nv);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) O[dt] = mfma16(cat(r.va[dt], r.vb[dt]), pf[0], O[dt]);
            settle();
        };

        // Blocks wave, wave + 4, ... of a shared item; all blocks of a solo one.  Two register sets: inside the loop the
        // next block's loads are issued unconditionally before the current block is computed, so that the waits the
        // compiler makes leave exactly those in flight (a load behind a branch would have to be waited for with the rest).
        constexpr int STEP = SOLO ? 1 : 4;
        int b = SOLO ? 0 : wave;
        if (b < n_blocks) {
            KVRegs<D>& r0 = w.kv;
            while (b + 2 * STEP < n_blocks) {
                KVRegs<D> r1;
                hold();
                load_block<D>(in, hk, lane, pid_a, pid_b, r1);
                fetch_ids(b + 2 * STEP);
                compute_block(b, r0, std::false_type{});
                hold();
                load_block<D>(in, hk, lane, pid_a, pid_b, r0);
                fetch_ids(b + 3 * STEP);
                compute_block(b + STEP, r1, std::false_type{});
                b += 2 * STEP;
            }
            // (the last block is computed from where it lies: moved to r0 it would have to be there as a whole first)
            if (b + STEP < n_blocks) {
                KVRegs<D> r1;
                hold();
                load_block<D>(in, hk, lane, pid_a, pid_b, r1);
                compute_block(b, r0, std::false_type{});
                tail();
                compute_block(b + STEP, r1, std::true_type{});
            } else {
                tail();
                compute_block(b, r0, std::true_type{});
            }
        } else {
            tail();
        }

        if constexpr (SOLO) {  // this wave holds the whole state of the item's rows
            next();
            l = sum_lane_groups(l);
            const float inv = 1.0f / l;
            const int h = hk * g + n;
            float2 sc = make_float2(1.f, 1.f);
            if (PF == PF_F16S && !sole) {
                float mx = 0.f;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) mx = fmaxf(mx, maxabs4(O[dt]));
                sc = row_scale(max_lane_groups(mx) * inv);
            }
            if (n < g) {
                __bf16* orow = (__bf16*)a.out + ((int64_t)item.seq0 * in.n_q_heads + h) * D;
                const int64_t slot = (int64_t)item.part_base + h;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    f32x4 v = O[dt] * inv;
                    if (sole) {
                        *(bf16x4*)(orow + 16 * dt + 4 * qd) = __builtin_convertvector(v, bf16x4);
                    } else {
                        if constexpr (PF == PF_F16S) v *= sc.y;
                        partial_store4<PF>(a.ws_o, slot * D + 16 * dt + 4 * qd, v);
                    }
                }
                if (qd == 0) {
                    if (!sole) stats_store<PF>(a.ws_ml + slot, m, l, sc.x);
                    else if (a.lse) a.lse[(int64_t)item.seq0 * in.n_q_heads + h] = (m + __log2f(l)) * 0.6931471805599453f;
                }
            }
            return;
        }

        // combine the four waves' states
        l = sum_lane_groups(l);
        if (n < g) {
            if (qd == 0) sm_ml[wave][n] = make_float2(m, l);
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) *(f32x4*)&sm_o[wave][n][16 * dt + 4 * qd] = O[dt];
        }
        __syncthreads();
        if (!sole) meta_store(sm.meta, mr, 1, threadIdx.x);  // (after the barrier: nobody still merges the previous item)
        for (int idx = threadIdx.x; idx < g * (D / 4); idx += 256) {
            const int r = idx / (D / 4), d4 = idx % (D / 4);
            float mw[4], M = -INFINITY;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                mw[w] = sm_ml[w][r].x;
                M = fmaxf(M, mw[w]);
            }
            float L = 0.f;
            f32x4 acc = (f32x4)(0.f);
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float wg = fast_exp2(mw[w] - M);
                L += wg * sm_ml[w][r].y;
                acc += wg * *(const f32x4*)&sm_o[w][r][4 * d4];
            }
            if (sole) {
                const int h = hk * g + r;
                const f32x4 res = acc * (1.0f / L);
                *(bf16x4*)((__bf16*)a.out + ((int64_t)item.seq0 * in.n_q_heads + h) * D + 4 * d4) = __builtin_convertvector(res, bf16x4);
                if (a.lse && d4 == 0) a.lse[(int64_t)item.seq0 * in.n_q_heads + h] = (M + __log2f(L)) * 0.6931471805599453f;
                continue;
            }
            const int64_t slot = (int64_t)item.part_base + hk * g + r;
            f32x4 row = acc * (1.0f / L);
            float2 sc = make_float2(1.f, 1.f);
            if constexpr (PF == PF_F16S) {  // the row's D/4 lanes are neighbours inside one wave, all of them in this loop
                float mx = maxabs4(row);
#pragma unroll
                for (int o = 1; o < D / 4; o *= 2) mx = fmaxf(mx, __shfl_xor(mx, o));
                sc = row_scale(mx);
                row *= sc.y;
            }
            partial_store4<PF>(a.ws_o, slot * D + 4 * d4, row);
            if (d4 == 0) stats_store<PF>(a.ws_ml + slot, M, L, sc.x);
        }
        if (sole || after) {
            __syncthreads();  // the combine buffers are free for the next item
            return;
        }
        // publish the partial; whoever completes the sequence's set merges it
        stores_done();
        __syncthreads();
        if (threadIdx.x == 0) sm.last = arrive_last(a, item.seq0, hk, sm.meta.ms[1] - sm.meta.ms[0]);
        __syncthreads();
#ifdef TAPER_WG_TRACE
        const long long t_m0 = wall_clock64();
#endif
        if (sm.last) merge_rows<D, 1, PF>(a, sm.meta, item.seq0, hk, sm.meta.ms[0], sm.meta.ms[1], threadIdx.x, 256);
#ifdef TAPER_WG_TRACE
        if (threadIdx.x == 0 && a.trace) a.trace[4 * blockIdx.x + 3] += wall_clock64() - t_m0;
#endif
    }
}

// Solo items [first, end) of a share, dealt to the waves (the plan lists them longest first; taking them as they get free cost tiny steps
// 0.3 us, a barrier and a counter, and evened out nothing that was seen).  Their partials are announced together; the sequences that are then complete (few: what the other items of a step deliver comes later as a rule) are
// merged by a wave each.  `announce`: there are partials among them, and merges are made in this launch.
// The next item's first block is asked for before this one's rows are stored, behind items of more than 32 tokens (before / behind, us, inputs taking turns: 2048 items of
// 40 tokens 92.6 / 94.9, 41.5 / 42.5 at head_dim 64; 1024 of 128 97.0 / 98.0; 2048 of 96 157.0 / 155.4; 4096 of 6 88 / 80; 8 kv heads here and below).
// It is also brought into the L2 while this one's last block is computed, behind items of more than 96 tokens: beside shared-prefix work (455 of 84 to 133 beside 4
// prefixes of 30000 tokens 172.5 touched, 175.2 not; 150 of 91 to 169 beside 2 of 150 to 300 at head_dim 64 16.4 / 16.6), and in launches of private work alone at head_dim 128 in runs
// of at most kSoloTouchRun.  Touched / not: 512 of 256 tokens (8 items a run) 91.0 / 94.2, 512 of 32 to 512 95.6 / 97.7, 600 of 130 (9 or 10) 59.0 / 60.3, 655 of 200 (10) 97.1 / 98.0.  In longer runs the waves
// drift apart and the machine is busy throughout, so that what is touched only waits in front of what is needed: 1500 of 130 on 4 kv heads (12) 88.3 / 81.9, 1008
// of 130 (16) 109.3 / 103.1, 1310 of 100 (20) 120.6 / 111.0, 1024 of 300 224.7 / 219.3.  Behind short items as well: 4096 of 6 107 / 91.  At head_dim 64 a block is half the bytes:
// 655 of 200 47.3 / 46.5, 400 of 100 to 400 35.0 / 34.6, 1310 of 100 52.8 / 52.3, the other way 1024 of 128 44.4 / 46.2.
constexpr int kSoloTouchFrom = 96, kSoloTouchRun = 10, kSoloAheadFrom = 32;
template <int D, int PF>
DEV void solo_run(const DecodeArgs& a, const Inputs& in, const Start& start, const int end, const int hk, const bool announce, PrivateSmem<D>& sm) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), first = start.first;
    // (back and forth: the wave with the longest item of one round has the shortest of the next)
    int k = first, turn = wave;
    if (k + turn < end) {
        taper_work_item item = start.item, after_it = {};
        i32x4 page = start.page, after_page = {};
        Ahead<D> w;
        begin_item<D>(in, item, page, hk, opaque(threadIdx.x) & 63, 0, w);
        for (bool more = true; more;) {
            k += 4;
            turn ^= 3;
            more = k + turn < end;
            if (more) {
                after_it = load_item(a, k + turn);
                after_page = private_pages(a, after_it, 0, 1);
            }
            const bool touch = more && item.n_tokens > kSoloTouchFrom && (in.n_parts_shared || (D == 128 && end - first <= kSoloTouchRun)), ahead = more && item.n_tokens > kSoloAheadFrom;
            const auto begin = [&] { begin_item<D>(in, after_it, after_page, hk, opaque(threadIdx.x) & 63, 0, w); };
            private_item<D, true, PF, false>(
                a, in, item, page, hk, 0, sm, w, [&] { if (touch) touch_block<D>(in, hk, after_page[0], after_page[1], sm.sink[wave]); }, [&] { if (ahead) begin(); });
            if (more && !ahead) begin();
            item = after_it;
            page = after_page;
        }
    }
    if (!announce) {
        __syncthreads();
        return;
    }
    stores_done();
    for (int it = first; it < end; it += 64) {
        __syncthreads();  // everyone's partial rows are stored; `todo` is free
        if (threadIdx.x < 64) {
            const int lane = opaque(threadIdx.x) & 63;
            bool mine = false;
            int seq = 0;
            if (it + lane < end && a.items[it + lane].kind == 1) {
                seq = a.items[it + lane].seq0;
                mine = arrive_last(a, seq, hk, a.merge_start[seq + 1] - a.merge_start[seq]);
            }
            const unsigned long long mask = __ballot(mine);
            if (mine) sm.todo[__popcll(mask & ((1ull << lane) - 1))] = seq;
            if (lane == 0) {
                sm.n_todo = __popcll(mask);
                sm.meta.ms[0] = -2 * kMetaWindow;  // (their merge entries are not in the window)
            }
        }
        __syncthreads();
        for (int i = wave; i < sm.n_todo; i += 4) {
            const int seq = __builtin_amdgcn_readfirstlane(sm.todo[i]);
            merge_rows<D, D / PartialVec<PF>::N / 8, PF>(a, sm.meta, seq, hk, a.merge_start[seq], a.merge_start[seq + 1], opaque(threadIdx.x) & 63, 64);
        }
    }
    __syncthreads();
}

// The private items of a workgroup: its share's solo items [it0, solo_end), the others [solo_end, it1) in order, then whatever it
// can take from its kv head's pool.  Every workgroup makes exactly one claim past the end of
// the pool; the one that makes the last of those puts the counter back to zero for the next
// launch.
//
// At an item's end nothing of the next one is in flight: its page ids and then its first blocks are asked for one after the other, 4 to 5 us each on a
// saturated machine.  Where the item is long the share's next item and its page ids are read at its start, and its first blocks are brought into the L2 while
// the last of this one is computed.  Touched / not, us, inputs taking turns, 8 kv heads.  Beside shared-prefix work behind items of more than 512 tokens: mixed batch 83.4 / 83.9,
// 44.9 / 45.1 at head_dim 64, 178.0 / 178.6 with half of its requests in the reduce phase.  In launches of private work alone at head_dim 128 behind more than 768: 163 items of 800 tokens
// 88.8 / 91.4, 256 of 1200 197.3 / 199.4, 100 of 1300 83.9 / 86.9, 50 of 2600 84.2 / 86.0; shorter ones end all at once, and what is touched waits in front of what is
// needed: 500 of 600 211.6 / 205.3, 400 of 700 199.5 / 195.0, 600 of 600 on 4 kv heads 138.5 / 131.4.  At head_dim 64 not in those: 512 of 600 107.5 / 103.5, 131 of 1000
// 51.1 / 50.0, 50 of 2600 43.9 / 43.4, the other way 256 of 1200 96.7 / 98.2.
DEV int touch_from(const Inputs& in, int d) { return in.n_parts_shared ? 512 : d == 128 ? 768 : INT_MAX; }
template <int D, int PF, bool HOLD>
DEV void private_items(const DecodeArgs& a, const Inputs& in, const Start& start, const bool announce, const int hk, const int after, PrivateSmem<D>& sm) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    int it0 = start.first;
    const int solo_end = it0 + start.n_solo, it1 = start.end;
    const int wgs_per_head = in.n_parts_shared + a.n_parts_private;  // = gridDim.x / n_kv_heads
    taper_work_item item = start.item;
    i32x4 page = start.page;
    bool given = it0 < it1 && it0 == solo_end;  // item and page are the next item's (at first the start record's)
    if (it0 < solo_end) {
        solo_run<D, PF>(a, in, start, solo_end, hk, announce, sm);
        it0 = solo_end;
    }
#ifdef TAPER_WG_TRACE
    bool turned = false;
#endif
    Ahead<D> w;
    for (;;) {
        int it = it0;
        if (it0 < it1) {
            ++it0;
        } else {
            if (a.n_pool_items == 0) return;
#ifdef TAPER_WG_TRACE
            if (threadIdx.x == 0 && a.trace && !turned) a.trace[4 * blockIdx.x + 1] = wall_clock64();  // own share done
            turned = true;
#endif
            if (threadIdx.x == 0) sm.pick = atomicAdd(a.pool_ctr + hk, 1);
            __syncthreads();
            const int i = __builtin_amdgcn_readfirstlane(sm.pick);
            __syncthreads();
            if (i >= a.n_pool_items) {
                if (threadIdx.x == 0 && i == a.n_pool_items + wgs_per_head - 1)
                    __hip_atomic_store(a.pool_ctr + hk, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                return;
            }
            it = a.pool_first + i;
        }
        if (!given) {
            item = load_item(a, it);
            page = private_pages(a, item, wave, 4);
        }
        given = it0 < it1 && item.n_tokens > touch_from(in, D);
        taper_work_item own = {};
        i32x4 own_page = {};
        if (given) {
            own = load_item(a, it0);
            own_page = private_pages(a, own, wave, 4);
        }
        private_item<D, false, PF, HOLD>(
            a, in, item, page, hk, after, sm, w,
            [&] { if (given && wave < (own.n_tokens + 31) >> 5) touch_block<D>(in, hk, own_page[0], own_page[1], sm.sink[wave]); }, [] {});
        item = own;
        page = own_page;
    }
}

// ---------------------------------------------------------------------------
// Shared-prefix kernel: a chunk of one request's prefix pages is staged in LDS
// once and multiplied against the query rows of all n_branch admitted branches x g
// heads.  16-row tiles are dealt round-robin to the four waves, up to 3 tiles per wave.
//
// KV goes from global memory straight into LDS, 16 KiB blocks (32 tokens at head_dim 128, 64 at 64), K in a ring of four
// halves, V in one of five: scores are made from K of one block while V of the block before is used, and three more are in flight,
// whatever the number of tiles.  Every wave-level 16-byte load lands as 1 KiB at a wave-uniform LDS address, lane after lane.  Which 16
// bytes of memory a lane fetches is free, and that is where V's bank swizzle is made: inside an odd 4-token quarter the two
// 128-byte halves of each 256 bytes change places, so that the 8-byte fragment reads of lane groups 0/1
// (2/3) hit different bank halves.
//
// The loads are written in assembly because the compiler does not see which buffer an LDS read touches and
// would wait for every outstanding load before each one; it is kept from moving anything across the waits by
// their memory clobbers.  (The loads have no register results, and the waits the compiler makes for its own
// loads only get longer by loads it does not know of.)
//
// What bounds it: on a saturated machine HBM, and above some ten branches the block's own instructions (a launch of shared work alone, 16
// requests of 32768 tokens, of the 310 us a bare read of the same pages takes, the loads without the computation 314 to 325: 2 branches
// 322 us, 8 339, 16 361 to 373, 24 484; before / with the loop described below 332 / 338 / 400 to 410 / 514).  Alone on the machine, the chain of a
// block: 0.39, 0.47, 0.70 to 0.74 and 0.89 us with 1 to 4, 4, 8 and 12 tiles (2, 8, 16, 24 branches), 0.25 of it the loads' issue and the barrier; 0.58, 0.64,
// 0.88 and 1.02 before.  What made the difference, in this order: page ids by one load in the middle of a block's work, not behind it
// (0.05); the maximum of eight scores in four instructions and page offsets by 32-bit products; V's two fragments of an operand by one
// read into its four registers (32 moves a block less); the scores a block ahead.  What is left is 16 matrix instructions a tile, 17 cycles each, and some
// 60 vector instructions.
// ---------------------------------------------------------------------------
template <int D>
struct SharedSmem {
    static constexpr int TILE_BYTES = 32 * D;                  // one (page, K or V, kv head) tile
    static constexpr int PAGE_BYTES = 2 * TILE_BYTES;
    static constexpr int BLOCK_BYTES = 16384;
    static constexpr int PAGES = BLOCK_BYTES / PAGE_BYTES;     // pages per block: 2 at head_dim 128, 4 at 64
    static constexpr int TOKENS = 16 * PAGES;
    // K of a block: the tiles of its pages one after the other.  V in 1 KiB chunks (token quarters at head_dim 128, pairs
    // of quarters at 64): pair of pages, chunk, page of the pair.  The two pages' fragments that make up one operand
    // are then 1 KiB apart, which one two-address read fetches into neighbouring registers.
    static constexpr int v_chunk(int page, int chunk) { return (page >> 1) * 2 * TILE_BYTES + chunk * 2048 + (page & 1) * 1024; }
    static constexpr int HALF = BLOCK_BYTES / 2;               // K or V of a block
    static constexpr int K_RING = 4, V_RING = 5;               // (a block's scores are made one iteration before its V is used)
    char k[K_RING * HALF], v[V_RING * HALF];
    int todo[64];  // branches of the current item whose partials are complete
    int n_todo;
    MergeMeta meta;
};

// The same through registers, for a pool that does not start at a multiple of 16 bytes (a view into a larger buffer, say):
// ordinary loads take any address, and that direct ones do is nothing to rely on.  Tiles are multiples of 2 KiB, so
// that the pool's start decides for all of them.
DEV void copy_to_lds(const char* base, unsigned off, char* lds, int lane) {
    u32x4 v;
    __builtin_memcpy(&v, base + off, 16);
    *(u32x4*)(lds + lane * 16) = v;
}
// All but this wave's N youngest loads have landed, its LDS reads are done, and every wave of the workgroup is here.
template <int N>
DEV void wait_loads_and_meet() {
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)\n\ts_barrier" ::"n"(N) : "memory");
}

// The partial rows of a shared-prefix item: tile k of this wave holds row 16 * (wave + 4k) + n of the
// item's R rows in lane column n, 4 values per 16-dim group and lane group.
template <int D, int NTW, int PF>
DEV void store_shared_partials(const DecodeArgs& a, const taper_work_item& item, const int hk, const int R, const int wave, const int n, const int qd, const float (&m)[NTW], const float (&l)[NTW],
                               const f32x4 (&O)[NTW][D / 16]) {
    constexpr int DT = D / 16;
#pragma unroll
    for (int k = 0; k < NTW; ++k) {
        {
            const float lt = sum_lane_groups(l[k]);
            const float inv = 1.0f / lt;
            float2 sc = make_float2(1.f, 1.f);
            if constexpr (PF == PF_F16S) {
                float mx = 0.f;
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) mx = fmaxf(mx, maxabs4(O[k][dt]));
                sc = row_scale(max_lane_groups(mx) * inv);
            }
            const int r = 16 * (wave + 4 * k) + n;
            if (r < R) {
                const int64_t slot = (int64_t)item.part_base + (int64_t)hk * R + r;
                if (qd == 0) stats_store<PF>(a.ws_ml + slot, m[k], lt, sc.x);
#pragma unroll
                for (int dt = 0; dt < DT; ++dt) {
                    f32x4 v = O[k][dt] * inv;
                    if constexpr (PF == PF_F16S) v *= sc.y;
                    partial_store4<PF>(a.ws_o, slot * D + 16 * dt + 4 * qd, v);
                }
            }
        }
    }
}

// Streams the item's tokens against the NA tiles wave, wave + 4, ... of its rows and stores their partial rows.
// Every wave of the workgroup takes its part in staging and meets the others once per block, whatever its NA.
template <int D, int NA, int PF, bool ANY>
DEV void shared_stream(const DecodeArgs& a, const Inputs& in, const taper_work_item& item, const i32x4 page, const i32x4 page2, const int hk,
                       SharedSmem<D>& sm, const int tid, const int wave) {
    typedef SharedSmem<D> Sm;
    constexpr int KS = D / 32, DT = D / 16, NT = NA ? NA : 1, QB = 8 * D;  // QB: bytes of a 4-token quarter of a V tile
    constexpr int LOADS = 4;  // wave-level loads per wave and block
    const int lane = tid & 63, n = lane & 15, qd = lane >> 4;
    const int Hkv = in.n_kv_heads, g = in.gqa;
    const unsigned page_bytes = Hkv * Sm::PAGE_BYTES;
    const char* kvb = (const char*)in.kv + (int64_t)hk * Sm::TILE_BYTES;
    const float c = a.scale_log2e;
    const scalar_row row = table_row(a, item);  // (wave-uniform: page ids come by scalar loads)
    const int n_tok = item.n_tokens, n_pages = (n_tok + 15) >> 4, n_blocks = (n_tok + Sm::TOKENS - 1) / Sm::TOKENS;
    const int R = item.n_branch * g;

    bf16x8 qf[NT][KS];
    float m[NT], l[NT];
    f32x4 O[NT][DT];

    // staging: at head_dim 128 a wave loads quarter `wave` of K and V of both pages, at 64 all of page `wave`
    const unsigned k_ring = lds_address(sm.k), v_ring = lds_address(sm.v);
    const unsigned off_k = lane * 16;
    const unsigned off_v = (lane ^ ((D == 128 ? wave & 1 : lane >> 5) << 3)) * 16;
    int pid[D == 128 ? 2 : 1];  // the pool pages this wave stages next
    auto fetch_ids = [&](int b) {  // past the last page (a block that ends early or does not exist): the last page
        if constexpr (D == 128) {
            typedef int i32x2 __attribute__((ext_vector_type(2), aligned(4)));
            const int bb = b < n_blocks ? b : n_blocks - 1;
            const i32x2 two = *(CONSTANT i32x2*)(row + 2 * bb);  // (a row of an odd number of pages: the entry behind it is read, not used)
            pid[0] = two[0];
            pid[1] = 2 * bb + 1 < n_pages ? two[1] : two[0];
        } else {
            const int i = 4 * b + wave;
            pid[0] = row[i < n_pages ? i : n_pages - 1];
        }
    };
    const unsigned v_bytes = Hkv * Sm::TILE_BYTES;  // from a page's K tiles to its V tiles
    auto stage = [&](int k_slot, int v_slot) {      // (byte offsets in the rings)
#pragma unroll
        for (int i = 0; i < 2; ++i) {  // (a page of two at head_dim 128, a half of a tile at 64)
            const char* from = kvb + (uint64_t)(unsigned)pid[D == 128 ? i : 0] * page_bytes + (D == 128 ? wave : i) * 1024;
            const int k_to = k_slot + (D == 128 ? i * Sm::TILE_BYTES + wave * 1024 : wave * Sm::TILE_BYTES + i * 1024);
            const int v_to = v_slot + (D == 128 ? Sm::v_chunk(i, wave) : Sm::v_chunk(wave, i));
            if constexpr (ANY) {
                copy_to_lds(from, off_k, sm.k + k_to, lane);
                copy_to_lds(from + v_bytes, off_v, sm.v + v_to, lane);
            } else {
                load_to_lds(from, off_k, k_ring + k_to);
                load_to_lds(from + v_bytes, off_v, v_ring + v_to);
            }
        }
    };
    // this lane's V fragment of 16-dim group dt (the swizzle: odd quarters have their 128-byte halves exchanged)
    const int v_lane = v_ring + (D == 128 ? qd * 2048 : (qd >> 1) * 2048 + (qd & 1) * QB) + n * 8;
    const int v_even = v_lane + (qd & 1) * 128, v_odd = v_lane - (qd & 1) * 128;
    // The scores of a block are made one iteration ahead of its exponentials, so that the matrix instructions of the one fill the time of
    // the vector instructions of the other.
    constexpr int H = Sm::PAGES / 2;  // halves of 32 tokens
    f32x4 sx[H][NT], sy[H][NT];
    bf16x8 kx[H][KS], ky[H][KS];
    auto read_k = [&](int k_slot, int hf) {
        const char* kp = sm.k + k_slot + hf * 2 * Sm::TILE_BYTES + lane * 16;
#pragma unroll
        for (int j = 0; j < KS; ++j) {
            kx[hf][j] = *(const bf16x8*)(kp + j * 1024);
            ky[hf][j] = *(const bf16x8*)(kp + Sm::TILE_BYTES + j * 1024);
        }
    };
    auto scores = [&](int hf) {
#pragma unroll
        for (int k = 0; k < NA; ++k) {
            sx[hf][k] = sy[hf][k] = (f32x4)(0.f);
#pragma unroll
            for (int j = 0; j < KS; ++j) {
                sx[hf][k] = mfma16(kx[hf][j], qf[k][j], sx[hf][k]);
                sy[hf][k] = mfma16(ky[hf][j], qf[k][j], sy[hf][k]);
            }
        }
    };
    auto read_v = [&](int v_slot, int hf, int h, bf16x4 (&va)[4], bf16x4 (&vb)[4]) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            // (an address of its own for each pair, so that the pair is one two-address read into the operand's four registers;
            // else the compiler joins reads of different pairs and moves half of the registers)
            const auto v = (__attribute__((address_space(3))) const bf16x4*)(uintptr_t)(unsigned)opaque(v_slot + hf * 2 * Sm::TILE_BYTES + (i & 1 ? v_odd : v_even) + (4 * h + i) * 128);
            va[i] = v[0];
            vb[i] = v[128];
        }
    };
    auto compute = [&](int b, int k_next, int v_slot, auto tail) {
        if constexpr (NA > 0) {
#pragma unroll
            for (int hf = 0; hf < H; ++hf) {
                const int nv = n_tok - Sm::TOKENS * b - 32 * hf;
                if (tail && nv <= 0) break;
                if (!tail) read_k(k_next, hf);
                bf16x4 vas[DT], vbs[DT];
                if constexpr (NA == 2) {
#pragma unroll
                    for (int h = 0; h < DT / 4; ++h) {
                        bf16x4 va[4], vb[4];
                        read_v(v_slot, hf, h, va, vb);
#pragma unroll
                        for (int i = 0; i < 4; ++i) vas[4 * h + i] = va[i], vbs[4 * h + i] = vb[i];
                    }
                }
                if (!tail && hf == 0) fetch_ids(b + 5);
                if (tail && nv < 32) {
#pragma unroll
                    for (int k = 0; k < NA; ++k) mask_tail(sx[hf][k], sy[hf][k], qd, nv);
                }
                bf16x8 pf[NA];
                softmax_block<DT, NA>(sx[hf], sy[hf], c, m, l, O, pf);
                if (!tail) scores(hf);
#pragma unroll
                for (int h = 0; h < DT / 4; ++h) {
                    bf16x4 va[4], vb[4];
                    if constexpr (NA == 2) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) va[i] = vas[4 * h + i], vb[i] = vbs[4 * h + i];
                    } else {
                        read_v(v_slot, hf, h, va, vb);
                    }
                    if (tail && nv < 32) zero_tail(va, vb, qd, nv);
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        const bf16x8 vf = cat(va[i], vb[i]);
#pragma unroll
                        for (int k = 0; k < NA; ++k) O[k][4 * h + i] = mfma16(vf, pf[k], O[k][4 * h + i]);
                    }
                }
                settle();
            }
        } else if (!tail) {
            fetch_ids(b + 5);
        }
    };

    // (the previous item's LDS reads of these buffers ended before its closing barriers)
#pragma unroll
    for (int b = 0; b < 4; ++b) {
        if constexpr (D == 128) {
            pid[0] = b < 2 ? page[2 * (b & 1)] : page2[2 * (b & 1)];
            pid[1] = b < 2 ? page[2 * (b & 1) + 1] : page2[2 * (b & 1) + 1];
        } else {
            pid[0] = page[b];
        }
        if (b < n_blocks) stage(b * Sm::HALF, b * Sm::HALF);
    }
    fetch_ids(4);
    const MetaRegs mr = meta_load(a, item, tid);
    if constexpr (NA > 0) {
#pragma unroll
        for (int k = 0; k < NA; ++k) {
            const int r = 16 * (wave + 4 * k) + n, rr = r < R ? r : 0;  // (lane columns past the last row repeat the first; not stored)
            const __bf16* qrow = (const __bf16*)in.q + ((int64_t)(item.seq0 + rr / g) * in.n_q_heads + hk * g + rr % g) * D;
#pragma unroll
            for (int j = 0; j < KS; ++j) qf[k][j] = *(const bf16x8*)(qrow + 8 * (4 * j + qd));
            m[k] = -INFINITY;
            l[k] = 0.f;
#pragma unroll
            for (int dt = 0; dt < DT; ++dt) O[k][dt] = (f32x4)(0.f);
        }
    }
    meta_store(sm.meta, mr, item.n_branch, tid);
    // (the queries' loads are waited for here: inside the loop that wait would also drain the blocks in flight, every time)
    if constexpr (NA > 0) {
#pragma unroll
        for (int k = 0; k < NA; ++k)
#pragma unroll
            for (int j = 0; j < KS; ++j) asm volatile("" : "+v"(qf[k][j]));
    }
    wait_loads_and_meet<0>();
    if constexpr (NA > 0) {
#pragma unroll
        for (int hf = 0; hf < H; ++hf) {
            read_k(0, hf);
            scores(hf);
        }
    }
    int v_slot = 0, k_slot = 0;  // of block b
    for (int b = 0; b < n_blocks - 1; ++b) {
        // block b + 1 is in LDS for every wave; everyone is done with K of block b and V of block b - 1
        if (b + 3 < n_blocks) wait_loads_and_meet<2 * LOADS>();
        else if (b + 3 == n_blocks) wait_loads_and_meet<LOADS>();
        else wait_loads_and_meet<0>();
        if (b + 4 < n_blocks) stage(k_slot, v_slot == 0 ? 4 * Sm::HALF : v_slot - Sm::HALF);  // block b + 4, where K of b and V of b - 1 were
        k_slot = (k_slot + Sm::HALF) & (Sm::K_RING * Sm::HALF - 1);
        compute(b, k_slot, v_slot, std::false_type{});
        v_slot = v_slot == 4 * Sm::HALF ? 0 : v_slot + Sm::HALF;
    }
    compute(n_blocks - 1, 0, v_slot, std::true_type{});
    if constexpr (NA > 0) {
        // (lane coordinates are derived afresh: shared with the ones above, they would stay live through the streaming loop)
        const int tid_e = opaque(threadIdx.x);
        store_shared_partials<D, NA, PF>(a, item, hk, R, wave, tid_e & 15, (tid_e & 63) >> 4, m, l, O);
    }
}

template <int D, int NTW, int PF, bool ANY>
DEV void shared_path(const DecodeArgs& a, const Inputs& in, const Start& start, const int hk, const int after, SharedSmem<D>& sm) {
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int it0 = start.first, it1 = start.end;
    taper_work_item item = start.item;
    i32x4 page = start.page, page2 = start.more;
    for (int it = it0; it < it1; ++it) {
        if (it != it0) {
            item = load_item(a, it);
            const scalar_row row = table_row(a, item);
            const int last = ((item.n_tokens + 15) >> 4) - 1;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                page[i] = row[min(D == 128 ? i : 4 * i + wave, last)];
                if (D == 128) page2[i] = row[min(4 + i, last)];
            }
        }
        const int tid = opaque(threadIdx.x);
        const int tiles = (item.n_branch * in.gqa + 15) >> 4;
        const int n_act = (tiles - wave + 3) >> 2;  // tiles wave, wave + 4, ...; 0 for a wave past the last tile (tiles >= 1)
        if (NTW >= 3 && n_act >= 3) shared_stream<D, NTW >= 3 ? 3 : 1, PF, ANY>(a, in, item, page, page2, hk, sm, tid, wave);
        else if (NTW >= 2 && n_act == 2) shared_stream<D, NTW >= 2 ? 2 : 1, PF, ANY>(a, in, item, page, page2, hk, sm, tid, wave);
        else if (n_act == 1) shared_stream<D, 1, PF, ANY>(a, in, item, page, page2, hk, sm, tid, wave);
        else shared_stream<D, 0, PF, ANY>(a, in, item, page, page2, hk, sm, tid, wave);
        if (after) {
            __syncthreads();  // the ring is free for the next item
            continue;
        }
        // publish the partials; merge every branch whose set is now complete
        stores_done();
        __syncthreads();
#ifdef TAPER_WG_TRACE
        const long long t_m0 = wall_clock64();
#endif
        arrive_and_merge<D, PF>(a, sm.meta, sm.todo, &sm.n_todo, item, hk, opaque(threadIdx.x));
#ifdef TAPER_WG_TRACE
        __syncthreads();
        if (tid == 0 && a.trace) a.trace[4 * blockIdx.x + 3] += wall_clock64() - t_m0;
#endif
        __syncthreads();
    }
}

// ---------------------------------------------------------------------------
// The attention launch of a layer: workgroup (share, kv head).  Shares below n_parts_shared
// stream shared prefixes, the others private tokens; both kinds run side by side.
// ---------------------------------------------------------------------------
template <int D>
union StepSmem {
    SharedSmem<D> sh;
    PrivateSmem<D> pr;
};
// ALLP: a launch without shared-prefix work (no shared path in the kernel).  ANY: the pool may start at any address.
template <int D, int NTW, int PF, bool ALLP, bool ANY>
DEV void run_share(const DecodeArgs& a, const Inputs& in, char* smem_raw) {
    const int part = blockIdx.x / in.n_kv_heads;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    Start start = load_start(in, part, wave);
    int hk = blockIdx.x - part * in.n_kv_heads + (start.turn & kPartTurnMask);
    if (hk >= in.n_kv_heads) hk -= in.n_kv_heads;
    int after = a.merge_after;  // (kept: read from the arguments where it is used it costs a trip at every item's end)
    asm volatile("" : "+s"(after));
#ifdef TAPER_WG_TRACE  // trace builds only (wg_trace.py): per-workgroup clocks -- start, own share done, left, time in merges
    long long* trace = a.trace;
    if (threadIdx.x == 0 && trace) trace[4 * blockIdx.x] = wall_clock64();
#endif
    if (!ALLP && part < in.n_parts_shared) {
        shared_path<D, NTW, PF, ANY>(a, in, start, hk, after, *reinterpret_cast<SharedSmem<D>*>(smem_raw));
        __syncthreads();
        start.first = start.end = start.n_solo = 0;  // (what is left for it is the pool)
    }
#ifdef TAPER_WG_TRACE
    if (threadIdx.x == 0 && trace) trace[4 * blockIdx.x + 1] = wall_clock64();  // shared share done (a private share: overwritten when it is done)
#endif
    private_items<D, PF, !ALLP && D == 128>(a, in, start, !after && (start.turn & kPartSoloPartials), hk, after, *reinterpret_cast<PrivateSmem<D>*>(smem_raw));
#ifdef TAPER_WG_TRACE
    if (threadIdx.x == 0 && trace) trace[4 * blockIdx.x + 2] = wall_clock64();
#endif
}

template <int D, int NTW, int PF, bool ALLP>
__global__ __launch_bounds__(256, 2) void decode_kernel(u32x4 pointers, u32x4 queries, DecodeArgs) {
    __shared__ __attribute__((aligned(16))) char smem_raw[sizeof(StepSmem<D>)];
    run_share<D, NTW, PF, ALLP, false>(decode_args(), unpack_inputs(pointers, queries), smem_raw);
}
// Steps with shared-prefix work over a pool that does not start at a multiple of 16 bytes (a kernel of its own: a branch per block
// in the others cost them 1 to 2 %, mixed batch on one kv head 26.4 -> 26.7 us, 64 branches 270 -> 274).
template <int D, int PF>
__global__ __launch_bounds__(256, 2) void any_start_kernel(u32x4 pointers, u32x4 queries, DecodeArgs) {
    __shared__ __attribute__((aligned(16))) char smem_raw[sizeof(StepSmem<D>)];
    run_share<D, 3, PF, false, true>(decode_args(), unpack_inputs(pointers, queries), smem_raw);
}

// ---------------------------------------------------------------------------
// The merges of a step as a launch behind the attention launch: workgroup (sequence, kv head), a wave per query head.
//
// A sequence's partials are complete when its last item is, and where a step's items all end together the workgroup that is
// last merges a whole request alone, a few rows at a time: 12 us after 16 us of streaming in the mixed batch on one kv
// head (36 partials), 37 after 22 for 13 branches of 40 partials.  Here every row has a wave of its own: three dependent trips to memory (the
// sequence's entry range, the entries, statistics and rows together) for up to 32 partials, whatever their number of rows.
//
// Slots of LPR lanes (16 bytes each) hold one partial row; slot i takes entries i, i + SLOTS, ...  Lane k has the statistics of the
// k-th entry.  The order of the sum follows from the number of entries alone.
// ---------------------------------------------------------------------------
template <int CTRL>
DEV float row_rotate(float v) {
    return __uint_as_float(__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), 0x120 + CTRL, 0xf, 0xf, true));
}
DEV float wave_max(float v) {
    v = fmaxf(v, row_rotate<8>(v));
    v = fmaxf(v, row_rotate<4>(v));
    v = fmaxf(v, row_rotate<2>(v));
    return max_lane_groups(fmaxf(v, row_rotate<1>(v)));
}
DEV float wave_sum(float v) {
    v += row_rotate<8>(v);
    v += row_rotate<4>(v);
    v += row_rotate<2>(v);
    return sum_lane_groups(v + row_rotate<1>(v));
}
template <int D, int PF>
__global__ __launch_bounds__(1024) void merge_kernel(DecodeArgs a) {
    typedef PartialVec<PF> Vec;
    typedef typename Vec::type vec;
    constexpr int LPR = D / Vec::N, SLOTS = 64 / LPR, ROW_BYTES = LPR * 16, T = 32 / SLOTS;
    const int lane = threadIdx.x & 63, j = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int s = blockIdx.x / a.n_kv_heads, hk = blockIdx.x % a.n_kv_heads;
    typedef const __attribute__((address_space(4))) int32_t* scalar_row;
    const int e0 = ((scalar_row)a.merge_start)[s], e1 = ((scalar_row)a.merge_start)[s + 1];
    const int slot = lane / LPR, col = lane % LPR;
    const auto rows = partial_buffer(a.ws_o), stats = partial_buffer(a.ws_ml);
    float M = -INFINITY, L = 0.f;
    vec acc = (vec)(0.f);
    for (int c = e0; c < e1; c += 64) {
        const bool real = c + lane < e1;
        const taper_merge_entry me = a.merge[real ? c + lane : e0];
        // (a single private item is its sequence's whole context and wrote the result)
        if (e1 - e0 == 1 && __builtin_amdgcn_readfirstlane(me.rows_per_head) == a.gqa) return;
        const int row = real ? me.first_row + hk * me.rows_per_head + j : -1;
        const u32x4 st = coherent_load16(stats, real ? (unsigned)row * 16 : kNoLoad);
        u32x4 o[T];
        auto fetch = [&](const int t0) {
#pragma unroll
            for (int t = 0; t < T; ++t) {
                const int r = __shfl(row, (t0 + t) * SLOTS + slot);
                o[t] = coherent_load16(rows, r >= 0 ? (unsigned)r * ROW_BYTES + 16 * col : kNoLoad);
            }
        };
        fetch(0);
        const float m = real ? __uint_as_float(st[0]) : -INFINITY;
        const float mn = fmaxf(M, wave_max(m)), keep = fast_exp2(M - mn);  // first entries: exp2(-inf) = 0
        const float w = fast_exp2(m - mn) * __uint_as_float(st[1]);       // (the row was stored divided by its sum)
        const float ws = PF == PF_F16S ? w * __uint_as_float(st[2]) : w;
        L = L * keep + wave_sum(w);
        acc *= keep;
        M = mn;
        auto add = [&](const int t0) {
#pragma unroll
            for (int t = 0; t < T; ++t) acc += __shfl(ws, (t0 + t) * SLOTS + slot) * Vec::unpack(o[t]);
        };
        add(0);
        if (e1 - c > 32) {
            fetch(T);
            add(T);
        }
    }
#pragma unroll
    for (int o = LPR; o < 64; o *= 2)
#pragma unroll
        for (int i = 0; i < Vec::N; ++i) acc[i] += __shfl_xor(acc[i], o);
    if (slot == 0) {
        const int64_t h = (int64_t)s * a.n_q_heads + hk * a.gqa + j;
        *(typename Vec::out_type*)((__bf16*)a.out + h * D + Vec::N * col) = __builtin_convertvector(acc * (1.0f / L), typename Vec::out_type);
        if (a.lse && col == 0) a.lse[h] = (M + __log2f(L)) * 0.6931471805599453f;
    }
}

// Physical slot of every logical position, from the device copy of the plan.
__global__ __launch_bounds__(256) void resolve_slots_kernel(StepArgs a, int64_t* slots, int64_t stride) {
    const int s = blockIdx.x;
    const int64_t t = (int64_t)blockIdx.y * 256 + threadIdx.x;
    if (t >= stride) return;
    int64_t v = -1;
    if (t < a.ctx_len[s]) {
        const int32_t* row = a.bt + (int64_t)s * a.bt_stride;
        const int pl = a.prefix_len[s];
        if (t < pl) {
            v = (int64_t)row[t >> 4] * 16 + (t & 15);
        } else {
            int64_t jj = t - pl;
            int k = a.seg_start[s];
            while (jj >= a.seg_len[k]) jj -= a.seg_len[k++];  // t < ctx_len: k stays inside the sequence's segments
            v = (int64_t)row[a.seg_page0[k] + (jj >> 4)] * 16 + (jj & 15);
        }
    }
    slots[(int64_t)s * stride + t] = v;
}

// KV append: the new key and value rows of every sequence (bf16 [S][Hkv][D]) go to
// slot[s] = page * 16 + token of the pool, in the tile layouts the attention kernels read:
// K element d at (d/8)*128 + tok*8 + d%8 (16-byte groups of 8 dims), V element d at
// (tok/4)*4D + d*4 + tok%4.  One workgroup per sequence, thread = (K or V, kv head, group of 8 dims).  Bound by
// the launch and two trips to memory side by side (the slot, the row); K and V of a group are different threads'
// work so that each has one load and one address to make.
__global__ __launch_bounds__(256) void kv_append_kernel(const __bf16* __restrict__ k_new, const __bf16* __restrict__ v_new,
                                                        const int64_t* __restrict__ slot, __bf16* __restrict__ kv,
                                                        const int n_kv_heads, const int D) {
    const int s = blockIdx.x, rows = n_kv_heads * (D / 8);
    const int shift = D == 128 ? 4 : 3;  // (D is 64 or 128)
    for (int i = threadIdx.x; i < 2 * rows; i += blockDim.x) {
        const bool is_v = i >= rows;
        const int r = is_v ? i - rows : i, hk = r >> shift, d8 = r & (D / 8 - 1);
        const bf16x8 x = *(const bf16x8*)((is_v ? v_new : k_new) + ((int64_t)s * rows + r) * 8);
        const int64_t sl = slot[s];
        const int tok = (int)(sl & 15);
        __bf16* t = kv + (((sl >> 4) * 2 + is_v) * n_kv_heads + hk) * (16LL * D);
        if (is_v) {
#pragma unroll
            for (int j = 0; j < 8; ++j) t[(tok >> 2) * (4 * D) + (8 * d8 + j) * 4 + (tok & 3)] = x[j];
        } else {
            *(bf16x8*)(t + d8 * 128 + tok * 8) = x;
        }
    }
}

// ---------------------------------------------------------------------------
hipError_t launch_kv_append(const void* k_new, const void* v_new, const int64_t* slot, void* kv, int n_seqs, int n_kv_heads,
                            int head_dim, hipStream_t s) {
    if (n_seqs == 0) return hipSuccess;
    hipLaunchKernelGGL(kv_append_kernel, dim3(n_seqs), dim3(256), 0, s, (const __bf16*)k_new, (const __bf16*)v_new, slot,
                       (__bf16*)kv, n_kv_heads, head_dim);
    return hipGetLastError();
}

// ---------------------------------------------------------------------------
// Measurement aid, not a step of the path: a plain streaming read.  Every workgroup reads a
// contiguous slice in 4 KiB pieces, 16 bytes per lane, nontemporal, two pieces per wave in
// flight; nothing is computed but an XOR that keeps the loads alive.  What this reaches on the
// same bytes and launch shape is the rate the machine leaves for any read-bound kernel.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(256) void stream_read_kernel(const u32x4* __restrict__ base, int64_t pieces_per_wg, unsigned* sink) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const u32x4* mine = base + (int64_t)blockIdx.x * pieces_per_wg * 256;  // 256 x 16 B = one 4 KiB piece
    u32x4 acc = {0, 0, 0, 0};
    for (int64_t i = 2 * wave; i < pieces_per_wg; i += 8) {
        u32x4 v[2][4];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int64_t piece = i + u < pieces_per_wg ? i + u : i;
#pragma unroll
            for (int k = 0; k < 4; ++k) v[u][k] = __builtin_nontemporal_load(mine + piece * 256 + 64 * k + lane);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int k = 0; k < 4; ++k) acc ^= v[u][k];
    }
    if ((acc.x ^ acc.y ^ acc.z ^ acc.w) == 0x9e3779b9u && sink) sink[0] = 1;  // (practically never: the loads must not be dropped)
}

hipError_t launch_stream_read(const void* base, int64_t pieces_per_wg, int n_workgroups, unsigned* sink, hipStream_t s) {
    hipLaunchKernelGGL(stream_read_kernel, dim3(n_workgroups), dim3(256), 0, s, (const u32x4*)base, pieces_per_wg, sink);
    return hipGetLastError();
}

template <int D, int PF>
static hipError_t launch_decode_as(const StepArgs& a, const dim3 grid, const int ntw, hipStream_t s) {
    const dim3 block(256);
    if (a.n_parts_shared == 0) hipLaunchKernelGGL((decode_kernel<D, 1, PF, true>), grid, block, 0, s, pack_pointers(a), pack_queries(a), static_cast<const DecodeArgs&>(a));
    else if (ntw > 3) return hipErrorInvalidValue;
    else if ((uintptr_t)a.kv & 15) hipLaunchKernelGGL((any_start_kernel<D, PF>), grid, block, 0, s, pack_pointers(a), pack_queries(a), static_cast<const DecodeArgs&>(a));
    else if (ntw <= 1) hipLaunchKernelGGL((decode_kernel<D, 1, PF, false>), grid, block, 0, s, pack_pointers(a), pack_queries(a), static_cast<const DecodeArgs&>(a));
    else if (ntw == 2) hipLaunchKernelGGL((decode_kernel<D, 2, PF, false>), grid, block, 0, s, pack_pointers(a), pack_queries(a), static_cast<const DecodeArgs&>(a));
    else hipLaunchKernelGGL((decode_kernel<D, 3, PF, false>), grid, block, 0, s, pack_pointers(a), pack_queries(a), static_cast<const DecodeArgs&>(a));
    if (a.merge_after) hipLaunchKernelGGL((merge_kernel<D, PF>), dim3(a.n_seqs * a.n_kv_heads), dim3(64 * a.gqa), 0, s, static_cast<const DecodeArgs&>(a));
    return hipGetLastError();
}

hipError_t launch_decode(const StepArgs& a, hipStream_t s) {
    const int n_parts = a.n_parts_shared + a.n_parts_private;
    if (n_parts == 0) return hipSuccess;
    const dim3 grid(n_parts * a.n_kv_heads);
    const int ntw = a.n_parts_shared ? (a.max_row_tiles_shared + 3) / 4 : 1;
    const bool f32 = a.partial_format == PF_F32;
    if (a.head_dim == 128) return f32 ? launch_decode_as<128, PF_F32>(a, grid, ntw, s) : launch_decode_as<128, PF_F16S>(a, grid, ntw, s);
    if (a.head_dim == 64) return f32 ? launch_decode_as<64, PF_F32>(a, grid, ntw, s) : launch_decode_as<64, PF_F16S>(a, grid, ntw, s);
    return hipErrorInvalidValue;
}

hipError_t launch_resolve_slots(const StepArgs& a, int64_t* slots, int64_t stride, hipStream_t s) {
    if (stride <= 0) return hipSuccess;
    const dim3 grid(a.n_seqs, (unsigned)((stride + 255) / 256)), block(256);
    hipLaunchKernelGGL(resolve_slots_kernel, grid, block, 0, s, a, slots, stride);
    return hipGetLastError();
}

}  // namespace taper
