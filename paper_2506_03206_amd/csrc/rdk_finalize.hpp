// Per-row finish of the verification step (Alg. 4, steps 2 and 4-10), shared by the stand-alone
// verify call and by the fused redistribute+verify calls.
//
// Input: for every row three partial sums per block of BLOCK ids (sum q', sum max(0, p - q'),
// sum min(p, q')), written by a streaming pass.  One workgroup per row (verify_finalize_wide_kernel, finish_row_quarters;
// the bonus draw takes one wavefront per row) then
//   1. adds the partials in fp64 (alpha, residual mass, sum q'), draws the Philox uniforms,
//   2. finds the blocks in which the two inverse-CDF thresholds are crossed,
//   3. re-reads (or re-computes) those blocks and scans them in fp64 for the exact ids,
//   4. decides acceptance in fp64, and, when its row is the last of its sequence to arrive, runs the first-rejection scan.
// Where q' comes from is the `QP` policy: memory (a materialised q' row) or a formula.  A policy hands out q' of
// four consecutive ids in kStages steps on a `Pending` record, each step issuing the loads whose addresses the
// step before produced; the kernel runs step k for ALL blocks it needs before step k + 1, so a chain of dependent
// loads costs kStages round trips in total rather than per block.
#pragma once
#include <type_traits>

#include "rdk_rowstats.hpp"

namespace rdk {

struct FinalizeArgs {
    rdk_verify_desc_t d;
    const void *p;
    int64_t ldp;
    const SoftStat *pstat;   // [B, p_splits] (logit p only)
    int p_splits;
    const float *part_q, *part_r, *part_a;   // [B, nblk]
    int nblk;
    int32_t *draft_ids;
    uint8_t *accept;
    float *alpha, *resid_mass;
    int32_t *resid_ids, *n_accepted, *out_tokens;
    uint64_t *seq_rec;       // [B, 2] one record per row for the per-sequence scan in the finish (NULL: the scan is not done there)
    uint64_t nonce;          // its bits mark a record as written by this call
};

// ---- A meeting of workgroups without a second launch.  Each party stores its record -- what the others need of it, tagged
// with bits of a number that no other call uses, so that the records need no clearing beforehand -- with device-scope
// stores (they go through to the memory that all XCDs share), waits until it has arrived there, and reads the records of
// all.  The party whose record arrives last finds all of them: it carries on alone, the others are done.  (Several may find
// all of them: what follows has to give the same result when it is done twice.)  Nobody waits for anybody, so the order in
// which workgroups run does not matter.  The one that carries on clears the records, so that a replay of the same call from
// a HIP graph, which brings the same number again, starts from cleared ones.  Two round trips to memory, about 2.5 us,
// where a launch of its own takes about 4.
// That somebody finds all records rests on gfx950 and not on the language: two parties that each store and then read the other
// are ordered by sequentially consistent fences only, and with relaxed atomics both may read the old value there.  Here a store of
// device scope is written through to the memory that device-scope loads read (both pass by what the caches of an XCD hold for
// themselves), stores count in vmcnt, and a wavefront past `s_waitcnt vmcnt(0)` has its record there before its loads are
// issued; the compiler moves nothing across the asm.  On another target each of the three has to be looked at again: were it
// not so, nobody would scan, and n_accepted and out_tokens would keep what they held.  The fence that the language asks for
// (seq_cst, device scope, in the place of the wait) writes back and invalidates caches, once per row: 256 rows of 128256 ids
// 122.3 -> 127.7 us sparse, 39.9 -> 43.6 Eq. 3, 1024 rows of 151936 ids 914 -> 943.
template <typename T>
__device__ __forceinline__ void agent_store(T *p, T v)
{
    __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
template <typename T>
__device__ __forceinline__ T agent_load(const T *p)
{
    return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
__device__ __forceinline__ void wait_for_stores() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

constexpr int kScanMaxGamma = 63;   // one lane per token of a sequence: gamma drafts and the residual token

// Steps 4-10 of Alg. 4 for the sequence of `row`, done by the row of the sequence whose record arrives last.  Called by one
// wavefront of the row's workgroup, with the row's draft, residual token and accept flag in lane 0.
// Record of a row: {draft, tag} and {residual token, tag with the accept flag as its lowest bit}.
__device__ __forceinline__ void scan_sequence(const FinalizeArgs &a, int64_t row, int32_t dtok, int32_t rtok, uint8_t acc)
{
    if (a.seq_rec == nullptr) return;
    const int g = a.d.gamma, lane = lane_id();
    const int64_t s = row / g, b0 = s * g;
    const uint64_t tag0 = a.nonce & 0xFFFFFFFF00000000ull, tag1 = (a.nonce << 32) & 0xFFFFFFFE00000000ull;
    if (lane == 0) {
        agent_store(a.seq_rec + 2 * row, tag0 | (uint32_t)dtok);
        agent_store(a.seq_rec + 2 * row + 1, tag1 | ((uint64_t)(acc != 0) << 32) | (uint32_t)rtok);
    }
    wait_for_stores();
    const bool in = lane < g;
    uint64_t r0 = tag0, r1 = tag1;
    if (in) {
        r0 = agent_load(a.seq_rec + 2 * (b0 + lane));
        r1 = agent_load(a.seq_rec + 2 * (b0 + lane) + 1);
    }
    if (__ballot((r0 & 0xFFFFFFFF00000000ull) != tag0 || (r1 & 0xFFFFFFFE00000000ull) != tag1) != 0ull) return;
    if (in) {
        agent_store(a.seq_rec + 2 * (b0 + lane), (uint64_t)0);
        agent_store(a.seq_rec + 2 * (b0 + lane) + 1, (uint64_t)0);
    }
    const unsigned long long rejected = __ballot(in && ((r1 >> 32) & 1ull) == 0ull);
    const int j = rejected ? __ffsll(rejected) - 1 : g;
    if (lane == 0 && a.n_accepted) a.n_accepted[s] = j;
    if (lane <= g && a.out_tokens)
        a.out_tokens[s * (g + 1) + lane] = lane < j ? (int32_t)(uint32_t)r0 : (lane == j && in) ? (int32_t)(uint32_t)r1 : -1;
}

// q' read back from memory.
struct QpMemory {
    static constexpr bool kSpreadRows = false;
    static constexpr int kStages = 1;
    const float *q;
    int64_t ldq;
    int N;
    struct Row {
        const float *qr;
        int N;
        struct Pending {
            float4 v;
        };
        template <int K>
        __device__ __forceinline__ void stage(Pending &t, int64_t idx) const
        {
            t.v = rdk::load4<RDK_PROB_F32>(qr, idx, N, 0.f);
        }
        __device__ __forceinline__ float4 result(Pending &t, int64_t) const { return t.v; }
        __device__ __forceinline__ float load1(int j) const { return qr[j]; }
    };
    __device__ __forceinline__ Row row(int64_t b) const { return Row{q + b * ldq, N}; }
};

// Runs step K of the policy on the SUB records of one block (nothing when the block is not wanted).
template <int K, int SUB, class Row>
__device__ __forceinline__ void stage_block(const Row &r, typename Row::Pending (&t)[SUB], int base, bool wanted)
{
    if (!wanted) return;   // also false for the lanes beyond a block shorter than 256 ids
#pragma unroll
    for (int i = 0; i < SUB; ++i) r.template stage<K>(t[i], (int64_t)base + i * 256 + lane_id() * 4);
}

__device__ __forceinline__ double lane_partial_sum(const float *part, int nblk, int per_lane)
{
    const int c0 = lane_id() * per_lane;
    double s = 0.0;
    for (int t = 0; t < per_lane; t += 4) {   // four loads in flight at a time
        float v[4];
#pragma unroll
        for (int x = 0; x < 4; ++x) v[x] = (t + x < per_lane && c0 + t + x < nblk) ? part[c0 + t + x] : 0.f;
#pragma unroll
        for (int x = 0; x < 4; ++x) s += (double)v[x];
    }
    return s;
}

// Block in which the inclusive prefix of `part` first exceeds thr (-1 if none) and the prefix before it.  Lane l has added up
// the per_lane consecutive blocks from l * per_lane (lane_sum); those of the lane in which the threshold is crossed are read again,
// one per lane: a scan of 64 lanes takes a fifth of the instructions that one lane needs to walk through 32 blocks of its own
// (N = 128256, 8 positions: fused 18.8 -> 18.1 us a call, draft draw 15.6 -> 14.8; N = 1024, 16 positions 8.63 -> 8.31).  Only
// blocks with mass can be crossed: the scan adds in another order for every lane, so a lane behind the last block may hold an ulp
// more than that block.  Where rounding leaves no crossing among them it is the last block with a positive sum.
__device__ __forceinline__ int locate_block(const float *part, int nblk, int per_lane, double lane_sum, double thr,
                                            double &prefix_before)
{
    const double incl = wave_inclusive_scan(lane_sum);
    const unsigned long long hits = __ballot(incl > thr);
    if (hits == 0ull) return -1;
    const int src = __ffsll(hits) - 1, c0 = src * per_lane, c1 = min(c0 + per_lane, nblk);
    double before = lane_value(incl - lane_sum, src);
    int blk = -1;
    for (int c = c0; c < c1; c += kWave) {
        const double x = c + lane_id() < c1 ? (double)part[c + lane_id()] : 0.0;
        const double to = before + wave_inclusive_scan(x);
        const unsigned long long over = __ballot(x > 0.0 && to > thr), some = __ballot(x > 0.0);
        if (over != 0ull || some != 0ull) {
            const int at = over != 0ull ? __ffsll(over) - 1 : 63 - __clzll(some);
            blk = c + at;
            prefix_before = lane_value(to - x, at);
        }
        if (over != 0ull) break;
        before = lane_value(to, kWave - 1);
    }
    return blk;
}

// The block sums of a lane, v[t] = that of block lane * per_lane + t (0 beyond nblk); R = blocks a lane can hold.
// A lane's blocks are consecutive in memory, so the lanes of one load are per_lane words apart and every load
// instruction touches up to 64 cache lines.  When the row, the blocks per lane and the block count all are multiples
// of four words, groups of four blocks are read by one unconditional 16-byte load each (a group is then wholly inside
// or wholly outside the row; the address of an outside group is clamped and its values dropped): a quarter of the
// line requests and no branch around any load.
template <int R>
__device__ __forceinline__ void load_partials(const float *part, int nblk, int per_lane, float (&v)[R])
{
    static_assert(R % 4 == 0, "a lane holds whole groups of four block sums");
    const int c0 = lane_id() * per_lane;
    if (((uintptr_t)part & 15) == 0 && per_lane % 4 == 0 && nblk % 4 == 0 && nblk >= 4) {   // the same for all lanes
#pragma unroll
        for (int t = 0; t < R; t += 4) {
            float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
            if (t < per_lane) {
                const float4 y = *(const float4 *)(part + min(c0 + t, nblk - 4));
                if (c0 + t < nblk) x = y;
            }
            v[t] = x.x; v[t + 1] = x.y; v[t + 2] = x.z; v[t + 3] = x.w;
        }
    } else {
#pragma unroll
        for (int t = 0; t < R; ++t) v[t] = (t < per_lane && c0 + t < nblk) ? part[c0 + t] : 0.f;
    }
}

template <int R>
__device__ __forceinline__ double sum_partials(const float (&v)[R])
{
    double s = 0.0;
#pragma unroll
    for (int t = 0; t < R; ++t) s += (double)v[t];
    return s;
}

// Element (i, e) of a lane's block registers: sub-block i, component e, both run-time values.
template <int SUB>
__device__ __forceinline__ float pick(const float4 (&w)[SUB], int i, int e)
{
    float r = 0.f;
#pragma unroll
    for (int ii = 0; ii < SUB; ++ii) {
        const float t = e == 0 ? w[ii].x : e == 1 ? w[ii].y : e == 2 ? w[ii].z : w[ii].w;
        r = ii == i ? t : r;
    }
    return r;
}

// Which of a lane's four ids the threshold crosses, given that it crosses one: excl = the prefix before them, l0 .. l2 their own
// first sums.  Like a block (locate_block), an id is crossed only if it has a weight: the sums beside it may differ by an ulp.
__device__ __forceinline__ int crossed_id(float w0, float w1, float w2, double l0, double l1, double l2, double excl, double thr)
{
    return w0 > 0.f && excl + l0 > thr ? 0 : w1 > 0.f && excl + l1 > thr ? 1 : w2 > 0.f && excl + l2 > thr ? 2 : 3;
}

// Smallest id of the block with a positive weight whose inclusive prefix of weights exceeds thr_local; if rounding leaves none,
// the last id of the block with a positive weight.  wv[i] = weights of ids base + i*256 + lane*4 .. +3.
template <int SUB>
__device__ __forceinline__ int search_block(const float4 (&wv)[SUB], int base, double thr_local)
{
    const int lane = lane_id();
    double carried = 0.0;
    int last_positive = -1;
#pragma unroll
    for (int i = 0; i < SUB; ++i) {
        const int idx = base + i * 256 + lane * 4;
        const double l0 = (double)wv[i].x, l1 = l0 + (double)wv[i].y, l2 = l1 + (double)wv[i].z, l3 = l2 + (double)wv[i].w;
        const double incl = wave_inclusive_scan(l3);
        const double excl = carried + (incl - l3);
        const unsigned long long hits = __ballot(l3 > 0.0 && excl + l3 > thr_local);
        if (hits != 0ull) {
            const int src = __ffsll(hits) - 1;
            const int e = crossed_id(wv[i].x, wv[i].y, wv[i].z, l0, l1, l2, excl, thr_local);
            return lane_value(idx + e, src);
        }
        const int mine = wv[i].w > 0.f ? 3 : wv[i].z > 0.f ? 2 : wv[i].y > 0.f ? 1 : wv[i].x > 0.f ? 0 : -1;
        const unsigned long long pos = __ballot(mine >= 0);
        if (pos != 0ull) {
            const int src = 63 - __clzll(pos);
            last_positive = lane_value(idx + mine, src);
        }
        carried += lane_value(incl, kWave - 1);
    }
    return last_positive;
}

// The same for a block of 64 ids held one per lane (w = weight of id base + lane).
__device__ __forceinline__ int search_block1(float w, int base, double thr_local)
{
    const double incl = wave_inclusive_scan((double)w);
    const unsigned long long hits = __ballot(w > 0.f && incl > thr_local);
    if (hits != 0ull) return base + (__ffsll(hits) - 1);
    const unsigned long long pos = __ballot(w > 0.f);
    return pos != 0ull ? base + (63 - __clzll(pos)) : -1;
}

// Which row a one-row workgroup takes when the policy re-computes q' from tables that the kernel before it left in the
// L2 of one XCD (the sparse product sweeps the rows of a 32-position block on one XCD when there are 8 k such blocks):
// consecutive workgroup ids go to consecutive XCDs, so workgroup i takes a row of the blocks that XCD i % 8 has swept.
// Any other batch shape keeps the identity; the mapping only decides which cache a row's lookups find warm.
__device__ __forceinline__ int64_t xcd_row(int64_t i, int B)
{
    if (B % 256 != 0) return i;
    const int64_t per_xcd = B / 8;
    return (i % 8) * per_xcd + i / 8;
}
constexpr int kFinalizeRows = 4;   // rows (wavefronts) per workgroup of the bonus draw

// The bonus draw t ~ p (Alg. 4, step 8, else-branch) of one row by one wavefront: part_r = the row's block sums of p.
template <int KIND, int BLOCK>
__global__ __launch_bounds__(kFinalizeRows * kWave) void bonus_finalize_kernel(FinalizeArgs a)
{
    constexpr int SUB = BLOCK / 256;
    constexpr int kRegBlocks = 8;                                   // block sums a lane keeps in registers
    const rdk_verify_desc_t &d = a.d;
    const int wid = threadIdx.x / kWave, lane = lane_id();
    const int64_t row = (int64_t)blockIdx.x * kFinalizeRows + wid;
    if (row >= d.B) return;                                         // a whole wavefront; the kernel has no barrier
    const void *pr = row_ptr<KIND>(a.p, a.ldp, row);
    float m = 0.f, inv = 1.f;
    if (KIND != RDK_PROB_F32) {
        const SoftStat rs = merged_row_stat<KIND>(a.pstat, a.p_splits, row);
        m = rs.m;
        inv = 1.0f / rs.s;
    }
    const float pfill = KIND == RDK_PROB_F32 ? 0.f : -INFINITY;
    const float *part = a.part_r + row * a.nblk;
    const int per_lane = ((a.nblk + kWave - 1) / kWave + 3) & ~3;   // blocks per lane, in whole groups of four
    const bool in_regs = per_lane <= kRegBlocks;
    float v[kRegBlocks];
    if (in_regs) load_partials(part, a.nblk, per_lane, v);
    const double lane_r = in_regs ? sum_partials(v) : lane_partial_sum(part, a.nblk, per_lane);
    uint32_t words[4];
    position_words(d.seed, d.offset + (uint64_t)row, words);
    const double R = wave_sum(lane_r);
    int32_t rtok = -1;
    if (R > 0.0) {
        const double thr = word_to_unit(words[3]) * R;
        double before = 0.0;
        const int blk = locate_block(part, a.nblk, per_lane, lane_r, thr, before);
        if (blk >= 0) {
            const int base = blk * BLOCK;
            float4 w[SUB];
#pragma unroll
            for (int i = 0; i < SUB; ++i) w[i] = load4<KIND>(pr, base + i * 256 + lane * 4, d.N, pfill);
#pragma unroll
            for (int i = 0; i < SUB; ++i)
                w[i] = make_float4(to_weight<KIND>(w[i].x, m, inv), to_weight<KIND>(w[i].y, m, inv), to_weight<KIND>(w[i].z, m, inv),
                                   to_weight<KIND>(w[i].w, m, inv));
            rtok = search_block<SUB>(w, base, thr - before);
        }
    }
    if (lane == 0) {
        a.accept[row] = 0;
        if (a.alpha) a.alpha[row] = 0.f;
        if (a.resid_mass) a.resid_mass[row] = (float)R;
        a.resid_ids[row] = rtok;
    }
}

// The finish of one row by a workgroup, for the policies that re-compute q' one id per lane (blocks of 64 ids).  A lone
// wavefront pays the full latency of every dependent instruction, and half of its time went into adding up and searching the
// three kinds of block sums one after the other; here wavefront 0 takes the sums of q' and the draft's block, wavefront 1
// the residual sums and the residual's block, wavefront 2 alpha (and the two values of a draft the caller supplied).  Every
// wavefront of the workgroup calls it.
//   REGS               block sums a lane keeps in registers (one kind per wavefront)
//   setup              hands out where q' comes from and the softmax maximum and 1 / normaliser of a logit target row (0 and 1 for
//                      probabilities); called once the block sums are asked for, so that what it reads comes with them
//   part_q, _r, _a     the row's a.nblk block sums of q', max(0, p - q') and min(p, q') (LDS or memory)
struct WideScratch {   // LDS
    double d[2];       // alpha, residual mass
    int i[2];          // the drafted id, the residual id
    float f[2];        // q' and p at the draft
};

template <class Row>
struct FinishSetup {
    Row row;
    float m, inv;
};

template <int KIND, int REGS, class Setup>
__device__ __forceinline__ void finish_row_wide(const FinalizeArgs &a, const Setup &setup, int64_t row, const void *pr, const float *part_q,
                                                const float *part_r, const float *part_a, WideScratch &sh, int wid, int lane)
{
    const rdk_verify_desc_t &d = a.d;
    const int N = d.N;
    const float pfill = KIND == RDK_PROB_F32 ? 0.f : -INFINITY;
    const bool draw_draft = d.sample_draft;
    const int per_lane = ((a.nblk + kWave - 1) / kWave + 3) & ~3;   // blocks per lane, in whole groups of four
    const bool in_regs = per_lane <= REGS;
    uint32_t words[4] = {0u, 0u, 0u, 0u};
    int blk = -1;                // the block of this wavefront's draw (-1: nothing to draw) and the threshold inside it
    double thr_local = 0.0;
    if (wid < 3) {
        // 1. one kind of block sums per wavefront
        const float *part = wid == 0 ? part_q : wid == 1 ? part_r : part_a;
        const bool wanted = wid == 0 ? draw_draft : true;
        float v[REGS];
        double lane_s = 0.0;
        if (wanted && in_regs) load_partials(part, a.nblk, per_lane, v);
        const auto given = setup();
        const auto &qrow = given.row;
        const float m = given.m, inv = given.inv;
        position_words(d.seed, d.offset + (uint64_t)row, words);   // while the sums are on their way
        if (wanted) lane_s = in_regs ? sum_partials(v) : lane_partial_sum(part, a.nblk, per_lane);
        const double T = wanted ? wave_sum(lane_s) : 0.0;
        if (wid < 2 && wanted && T > 0.0) {
            const double thr = word_to_unit(words[wid == 0 ? 0 : 2]) * T;
            double before = 0.0;
            blk = locate_block(part, a.nblk, per_lane, lane_s, thr, before);
            thr_local = thr - before;
        }
        if (lane == 0 && wid >= 1) sh.d[2 - wid] = T;   // wavefront 1: residual mass -> [1], wavefront 2: alpha -> [0]
        // 2. the block of the draft (wavefront 0) and of the residual draw (wavefront 1), one id per lane; the two values of
        //    a caller's draft (wavefront 2)
        if (wid < 2) {
            int tok = -1;
            if (blk >= 0) {
                const int base = blk * 64, id = base + lane;
                typename std::decay<decltype(qrow)>::type::Pending1 t;
                qrow.template stage1<0>(t, id);
                float pv = pfill;
                if (id < N) pv = load1<KIND>(pr, id);
                qrow.template stage1<1>(t, id);
                qrow.template stage1<2>(t, id);
                const float wq = qrow.result1(t, id);
                const float pw = to_weight<KIND>(pv, m, inv);
                tok = search_block1(wid == 0 ? wq : fmaxf(pw - wq, 0.f), base, thr_local);
                if (wid == 0 && tok >= 0) {
                    const float qd = lane_value(wq, tok - base), pd = lane_value(pw, tok - base);
                    if (lane == 0) {
                        sh.f[0] = qd;
                        sh.f[1] = pd;
                    }
                }
            }
            if (lane == 0) sh.i[wid] = tok;
        } else if (!draw_draft) {
            const int32_t dtok = a.draft_ids[row];
            if (dtok >= 0 && dtok < N) {
                const float pd = to_weight<KIND>(load1<KIND>(pr, dtok), m, inv), qd = qrow.load1(dtok);
                if (lane == 0) {
                    sh.f[0] = qd;
                    sh.f[1] = pd;
                }
            }
        }
    }
    __syncthreads();
    // 3. the accept test and the row's outputs
    int32_t dtok = -1;
    uint8_t acc = 0;
    if (threadIdx.x == 0) {
        dtok = draw_draft ? sh.i[0] : a.draft_ids[row];
        const bool d_ok = dtok >= 0 && dtok < N;
        if (d_ok) acc = (word_to_unit(words[1]) * (double)sh.f[0] < (double)sh.f[1]) ? 1 : 0;
        if (draw_draft) a.draft_ids[row] = dtok;
        a.accept[row] = acc;
        if (a.alpha) a.alpha[row] = (float)sh.d[0];
        if (a.resid_mass) a.resid_mass[row] = (float)sh.d[1];
        a.resid_ids[row] = sh.i[1];
    }
    if (wid == 0) scan_sequence(a, row, dtok, sh.i[1], acc);
}

// How many block sums a lane holds in registers (REGS): the code that adds and searches them is unrolled, runs once, and is
// fetched while it runs, so a row takes the shortest that holds its blocks; above 4096 of them they are read again from memory.
// Whole calls of 8 positions: draft draw, N = 32000 (500 blocks): 64 registers 14.7 us, 32 13.4, 8 12.6; N = 128256 (2004 blocks):
// 64 17.8, 32 16.4; N = 250000 (3908 blocks): read again 36.5, 64 24.7.  Fused, N = 32000: 64 17.4, 8 15.4; N = 128256: 64 20.6,
// 32 19.8.  The step of 16: draft draw, N = 48000 (752 blocks) 32 registers 14.9 us, 16 14.3; N = 64000 (1000) 15.1, 14.4; fused,
// N = 48000 17.7, 17.1, bf16 logits 24.0, 23.4.  The step of 40: draft draw, N = 151936 (2376) 64 registers 18.8, 40 17.8;
// N = 163840 (2560) 20.2, 19.2; fused, N = 151936 23.2, 22.7, bf16 logits 30.5, 29.6.
template <class F>
inline void with_block_regs(int nblk, const F &f)
{
    if (nblk <= 8 * kWave) f(std::integral_constant<int, 8>{});
    else if (nblk <= 16 * kWave) f(std::integral_constant<int, 16>{});
    else if (nblk <= 32 * kWave) f(std::integral_constant<int, 32>{});
    else if (nblk <= 40 * kWave) f(std::integral_constant<int, 40>{});
    else f(std::integral_constant<int, 64>{});
}

// One row per workgroup of four wavefronts, block sums over 64 ids in memory.
template <int KIND, int REGS, class QP>
__global__ __launch_bounds__(4 * kWave) void verify_finalize_wide_kernel(FinalizeArgs a, QP qp)
{
    __shared__ WideScratch sh;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    const int64_t row = xcd_row(blockIdx.x, a.d.B);
    const void *pr = row_ptr<KIND>(a.p, a.ldp, row);
    auto setup = [&]() {
        FinishSetup<typename QP::Row> r{qp.row(row), 0.f, 1.f};
        if (KIND != RDK_PROB_F32) {
            const SoftStat rs = merged_row_stat<KIND>(a.pstat, a.p_splits, row);
            r.m = rs.m;
            r.inv = 1.0f / rs.s;
        }
        return r;
    };
    finish_row_wide<KIND, REGS>(a, setup, row, pr, a.part_q + row * a.nblk, a.part_r + row * a.nblk, a.part_a + row * a.nblk, sh, wid, lane);
}

// ---- The finish of one row by eight wavefronts, for block sums over 1024 ids (Alg. 4, steps 2 and 4-6 for one position).
// A lone wavefront pays the full latency of every dependent step; here
//   1. three wavefronts add up one kind of block sum each in fp64 (sum q', residual mass, alpha) and find the block
//      in which the inverse-CDF threshold of the draft / of the residual draw is crossed;
//   2. eight wavefronts take a quarter of one of the two blocks each (256 ids, four per lane: the target values from
//      memory, q' from the policy) and scan it in fp64;
//   3. with the totals of the quarters before its own, each finds the crossing in its quarter (or its last id with
//      a positive weight, the answer when rounding leaves no crossing);
//   4. the first wavefront picks the first crossing, tests acceptance in fp64 and writes the row's outputs.
// The arithmetic, its order and the conventions are those of the one-wavefront search (search_block).
// Every wavefront of the workgroup calls it (more than eight may; the others only meet the barriers).
//   scratch        kFinishFloats floats of LDS
//   sq, sr, sa     the row's nblk block sums of q', max(0, p - q') and min(p, q') (LDS or memory)
//   pm, pinv       softmax maximum and 1 / normaliser of a logit target row (0 and 1 for probabilities)
//   words          the position's four uniforms (Alg. 4: draft, accept, residual, bonus)
//   quads          where q' comes from: begin() issues the loads that need no target value, end() hands out q' of four
//                  ids given their target weights, at() q' of one id
//   SCAN           whether the per-sequence scan follows (scan_sequence)
//   held           called by every thread with the two blocks once they are known: where the target weights and q' of both lie in
//                  LDS (block by block, 256 quads of either), put there by the wavefronts that hold them, or null
constexpr int kFinishFloats = 64;
constexpr int kHeldQuads = 4 * 256;

struct NotHeld {
    __device__ __forceinline__ const float4 *operator()(int, int) const { return nullptr; }
};

// Four quads of a lane, in the order of finish_row_quarters' quarters.
__device__ __forceinline__ void hold_block(float4 *to, const float (&v)[4][4], int lane)
{
#pragma unroll
    for (int i = 0; i < 4; ++i) to[i * kWave + lane] = make_float4(v[i][0], v[i][1], v[i][2], v[i][3]);
}

template <int KIND, bool SCAN, class Quads, class Held = NotHeld>
__device__ __forceinline__ void finish_row_quarters(float *scratch, const float *sq, const float *sr, const float *sa, int nblk,
                                                    const FinalizeArgs &fin, int64_t row, const void *pr, float pm, float pinv,
                                                    int N, const Quads &quads, const uint32_t (&words)[4], int wid,
                                                    int lane, const Held &held = Held{})
{
    constexpr int kBlock = 1024;
    double *fd = (double *)scratch;                   // [0..1] local thresholds, [2] alpha, [3] residual mass, [4..11] quarter totals
    int *fi = (int *)(scratch + 24);                  // [0..1] the two blocks (-1: nothing to draw)
    float4 *fc = (float4 *)(scratch + 32);            // per quarter: crossing id, last positive id, q' and p at the candidate
    const rdk_verify_desc_t &d = fin.d;
    const bool draw_draft = d.sample_draft;
    if (wid < 3) {
        const float *part = wid == 0 ? sq : wid == 1 ? sr : sa;
        const bool wanted = wid == 0 ? draw_draft : true;
        constexpr int kRegBlocks = 8;
        const int per_lane = ((nblk + kWave - 1) / kWave + 3) & ~3;
        const bool in_regs = per_lane <= kRegBlocks;
        float v[kRegBlocks];
        double lane_s = 0.0;
        if (wanted) {
            if (in_regs) {
                load_partials(part, nblk, per_lane, v);
                lane_s = sum_partials(v);
            } else {
                lane_s = lane_partial_sum(part, nblk, per_lane);
            }
        }
        const double T = wanted ? wave_sum(lane_s) : 0.0;
        int blk = -1;
        double thr = 0.0, before = 0.0;
        if (wid < 2 && wanted && T > 0.0) {
            thr = word_to_unit(words[wid == 0 ? 0 : 2]) * T;
            blk = locate_block(part, nblk, per_lane, lane_s, thr, before);
        }
        if (lane == 0) {
            if (wid < 2) {
                fi[wid] = blk;
                fd[wid] = thr - before;
            }
            if (wid >= 1) fd[4 - wid] = T;            // wavefront 1: residual mass -> [3], wavefront 2: alpha -> [2]
        }
    }
    __syncthreads();
    const float4 *in_lds = held(fi[0], fi[1]);
    const int fb = wid >> 2, fq = wid & 3;            // which of the two blocks, which quarter of it
    const int fblk = wid < 8 ? fi[fb] : -1;
    const bool factive = fblk >= 0;
    const int64_t fidx = (int64_t)max(fblk, 0) * kBlock + fq * 256 + lane * 4;
    float qp4[4] = {0.f, 0.f, 0.f, 0.f}, pv4[4] = {0.f, 0.f, 0.f, 0.f}, wv4[4] = {0.f, 0.f, 0.f, 0.f};
    double l0 = 0.0, l1 = 0.0, l2 = 0.0, l3 = 0.0, incl = 0.0;
    int last_pos = -1;
    if (factive) {
        if (in_lds) {
            const float4 pl = in_lds[fb * 512 + fq * kWave + lane], ql = in_lds[fb * 512 + 256 + fq * kWave + lane];
            pv4[0] = pl.x; pv4[1] = pl.y; pv4[2] = pl.z; pv4[3] = pl.w;
            qp4[0] = ql.x; qp4[1] = ql.y; qp4[2] = ql.z; qp4[3] = ql.w;
        } else {
            typename Quads::Token t = quads.begin(fblk, fq, fidx);
            const float4 pl = load4<KIND>(pr, fidx, N, KIND == RDK_PROB_F32 ? 0.f : -INFINITY);
            pv4[0] = to_weight<KIND>(pl.x, pm, pinv); pv4[1] = to_weight<KIND>(pl.y, pm, pinv);
            pv4[2] = to_weight<KIND>(pl.z, pm, pinv); pv4[3] = to_weight<KIND>(pl.w, pm, pinv);
            quads.end(t, fidx, pv4, qp4);
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) wv4[e] = fb == 0 ? qp4[e] : fmaxf(pv4[e] - qp4[e], 0.f);
        l0 = (double)wv4[0]; l1 = l0 + (double)wv4[1]; l2 = l1 + (double)wv4[2]; l3 = l2 + (double)wv4[3];
        incl = wave_inclusive_scan(l3);
        if (lane == kWave - 1) fd[4 + wid] = incl;
        const int mine = wv4[3] > 0.f ? 3 : wv4[2] > 0.f ? 2 : wv4[1] > 0.f ? 1 : wv4[0] > 0.f ? 0 : -1;
        const unsigned long long pos = __ballot(mine >= 0);
        if (pos != 0ull) last_pos = lane_value((int)fidx + mine, 63 - __clzll(pos));
    }
    __syncthreads();
    if (factive) {
        double carried = 0.0;
        for (int i = 0; i < fq; ++i) carried += fd[4 + 4 * fb + i];
        const double thr_local = fd[fb];
        const double excl = carried + (incl - l3);
        const unsigned long long hits = __ballot(l3 > 0.0 && excl + l3 > thr_local);
        int hit = -1;
        if (hits != 0ull) {
            const int e = crossed_id(wv4[0], wv4[1], wv4[2], l0, l1, l2, excl, thr_local);
            hit = lane_value((int)fidx + e, __ffsll(hits) - 1);
        }
        const int cand = hit >= 0 ? hit : last_pos;
        float qc = 0.f, pc = 0.f;
        if (cand >= 0) {
            const int off = cand - (fblk * kBlock + fq * 256), src = off / 4, e = off % 4;
            qc = lane_value(e == 0 ? qp4[0] : e == 1 ? qp4[1] : e == 2 ? qp4[2] : qp4[3], src);
            pc = lane_value(e == 0 ? pv4[0] : e == 1 ? pv4[1] : e == 2 ? pv4[2] : pv4[3], src);
        }
        if (lane == 0) fc[wid] = make_float4(__int_as_float(hit), __int_as_float(last_pos), qc, pc);
    }
    __syncthreads();
    int tok[2] = {-1, -1};
    int32_t dtok = -1;
    uint8_t acc = 0;
    if (threadIdx.x == 0) {
        float qd = 0.f, pd_w = 0.f;
        for (int b = 0; b < 2; ++b) {
            if (fi[b] < 0) continue;
            int chosen = -1;
            for (int i = 0; i < 4 && chosen < 0; ++i)
                if (__float_as_int(fc[4 * b + i].x) >= 0) chosen = i;
            if (chosen < 0)
                for (int i = 3; i >= 0 && chosen < 0; --i)
                    if (__float_as_int(fc[4 * b + i].y) >= 0) chosen = i;
            if (chosen >= 0) {
                const float4 c4 = fc[4 * b + chosen];
                tok[b] = __float_as_int(c4.x) >= 0 ? __float_as_int(c4.x) : __float_as_int(c4.y);
                if (b == 0) {
                    qd = c4.z;
                    pd_w = c4.w;
                }
            }
        }
        dtok = tok[0];
        if (!draw_draft) {                            // the caller's draft: its two values are fetched here
            dtok = fin.draft_ids[row];
            if (dtok >= 0 && dtok < N) {
                pd_w = to_weight<KIND>(load1<KIND>(pr, dtok), pm, pinv);
                qd = quads.at(dtok, pd_w);
            }
        }
        const bool d_ok = dtok >= 0 && dtok < N;
        if (d_ok) acc = (word_to_unit(words[1]) * (double)qd < (double)pd_w) ? 1 : 0;
        if (draw_draft) fin.draft_ids[row] = dtok;
        fin.accept[row] = acc;
        if (fin.alpha) fin.alpha[row] = (float)fd[2];
        if (fin.resid_mass) fin.resid_mass[row] = (float)fd[3];
        fin.resid_ids[row] = tok[1];
    }
    if (SCAN && wid == 0) scan_sequence(fin, row, dtok, tok[1], acc);
}

// q' of four ids from a policy's row (its steps run back to back: one quarter of a block per wavefront).
template <class Row, int STAGES>
struct PolicyQuads {
    const Row &r;
    typedef typename Row::Pending Token;
    __device__ __forceinline__ Token begin(int, int, int64_t fidx) const
    {
        Token t;
        r.template stage<0>(t, fidx);
        return t;
    }
    __device__ __forceinline__ void end(Token &t, int64_t fidx, const float (&)[4], float (&qp4)[4]) const
    {
        if (STAGES > 1) r.template stage<1>(t, fidx);
        if (STAGES > 2) r.template stage<2>(t, fidx);
        const float4 v = r.result(t, fidx);
        qp4[0] = v.x; qp4[1] = v.y; qp4[2] = v.z; qp4[3] = v.w;
    }
    __device__ __forceinline__ float at(int dtok, float) const { return r.load1(dtok); }
};

// One row per workgroup of eight wavefronts, block sums over 1024 ids in memory.
template <int KIND, class QP>
__global__ __launch_bounds__(8 * kWave) void verify_finalize_quarters_kernel(FinalizeArgs a, QP qp)
{
    __shared__ __attribute__((aligned(16))) float scratch[kFinishFloats];
    const rdk_verify_desc_t &d = a.d;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    const int64_t row = blockIdx.x;
    const void *pr = row_ptr<KIND>(a.p, a.ldp, row);
    float m = 0.f, inv = 1.f;
    if (KIND != RDK_PROB_F32) {
        const SoftStat rs = merged_row_stat<KIND>(a.pstat, a.p_splits, row);
        m = rs.m;
        inv = 1.0f / rs.s;
    }
    uint32_t words[4];
    position_words(d.seed, d.offset + (uint64_t)row, words);
    const typename QP::Row qrow = qp.row(row);
    const PolicyQuads<typename QP::Row, QP::kStages> quads{qrow};
    finish_row_quarters<KIND, true>(scratch, a.part_q + row * a.nblk, a.part_r + row * a.nblk, a.part_a + row * a.nblk, a.nblk, a, row, pr,
                              m, inv, d.N, quads, words, wid, lane);
}

// ---- Draft draw alone (Alg. 4 step 2 on the drafter's side, before a target row exists): one wavefront per row,
// block sums of q' in, the drafted id and q' at that id out.
struct DraftArgs {
    int32_t B, N;
    uint64_t seed, offset;
    const float *part_q;   // [B, nblk]
    int nblk;
    int32_t *draft_ids;
    float *q_draft;        // may be NULL
};

// One wavefront; pq = the row's block sums of q' (LDS or memory), REGS = how many of them a lane keeps in registers.
template <int BLOCK, int REGS, int STAGES, class Row>
__device__ __forceinline__ void draft_row(const DraftArgs &a, const Row &qrow, int64_t row, const float *pq)
{
    constexpr int SUB = BLOCK >= 256 ? BLOCK / 256 : 1;
    constexpr int kLanes = BLOCK >= 256 ? kWave : BLOCK / 4;
    constexpr int kRegBlocks = REGS;
    const int lane = lane_id();
    const int per_lane = ((a.nblk + kWave - 1) / kWave + 3) & ~3;   // blocks per lane, in whole groups of four
    const bool in_regs = per_lane <= kRegBlocks;
    float vq[kRegBlocks];
    double lane_q;
    if (in_regs) load_partials(pq, a.nblk, per_lane, vq);
    lane_q = in_regs ? sum_partials(vq) : lane_partial_sum(pq, a.nblk, per_lane);
    uint32_t words[4];
    position_words(a.seed, a.offset + (uint64_t)row, words);
    const double Q = wave_sum(lane_q);
    int blk = -1;
    double thr = 0.0, before = 0.0;
    if (Q > 0.0) {
        thr = word_to_unit(words[0]) * Q;
        blk = locate_block(pq, a.nblk, per_lane, lane_q, thr, before);
    }
    int32_t dtok = -1;
    float qd = 0.f;
    if (blk >= 0) {
        const int base = blk * BLOCK;
        if constexpr (BLOCK == 64) {
            typename Row::Pending1 td;
            const int id = base + lane;
            qrow.template stage1<0>(td, id);
            qrow.template stage1<1>(td, id);
            qrow.template stage1<2>(td, id);
            const float wdv = qrow.result1(td, id);
            dtok = search_block1(wdv, base, thr - before);
            if (dtok >= 0) qd = lane_value(wdv, dtok - base);
        } else {
            const bool holds = lane < kLanes;
            typename Row::Pending td[SUB];
            float4 wd[SUB];
            stage_block<0, SUB>(qrow, td, base, holds);
            if (STAGES > 1) stage_block<1, SUB>(qrow, td, base, holds);
            if (STAGES > 2) stage_block<2, SUB>(qrow, td, base, holds);
#pragma unroll
            for (int i = 0; i < SUB; ++i)
                wd[i] = holds ? qrow.result(td[i], (int64_t)base + i * 256 + lane * 4) : make_float4(0.f, 0.f, 0.f, 0.f);
            dtok = search_block<SUB>(wd, base, thr - before);
            if (dtok >= 0) {
                const int off = dtok - base;
                qd = lane_value(pick<SUB>(wd, off / 256, off % 4), (off % 256) / 4);
            }
        }
    }
    if (lane == 0) {
        a.draft_ids[row] = dtok;
        if (a.q_draft) a.q_draft[row] = qd;
    }
}

template <int BLOCK, int REGS, class QP>
__global__ __launch_bounds__(kWave) void draft_finalize_kernel(DraftArgs a, QP qp)
{
    const int64_t row = QP::kSpreadRows ? xcd_row(blockIdx.x, a.B) : (int64_t)blockIdx.x;
    const typename QP::Row qrow = qp.row(row);
    draft_row<BLOCK, REGS, QP::kStages>(a, qrow, row, a.part_q + row * a.nblk);
}

template <int BLOCK, class QP>
rdk_status_t launch_draft_finalize(const DraftArgs &a, QP qp, hipStream_t st)
{
    with_block_regs(a.nblk, [&](auto regs) {
        RDK_TIMED_LAUNCH("draft_finalize_kernel", (draft_finalize_kernel<BLOCK, decltype(regs)::value, QP>), dim3((unsigned)a.B), dim3(kWave),
                         0, st, a, qp);
    });
    RDK_LAUNCH_CHECK("draft_finalize_kernel");
    return RDK_OK;
}

// Per-sequence scan as a launch of its own (sequences longer than one workgroup's wavefronts).
__global__ void sequence_scan_kernel(int S, int gamma, const int32_t *draft_ids, const uint8_t *accept,
                                     const int32_t *resid_ids, int32_t *n_accepted, int32_t *out_tokens);

rdk_status_t launch_sequence_scan(const rdk_verify_desc_t &d, const int32_t *draft_ids, const uint8_t *accept,
                                  const int32_t *resid_ids, int32_t *n_accepted, int32_t *out_tokens, hipStream_t st);

// Whether the finish itself runs the per-sequence scan of a call, and the records for it.  rec: [B, 2] uint64 of scratch.
inline void set_scan(FinalizeArgs &a, uint64_t *rec)
{
    const bool wanted = a.d.gamma > 0 && a.d.gamma <= kScanMaxGamma && (a.n_accepted || a.out_tokens);
    a.seq_rec = wanted ? rec : nullptr;
    a.nonce = wanted ? call_nonce() : 0;
}

// The scan as a launch of its own where the finish has not done it.
inline rdk_status_t scan_if_left(const FinalizeArgs &a, hipStream_t st)
{
    if (a.d.gamma > 0 && !a.seq_rec && (a.n_accepted || a.out_tokens))
        return launch_sequence_scan(a.d, a.draft_ids, a.accept, a.resid_ids, a.n_accepted, a.out_tokens, st);
    return RDK_OK;
}

// rec: [B, 2] uint64 of scratch for the per-sequence scan.
template <int KIND, int BLOCK, bool HAS_Q, class QP>
rdk_status_t launch_finalize(FinalizeArgs a, QP qp, uint64_t *rec, hipStream_t st)
{
    const rdk_verify_desc_t &d = a.d;
    if constexpr (!HAS_Q) {
        // the bonus draw: one wavefront per row, four rows per workgroup
        const int blocks = (d.B + kFinalizeRows - 1) / kFinalizeRows;
        RDK_TIMED_LAUNCH("verify_finalize_kernel", (bonus_finalize_kernel<KIND, BLOCK>), dim3(blocks), dim3(kFinalizeRows * kWave), 0, st, a);
        RDK_LAUNCH_CHECK("verify_finalize_kernel");
        return RDK_OK;
    } else {
        // One wavefront per row is bound by its own chain of dependent steps: every row gets a workgroup, four wavefronts
        // for blocks of 64 ids whose q' is re-computed, eight for blocks of 1024.
        set_scan(a, rec);
        if constexpr (BLOCK == 64)
            with_block_regs(a.nblk, [&](auto regs) {
                RDK_TIMED_LAUNCH("verify_finalize_kernel", (verify_finalize_wide_kernel<KIND, decltype(regs)::value, QP>), dim3((unsigned)d.B),
                                 dim3(4 * kWave), 0, st, a, qp);
            });
        else
            RDK_TIMED_LAUNCH("verify_finalize_kernel", (verify_finalize_quarters_kernel<KIND, QP>), dim3((unsigned)d.B), dim3(8 * kWave),
                             0, st, a, qp);
        RDK_LAUNCH_CHECK("verify_finalize_kernel");
        return scan_if_left(a, st);
    }
}

}  // namespace rdk
