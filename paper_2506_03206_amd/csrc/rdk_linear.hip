// Linear-time redistribution (Alg. 1, steps 1-2) in its two forms:
//   * the first-order closed form, Eq. 3 of the paper (no matrix, needs the target row p);
//   * (the product M^T q' with the top-k sparse kernel lives in rdk_sparse.hip);
//   * the identity kernel: token-level intersection itself.
// Step 1 (token-level intersection, Eq. 1) is folded in: the drafter row is only ever used divided
// by its own sum over the kept slots.
#include <cfloat>

#include "rdk_finalize.hpp"

namespace rdk {

namespace {

constexpr int kThreads = 256;
constexpr int kWaves = kThreads / kWave;

struct LinearWs {
    SoftStat *pstat;   // [B, p_splits]  target row softmax statistics (logit p only)
    SoftStat *qstat;   // [B]            drafter row: (max, sum exp) or (0, sum)
    float *tpart;      // [B, t_splits, 8]  Taylor partial sums (4 used by the two-pass form, 8 by the one-pass form)
    int p_splits, t_splits;
};

LinearWs carve(const KernelHandle &h, int32_t B, void *ws)
{
    LinearWs w;
    w.p_splits = row_splits(B, h.N, kWaves);
    w.t_splits = w.p_splits;
    char *p = (char *)ws;
    w.pstat = (SoftStat *)p; p += align_up((size_t)B * w.p_splits * sizeof(SoftStat), 256);
    w.qstat = (SoftStat *)p; p += align_up((size_t)B * sizeof(SoftStat), 256);
    w.tpart = (float *)p;
    return w;
}

// ------------------------------------------------------------------------------------------------
// The kept ids ascend, so the kept ids inside one chunk of kChunk target ids own a contiguous run of slots
// lo .. hi-1 (chunk_lo of the kernel handle).  A wavefront reads that run of the drafter row and of kept_ids with
// coalesced loads and scatters it through a private LDS array (kChunk words + one spare word per lane) into id
// order; afterwards lane l holds the unnormalised drafter weights of the ids  base + i*256 + l*4 .. +3  (i = 0..3),
// the same ids whose target values it loads; ids that are not kept get 0.  This replaces one gather per id.
__device__ __forceinline__ void wave_lds_sync()
{
    // LDS operations of one wavefront execute in order: only the compiler has to be kept from moving them
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

template <int QK>
__device__ __forceinline__ void stage_chunk(float *lds, const void *qr, int n, float qm, const int32_t *kept, int lo,
                                            int hi, int base, float4 (&qd)[4])
{
    const int lane = lane_id();
    float4 *l4 = (float4 *)lds;
#pragma unroll
    for (int i = 0; i < 4; ++i) l4[i * kWave + lane] = make_float4(0.f, 0.f, 0.f, 0.f);
    wave_lds_sync();
    // All quads of the run lie inside the row (true for every chunk but, when n is not a multiple of four, the last):
    // the same answer for the whole wavefront.  Then the sweep over the run is uniform too: lanes past its end are
    // sent to the last quad of the row (they repeat what its own lane stores), and no load or store sits behind a
    // per-lane branch.
    if (((hi + 3) & ~3) <= n) {
        const int last_quad = (n & ~3) - 4;
        for (int s0 = lo & ~3; s0 < hi; s0 += 4 * kWave) {
            const int s = min(s0 + lane * 4, last_quad);
            const int4 kv = *(const int4 *)(kept + s);
            const float4 qv = load4_full<QK>(qr, s);
            const int ke[4] = {kv.x, kv.y, kv.z, kv.w};
            const float qe[4] = {qv.x, qv.y, qv.z, qv.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const bool mine = s + e >= lo && s + e < hi;
                lds[mine ? ((ke[e] - base) & (kChunk - 1)) : kChunk + lane] = to_weight<QK>(qe[e], qm, 1.f);
            }
        }
    } else {
        for (int s = (lo & ~3) + lane * 4; s < hi; s += 4 * kWave) {
            int4 kv = make_int4(0, 0, 0, 0);
            if (s + 3 < n) {
                kv = *(const int4 *)(kept + s);
            } else {
                if (s + 0 < n) kv.x = kept[s + 0];
                if (s + 1 < n) kv.y = kept[s + 1];
                if (s + 2 < n) kv.z = kept[s + 2];
            }
            const float4 qv = load4<QK>(qr, s, n, QK == RDK_PROB_F32 ? 0.f : -INFINITY);
            const int ke[4] = {kv.x, kv.y, kv.z, kv.w};
            const float qe[4] = {qv.x, qv.y, qv.z, qv.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {   // the weight is formed here, once per kept slot rather than once per target id
                const bool mine = s + e >= lo && s + e < hi;   // others go to a spare word per lane: no branch
                lds[mine ? ((ke[e] - base) & (kChunk - 1)) : kChunk + lane] = to_weight<QK>(qe[e], qm, 1.f);
            }
        }
    }
    wave_lds_sync();
#pragma unroll
    for (int i = 0; i < 4; ++i) qd[i] = l4[i * kWave + lane];
}

// Both passes hide memory latency by occupancy alone: they are held to 64 registers (eight wavefronts per SIMD).
// Eq. 3, first pass.  For the ids of one split of a row:
//   Zq += q^_s, Tn += q^_s p_j, An += N q^_s / (N + p_j)   over kept ids j (slot s),
//   Bs += p_j / (N + p_j)                                    over all ids j.
// Then theta = Tn / Zq and sum_j pt_j = An / Zq + theta * Bs, because
//   pt_j = N q'_j / (N + p_j) + theta p_j / (N + p_j)  with q'_j = q^_s / Zq on kept ids, 0 elsewhere.
// KEEP_P: the target rows are loaded as data that will be used again (the fused call: the second pass is their last
// reader and a batch fits the memory-side cache); otherwise they are streamed like every other single-use row.
template <int PK, int QK, bool KEEP_P>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8))) void taylor_stats_kernel(
    const void *p, int64_t ldp, const void *q, int64_t ldq,
                                                                const int32_t *kept, const int32_t *chunk_lo, int N, int n,
                                                                int splits, LinearWs w)
{
    __shared__ __attribute__((aligned(16))) float qchunk[kWaves][kChunk + kWave];
    const int64_t row = blockIdx.x / splits;
    const int split = blockIdx.x % splits;
    const int nchunks = (N + kChunk - 1) / kChunk;
    const int cpw = (nchunks + splits - 1) / splits;
    const int c_begin = split * cpw, c_end = min(nchunks, c_begin + cpw);
    const void *pr = row_ptr<PK>(p, ldp, row);
    const void *qr = row_ptr<QK>(q, ldq, row);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    float pm = 0.f, pinv = 1.f;
    if (PK != RDK_PROB_F32) {
        const SoftStat rs = merged_row_stat<PK>(w.pstat, w.p_splits, row);
        pm = rs.m;
        pinv = 1.0f / rs.s;
    }
    const float qm = QK == RDK_PROB_F32 ? 0.f : weight_reference(w.qstat[row].m);
    const float pfill = PK == RDK_PROB_F32 ? 0.f : -INFINITY;
    const float fN = (float)N;
    float zq = 0.f, tn = 0.f, an = 0.f, bs = 0.f;
    // the slot run of the next chunk is looked up one iteration ahead, so that no load of a chunk waits for another
    int c = c_begin + wid;
    int lo = 0, hi = 0;
    if (c < c_end) {
        lo = chunk_lo[c];
        hi = chunk_lo[c + 1];
    }
    for (; c < c_end; c += kWaves) {
        const int base = c * kChunk;
        float4 pv[4], qd[4];
        load_chunk<PK, !KEEP_P>(pr, base, N, pfill, pv);
        const int lo_now = lo, hi_now = hi;
        if (c + kWaves < c_end) {
            lo = chunk_lo[c + kWaves];
            hi = chunk_lo[c + kWaves + 1];
        }
        stage_chunk<QK>(qchunk[wid], qr, n, qm, kept, lo_now, hi_now, base, qd);
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float pe[4] = {to_weight<PK>(pv[i].x, pm, pinv), to_weight<PK>(pv[i].y, pm, pinv),
                                 to_weight<PK>(pv[i].z, pm, pinv), to_weight<PK>(pv[i].w, pm, pinv)};
            const float qe[4] = {qd[i].x, qd[i].y, qd[i].z, qd[i].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float r = __builtin_amdgcn_rcpf(fN + pe[e]);
                bs += pe[e] * r;
                const float qh = qe[e];                            // zero on ids that are not kept
                zq += qh;
                tn += qh * pe[e];
                an += qh * r;                                      // times N at the end
            }
        }
    }
    an *= fN;
    zq = wave_sum(zq);
    tn = wave_sum(tn);
    an = wave_sum(an);
    bs = wave_sum(bs);
    __shared__ float sh[kWaves][4];
    if (lane == 0) {
        sh[wid][0] = zq; sh[wid][1] = tn; sh[wid][2] = an; sh[wid][3] = bs;
    }
    __syncthreads();
    if (threadIdx.x < 4) {
        float s = sh[0][threadIdx.x];
        for (int i = 1; i < kWaves; ++i) s += sh[i][threadIdx.x];
        w.tpart[(row * splits + split) * 4 + threadIdx.x] = s;
    }
}

// Eq. 3, first pass for LOGIT target rows without a softmax pass of its own.  The sums of the pass above need the
// normalised p inside 1 / (N + p), i.e. the row maximum and normaliser first.  But p / N <= 1 / N, so with x = p / N
//   N / (N + p) = 1 - x + x^2 - x^3 + O(N^-4),      p / (N + p) = x - x^2 + x^3 + O(N^-4),
// and every term is a power sum of e = exp(z - m) that can be carried under a running maximum m and rescaled when
// the maximum grows (a factor exp(k (m_old - m_new)) for the k-th power).  Per split of a row, relative to the
// split's own maximum m:   S_k = sum_j e_j^k  and  Q_k = sum over kept ids of q^_s e_j^k,  k = 1..3,  and Q_0 = sum q^_s.
// The record (m, S1, S2, S3, Q0, Q1, Q2, Q3) goes to tpart, and (m, S1) also to pstat: the softmax statistics every
// later kernel reads, in the layout of the softmax pass this kernel replaces.  Used for N >= kOnePassMinN, where the
// truncation (a relative N^-3 of the smaller sum) is far below fp32 rounding.
constexpr int kOnePassMinN = 1024;

template <int PK, int QK, bool KEEP_P>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8))) void taylor_stats_onepass_kernel(
    const void *p, int64_t ldp, const void *q, int64_t ldq, const int32_t *kept, const int32_t *chunk_lo, int N, int n,
    int splits, LinearWs w)
{
    static_assert(PK != RDK_PROB_F32, "probabilities need no normaliser: the two-pass kernel serves them");
    __shared__ __attribute__((aligned(16))) float qchunk[kWaves][kChunk + kWave];
    const int64_t row = blockIdx.x / splits;
    const int split = blockIdx.x % splits;
    const int nchunks = (N + kChunk - 1) / kChunk;
    const int cpw = (nchunks + splits - 1) / splits;
    const int c_begin = split * cpw, c_end = min(nchunks, c_begin + cpw);
    const void *pr = row_ptr<PK>(p, ldp, row);
    const void *qr = row_ptr<QK>(q, ldq, row);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    const float qm = QK == RDK_PROB_F32 ? 0.f : weight_reference(w.qstat[row].m);
    float m = -INFINITY;                                         // running maximum, the same in all lanes
    float s1 = 0.f, s2 = 0.f, s3 = 0.f, q0 = 0.f, q1 = 0.f, q2 = 0.f, q3 = 0.f;
    int c = c_begin + wid;
    int lo = 0, hi = 0;
    if (c < c_end) {
        lo = chunk_lo[c];
        hi = chunk_lo[c + 1];
    }
    for (; c < c_end; c += kWaves) {
        const int base = c * kChunk;
        float4 pv[4], qd[4];
        load_chunk<PK, !KEEP_P>(pr, base, N, -INFINITY, pv);
        const int lo_now = lo, hi_now = hi;
        if (c + kWaves < c_end) {
            lo = chunk_lo[c + kWaves];
            hi = chunk_lo[c + kWaves + 1];
        }
        stage_chunk<QK>(qchunk[wid], qr, n, qm, kept, lo_now, hi_now, base, qd);
        float cm = -INFINITY;
#pragma unroll
        for (int i = 0; i < 4; ++i) cm = fmaxf(cm, fmaxf(fmaxf(pv[i].x, pv[i].y), fmaxf(pv[i].z, pv[i].w)));
        cm = wave_max(cm);
        if (cm > m) {                                            // the same decision in all lanes
            const float f = soft_exp(m - cm), f2 = f * f, f3 = f2 * f;   // 0 on the first chunk (m = -inf)
            s1 *= f; s2 *= f2; s3 *= f3;
            q1 *= f; q2 *= f2; q3 *= f3;
            m = cm;
        }
        const float ref = m > -INFINITY ? m : 0.f;               // only masked ids so far: their weights are 0 against any reference
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float pe[4] = {soft_exp(pv[i].x - ref), soft_exp(pv[i].y - ref), soft_exp(pv[i].z - ref), soft_exp(pv[i].w - ref)};
            const float qe[4] = {qd[i].x, qd[i].y, qd[i].z, qd[i].w};
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float e1 = pe[e], e2 = e1 * e1, e3 = e2 * e1;   // exp(-inf) = 0 beyond N
                const float qh = qe[e];                                // zero on ids that are not kept
                s1 += e1; s2 += e2; s3 += e3;
                q0 += qh; q1 += qh * e1; q2 += qh * e2; q3 += qh * e3;
            }
        }
    }
    s1 = wave_sum(s1); s2 = wave_sum(s2); s3 = wave_sum(s3);
    q0 = wave_sum(q0); q1 = wave_sum(q1); q2 = wave_sum(q2); q3 = wave_sum(q3);
    __shared__ float sh[kWaves][8];
    if (lane == 0) {
        sh[wid][0] = m; sh[wid][1] = s1; sh[wid][2] = s2; sh[wid][3] = s3;
        sh[wid][4] = q0; sh[wid][5] = q1; sh[wid][6] = q2; sh[wid][7] = q3;
    }
    __syncthreads();
    if (threadIdx.x == 0) {   // wavefronts without a chunk hold m = -inf and zeros: their factor is 0
        float mm = sh[0][0];
        for (int i = 1; i < kWaves; ++i) mm = fmaxf(mm, sh[i][0]);
        float r[8] = {mm, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int i = 0; i < kWaves; ++i) {
            const float f = sh[i][0] > -INFINITY ? soft_exp(sh[i][0] - mm) : 0.f, f2 = f * f, f3 = f2 * f;
            r[1] += sh[i][1] * f; r[2] += sh[i][2] * f2; r[3] += sh[i][3] * f3;
            r[4] += sh[i][4]; r[5] += sh[i][5] * f; r[6] += sh[i][6] * f2; r[7] += sh[i][7] * f3;
        }
        float *dst = w.tpart + (row * splits + split) * 8;
        *(float4 *)dst = make_float4(r[0], r[1], r[2], r[3]);
        *(float4 *)(dst + 4) = make_float4(r[4], r[5], r[6], r[7]);
        SoftStat st;
        st.m = mm;
        st.s = r[1];
        w.pstat[row * splits + split] = st;
    }
}

// Everything the second pass of Eq. 3 needs about one row; built by all lanes of a wavefront alike.
struct TaylorArgs {
    const void *p, *q;
    int64_t ldp, ldq;
    const int32_t *slot_of, *kept, *chunk_lo;
    int N, n, splits;
    bool onepass;   // the first pass was the one-pass kernel: tpart holds its eight-word records
    LinearWs w;
};

template <int PK, int QK>
struct TaylorRow {
    const void *pr, *qr;
    const int32_t *slot_of;
    int N;
    float pm, pinv, qm, inv_zq, theta, inv_S, fN, nzs, ths;   // nzs = N / (Zq S), ths = theta / S

    // Eq. 3 for one id: qh = unnormalised drafter weight of the id (0 if it is not kept), pe = its target weight
    __device__ __forceinline__ float value(float qh, float pe) const
    {
        return (nzs * qh + ths * pe) * __builtin_amdgcn_rcpf(fN + pe);
    }

    // q' of ids idx .. idx+3 (Eq. 3) in two steps: target values and slots first, then the drafter values
    struct Pending {
        float4 pv;
        int4 sv;
        float qraw[4];
    };
    template <int K>
    __device__ __forceinline__ void stage(Pending &t, int64_t idx) const
    {
        if (K == 0) {
            t.pv = rdk::load4<PK>(pr, idx, N, PK == RDK_PROB_F32 ? 0.f : -INFINITY);
            t.sv = make_int4(-1, -1, -1, -1);
            if (idx + 3 < N) {
                t.sv = *(const int4 *)(slot_of + idx);
            } else {
                if (idx + 0 < N) t.sv.x = slot_of[idx + 0];
                if (idx + 1 < N) t.sv.y = slot_of[idx + 1];
                if (idx + 2 < N) t.sv.z = slot_of[idx + 2];
            }
        } else {
            const int se[4] = {t.sv.x, t.sv.y, t.sv.z, t.sv.w};
#pragma unroll
            for (int e = 0; e < 4; ++e) t.qraw[e] = rdk::load1<QK>(qr, max(se[e], 0));   // unconditional: loads stay batched
        }
    }
    __device__ __forceinline__ float4 result(Pending &t, int64_t idx) const
    {
        const float pe[4] = {to_weight<PK>(t.pv.x, pm, pinv), to_weight<PK>(t.pv.y, pm, pinv), to_weight<PK>(t.pv.z, pm, pinv),
                             to_weight<PK>(t.pv.w, pm, pinv)};
        const int se[4] = {t.sv.x, t.sv.y, t.sv.z, t.sv.w};
        float o[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float qh = se[e] >= 0 ? to_weight<QK>(t.qraw[e], qm, 1.f) : 0.f;
            o[e] = idx + e < N ? value(qh, pe[e]) : 0.f;
        }
        return make_float4(o[0], o[1], o[2], o[3]);
    }
    __device__ __forceinline__ float load1(int j) const
    {
        const float pe = to_weight<PK>(rdk::load1<PK>(pr, j), pm, pinv);
        const int s = slot_of[j];
        const float qh = s >= 0 ? to_weight<QK>(rdk::load1<QK>(qr, max(s, 0)), qm, 1.f) : 0.f;
        return value(qh, pe);
    }
};

template <int PK, int QK>
__device__ __forceinline__ TaylorRow<PK, QK> make_taylor_row(const TaylorArgs &a, int64_t row)
{
    TaylorRow<PK, QK> r;
    r.pr = row_ptr<PK>(a.p, a.ldp, row);
    r.qr = row_ptr<QK>(a.q, a.ldq, row);
    r.slot_of = a.slot_of;
    r.N = a.N;
    r.pm = 0.f;
    r.pinv = 1.f;
    if (PK != RDK_PROB_F32) {
        const SoftStat rs = merged_row_stat<PK>(a.w.pstat, a.w.p_splits, row);
        r.pm = rs.m;
        r.pinv = 1.0f / rs.s;
    }
    r.qm = QK == RDK_PROB_F32 ? 0.f : weight_reference(a.w.qstat[row].m);
    // totals of the first pass, summed in split order by every wavefront alike
    r.fN = (float)a.N;
    float zq, tn, an, bs;
    if (PK != RDK_PROB_F32 && a.onepass) {
        // power sums relative to each split's own maximum, brought to the row maximum; then the series in x = p / N
        float s2 = 0.f, s3 = 0.f, q0 = 0.f, q1 = 0.f, q2 = 0.f, q3 = 0.f;
        for (int i = lane_id(); i < a.splits; i += kWave) {
            const float *rec = a.w.tpart + (row * a.splits + i) * 8;
            const float4 t0 = *(const float4 *)rec, t1 = *(const float4 *)(rec + 4);
            const float f = soft_exp(t0.x - r.pm), f2 = f * f, f3 = f2 * f;   // 0 for a split without ids
            s2 += t0.z * f2; s3 += t0.w * f3;
            q0 += t1.x; q1 += t1.y * f; q2 += t1.z * f2; q3 += t1.w * f3;
        }
        s2 = wave_sum(s2); s3 = wave_sum(s3);
        q0 = wave_sum(q0); q1 = wave_sum(q1); q2 = wave_sum(q2); q3 = wave_sum(q3);
        const float c = r.pinv / r.fN, c2 = c * c, c3 = c2 * c;               // x_j = e_j c
        zq = q0;
        tn = q1 * r.pinv;                                                     // sum q^ p
        an = q0 - q1 * c + q2 * c2 - q3 * c3;                                 // sum q^ N / (N + p)
        bs = 1.0f / r.fN - s2 * c2 + s3 * c3;                                 // sum p / (N + p);  sum x = 1 / N
    } else {
        float a0 = 0.f, a1 = 0.f, a2 = 0.f, a3 = 0.f;
        for (int i = lane_id(); i < a.splits; i += kWave) {
            const float4 t = *(const float4 *)(a.w.tpart + (row * a.splits + i) * 4);
            a0 += t.x; a1 += t.y; a2 += t.z; a3 += t.w;
        }
        zq = wave_sum(a0); tn = wave_sum(a1); an = wave_sum(a2); bs = wave_sum(a3);
    }
    r.inv_zq = inv_mass(zq);                                   // a drafter row without mass gives the zero row
    r.theta = tn * r.inv_zq;
    r.inv_S = inv_mass(an * r.inv_zq + r.theta * bs);
    r.nzs = r.fN * r.inv_zq * r.inv_S;
    r.ths = r.theta * r.inv_S;
    return r;
}

// Eq. 3, second pass: q'_j = ((N q0_j + theta p_j) / (N + p_j)) / sum_j pt_j.  WRITE_Q stores it; FUSE adds the
// verification sums per 1024-id block (sum q', sum max(0, p - q'), sum min(p, q')).  Whether q' is stored (out != NULL)
// is decided at run time, so that the sums do not depend on it by a single bit.
template <int PK, int QK, bool FUSE>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(8))) void taylor_write_kernel(
    TaylorArgs a, float *out, int64_t ldo, float *part_q,
                                                                float *part_r, float *part_a)
{
    __shared__ __attribute__((aligned(16))) float qchunk[kWaves][kChunk + kWave];
    const int64_t row = blockIdx.x / a.splits;
    const int split = blockIdx.x % a.splits;
    const int nchunks = (a.N + kChunk - 1) / kChunk;
    const int cpw = (nchunks + a.splits - 1) / a.splits;
    const int c_begin = split * cpw, c_end = min(nchunks, c_begin + cpw);
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    const float pfill = PK == RDK_PROB_F32 ? 0.f : -INFINITY;
    int c = c_begin + wid;
    int lo = 0, hi = 0;
    if (c < c_end) {   // requested before the row constants below are waited for
        lo = a.chunk_lo[c];
        hi = a.chunk_lo[c + 1];
    }
    const TaylorRow<PK, QK> tr = make_taylor_row<PK, QK>(a, row);
    float *orow = out ? out + row * ldo : nullptr;
    for (; c < c_end; c += kWaves) {
        const int base = c * kChunk;
        float4 pv[4], qd[4];
        load_chunk<PK>(tr.pr, base, a.N, pfill, pv);
        const int lo_now = lo, hi_now = hi;
        if (c + kWaves < c_end) {
            lo = a.chunk_lo[c + kWaves];
            hi = a.chunk_lo[c + kWaves + 1];
        }
        stage_chunk<QK>(qchunk[wid], tr.qr, a.n, tr.qm, a.kept, lo_now, hi_now, base, qd);
        float sq = 0.f, sr = 0.f, sa = 0.f;
        const bool full_o = base + kChunk <= a.N;   // the whole chunk is stored with 16-byte stores
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int64_t idx = (int64_t)base + i * 256 + lane * 4;
            const float pe[4] = {to_weight<PK>(pv[i].x, tr.pm, tr.pinv), to_weight<PK>(pv[i].y, tr.pm, tr.pinv),
                                 to_weight<PK>(pv[i].z, tr.pm, tr.pinv), to_weight<PK>(pv[i].w, tr.pm, tr.pinv)};
            const float qe[4] = {qd[i].x, qd[i].y, qd[i].z, qd[i].w};
            float oe[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float qh = qe[e];                              // zero on ids that are not kept
                oe[e] = tr.value(qh, pe[e]);   // ids beyond N: both weights are zero, and so is the value
            }
            if (orow) {
                if (full_o) {
                    store4(orow + idx, oe[0], oe[1], oe[2], oe[3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (idx + e < a.N) orow[idx + e] = oe[e];
                }
            }
            if (FUSE) {
                sq += (oe[0] + oe[1]) + (oe[2] + oe[3]);
                sr += (fmaxf(pe[0] - oe[0], 0.f) + fmaxf(pe[1] - oe[1], 0.f)) +
                      (fmaxf(pe[2] - oe[2], 0.f) + fmaxf(pe[3] - oe[3], 0.f));
                sa += (fminf(pe[0], oe[0]) + fminf(pe[1], oe[1])) + (fminf(pe[2], oe[2]) + fminf(pe[3], oe[3]));
            }
        }
        if (FUSE) {
            sq = wave_sum(sq);
            sr = wave_sum(sr);
            sa = wave_sum(sa);
            sr += tr.ths * 0.f;   // a row with a NaN or an infinity has a NaN in theta, which the minima and maxima above would hide
            sa += tr.ths * 0.f;
            if (lane == 0) {
                const int64_t o = row * nchunks + c;
                part_q[o] = sq;
                part_r[o] = sr;
                part_a[o] = sa;
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// Eq. 3 and the verification sums in ONE pass over the target row (the fused call when q' is not asked for).  The two-pass
// kernels above read p twice because the row constants (theta, sum of pt) are only known after the whole row has been seen.
// Here one workgroup owns one position and keeps what the second step needs on chip:
//   * an id j that is not kept has q'_j = (theta / S) p_j / (N + p_j), which is below p_j (theta <= 1, S >= 1/2,
//     N >= 2), so its share of the three block sums is a closed form of  P = sum p_j  and  A = sum p_j / (N + p_j)
//     over the not-kept ids of the block: sum q' = sum min(p, q') = (theta / S) A,  sum max(0, p - q') = P - (theta / S) A;
//   * a kept id needs its own p and q^: while the row streams by, the target values of the kept ids are scattered
//     into LDS, chunk by chunk in slot order (4 n bytes: one value per drafter slot; the run of every chunk starts
//     on a 16-byte boundary).
// The softmax of a logit row is not known while it streams, so step A works relative to the largest logit of each chunk:
// e = exp(z - chunk maximum) goes to LDS for the kept ids, and the chunk keeps its maximum and power sums of e, from which the
// sums of p / (N + p) and q^ / (N + p) follow once the scale is known (x = p / N: p / (N + p) = x - x^2 + ..., N / (N + p) = 1 -
// x + x^2 - ...): over the not-kept ids sum e and e^2, over the kept ids the same and sum q^, q^ e, q^ e^2.  Drafter logits are
// taken relative to the largest of the chunk's run in the same way.  (Probability rows: e = p, no maxima.)  The
// form is for N >= 4096, where the next power, (p / N)^2, is 2^-24 of the first at most.
// Step A streams p, guided by the kernel's lane map (L2-resident, shared by all rows), a wavefront per chunk.  The chunk's
// run of drafter values is fetched alongside (one contiguous piece of the drafter row); the wavefront reads its own
// scattered target values back in slot order and adds up the kept ids' sums -- those of the row constants cost no pass of
// their own.  After the barrier the chunks' sums are brought to the row maxima; their totals give the softmax normalisers
// and the row constants.  Step C forms q', max(0, p - q') and min(p, q') on the kept slots.  Its unit of work is a piece of
// at most 64 slots of one chunk (a table of the kernel), dealt out to groups of sixteen lanes in turn, so that vocabularies
// whose kept ids crowd into a few chunks keep every lane busy; the drafter values of the pieces are asked for before the
// constants are known, the sums of a piece take four register-speed lane exchanges, and the pieces of a chunk are added up
// in their order.  HBM traffic: p and q once.
// What bounds it, measured on MI355X: probability rows, HBM while the row streams and then, with one workgroup on a unit,
// about 10 us in the steps after it (N = 128256, n = 32064, 256 rows: 38.6 us a call; N = 151936, n = 16384, 1024 rows: 124.8
// us, 5.5 TB/s); bf16 logit rows, the vector unit in step A (same shape, half the bytes: 96.3 us, 3.6 TB/s; 184 before the loads
// stayed raw in registers -- a conversion next to a load waits for it, so nothing was ever in flight -- and before the
// scatter became a block on the execution mask, eight sums were reduced together, and two workgroups shared a unit; 125.7
// before the masks of the scatter came by scalar loads, the kept ids' sums took a slot a lane, and both maxima of a chunk were
// found together: 395 vector instructions per 1024 ids in all then, 301 now).  The sums of a chunk on the matrix units instead
// (seven products of 32 cycles) were 10 us slower: the products hold the vector unit's issue.
// A reference that the chunks of a wavefront share until a weight leaves its range does without the maxima (17 instructions, 4
// us), but weights of up to 256 are then rounded like any others where the largest of a chunk is exactly 1: alpha of rows whose
// mass lies in a few ids was 5 to 8 % further from 64-bit sums on average.
// q' of Eq. 3 re-computed from the row constants (the finish step needs the two blocks of the crossings).
template <int PK, int QK>
struct QpTaylor {
    static constexpr bool kSpreadRows = false;
    static constexpr int kStages = 2;
    TaylorArgs a;
    typedef TaylorRow<PK, QK> Row;
    __device__ __forceinline__ Row row(int64_t b) const { return make_taylor_row<PK, QK>(a, b); }
};

constexpr int kRowThreads = 1024;
constexpr int kRowWaves = kRowThreads / kWave;
constexpr int kRowHeld = 10;                   // pieces per group whose drafter values are requested ahead of the row constants

// What step A leaves behind per chunk (arrays in LDS).
enum { kRowS1n = 0, kRowS2n, kRowS1k, kRowS2k, kRowQ0, kRowQ1, kRowQ2, kRowMax, kRowQMax, kRowScale, kRowArrays };

struct RowLds {      // offsets in floats into the dynamic LDS block
    int pk, zero, blk, red, items, item_lo, sum_q, sum_r, sum_a, fin, total;
};

// Where the run of chunk c (first slot lo) starts in the LDS array of kept target values: a multiple of four floats, and
// far enough from the run before it (align down costs at most 3, the 4 c make up for it).
__host__ __device__ inline int row_run_start(int lo, int c) { return (lo & ~3) + 4 * c; }

// Upper bound on the number of pieces (the size of the kernel's table): one per chunk and one per 64 slots.
__host__ __device__ inline int row_max_items(int n, int nchunks) { return nchunks + n / 64 + 1; }

// waves: wavefronts of the workgroup.
__host__ __device__ inline RowLds row_lds_layout(int n, int nchunks, int waves)
{
    RowLds L;
    int off = 0;
    // target values of the kept ids: runs of slots, one per chunk, and room for the quads that a piece reads past its end
    // (their values are masked)
    L.pk = off; off += ((n + 3) & ~3) + 4 * nchunks + 4;
    L.zero = off; off += 4;                            // a quad of zeros for the lanes past the end of a piece
    L.blk = off; off += (kRowArrays * nchunks + 3) & ~3;   // what step A leaves behind per chunk
    L.red = off; off += waves * 8;                     // what the wavefronts hand to each other between the steps
    const int mi = (row_max_items(n, nchunks) + 1) & ~1;
    // the kernel's table of pieces; the sums of a piece (max(0, p - q') and min(p, q')) take the place of its entry
    L.items = off; off += 2 * mi;
    L.item_lo = off; off += (nchunks + 1 + 3) & ~3;    // first piece of every chunk
    // per chunk: the three block sums the finish step draws from.  They are formed when the kept target values have
    // served their purpose, and take their place (4 nchunks + 8 floats are there at least).
    L.sum_q = L.pk;
    L.sum_r = L.sum_q + ((nchunks + 3) & ~3);
    L.sum_a = L.sum_r + ((nchunks + 3) & ~3);
    L.fin = off; off += kFinishFloats + 4;             // what the wavefronts of the finish step hand to each other, the uniforms
    L.total = off;
    return L;
}

// 1 / (N + p) for 0 <= p <= 1, N >= 4096 (kRowMaskMinN): the first two terms of the series in p / N are exact to fp32
// rounding (the next term is (p / N)^2 <= 2^-24 of the result) and cost one multiply-add instead of a
// reciprocal, which the vector unit issues at a quarter of the rate.
struct RowRcp {
    float invN, invN2;
    __device__ __forceinline__ float operator()(float p) const { return fmaf(-p, invN2, invN); }
};

// q' of Eq. 3 for the finish of a row inside the one-pass kernels (finish_row_quarters): the drafter values of the kept ids
// of a quarter chunk through the lane map, the row constants nzs and ths, and 1 / (N + p) as the block sums took it.
template <int QK, class RCP>
struct Eq3Quads {
    const uint64_t *lane_map;
    const int32_t *chunk_lo, *slot_of;
    const void *qr;
    float qm, nzs, ths;
    const RCP &rcp;
    int N;
    struct Token {
        uint64_t map;
        int lo, fq;
    };
    __device__ __forceinline__ float value(float qh, float pe) const { return (nzs * qh + ths * pe) * rcp(pe); }
    __device__ __forceinline__ Token begin(int fblk, int fq, int64_t) const
    {
        return Token{lane_map[(int64_t)fblk * kWave + lane_id()], chunk_lo[fblk], fq};
    }
    __device__ __forceinline__ void end(Token &t, int64_t fidx, const float (&pv4)[4], float (&qp4)[4]) const
    {
        const uint32_t kb = (uint32_t)(t.map >> (4 * t.fq)) & 0xFu;
        int sl = t.lo + (int)((t.map >> (16 + 12 * t.fq)) & 0xFFFu);
        float qraw[4];
        bool kept_e[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            kept_e[e] = (kb >> e) & 1u;
            qraw[e] = load1<QK>(qr, kept_e[e] ? sl : 0);   // unconditional: the loads stay batched
            sl += kept_e[e] ? 1 : 0;
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float qh = kept_e[e] ? to_weight<QK>(qraw[e], qm, 1.f) : 0.f;
            qp4[e] = fidx + e < N ? value(qh, pv4[e]) : 0.f;
        }
    }
    __device__ __forceinline__ float at(int dtok, float pd_w) const
    {
        const int sg = slot_of[dtok];
        return value(sg >= 0 ? to_weight<QK>(load1<QK>(qr, sg), qm, 1.f) : 0.f, pd_w);
    }
};

// The finish of a row inside the one-pass kernels, out of the three block sums per chunk in LDS and the position's
// uniforms that the kernel left behind them (all wavefronts of the workgroup have to call it).
// pm, pinv: softmax maximum and 1 / normaliser of a logit target row (0 and 1 for probabilities).
template <int PK, int QK, bool SCAN, class RCP>
__device__ __forceinline__ void row_finish(float *lds, int l_fin, int l_sum_q, int l_sum_r, int l_sum_a,
                                           const FinalizeArgs &fin, int64_t row, int nchunks,
                                           const void *pr, float pm, float pinv, const void *qr, float qm,
                                           const uint64_t *lane_map, const int32_t *chunk_lo, const int32_t *slot_of, int N, float nzs, float ths, const RCP &rcp, int wid, int lane)
{
    const uint32_t *fw = (const uint32_t *)(lds + l_fin + kFinishFloats);
    const uint32_t words[4] = {fw[0], fw[1], fw[2], fw[3]};
    const Eq3Quads<QK, RCP> quads{lane_map, chunk_lo, slot_of, qr, qm, nzs, ths, rcp, N};
    finish_row_quarters<PK, SCAN>(lds + l_fin, lds + l_sum_q, lds + l_sum_r, lds + l_sum_a, nchunks, fin, row, pr, pm, pinv, N,
                            quads, words, wid, lane);
}

// ------------------------------------------------------------------------------------------------
// Eq. 3 of a whole row by one workgroup, q' written: both passes above, and the statistics of logit rows, in one launch.  A
// wavefront holds its chunks (one, or two sixteen chunks apart) of the target row and of the drafter row in id order in registers
// from the first sum to the store.  The kept ids of a quad own consecutive slots, so their drafter values are one 16-byte load at
// the slot that lane_map gives, and three selects a value put them in their places.  The terms are those of taylor_stats_kernel, with
// the row's own normaliser (no series), and the drafter row's mass is not needed at all.  Against 64-bit sums, 12 sets of 64 rows of
// each of 600 to 32000 ids, mean relative error with two passes -> this: q' of probabilities 8.9e-8 -> 8.1e-8, of fp32 logits 3.7e-7 ->
// 3.0e-7, of bf16 logits 2.9e-7 -> 2.4e-7; alpha and residual mass of probabilities 3.6e-8 and 3.3e-8 as before, of logits 6.8e-8 ->
// 5.0e-8 and 6.5e-8 -> 4.8e-8.  Rows of 2500 to 12000 logits without q' in one pass (taylor_row_kernel) -> this: alpha 6.5e-8 -> 5.1e-8,
// residual mass 5.1e-8 -> 4.8e-8.
// What bounds it: the chain of a launch, two dependent reads, one barrier (two for logits) and the stores.
constexpr int kWholeThreads = 1024, kFinishWaves = 8;   // of a workgroup at most; at least where it finishes its row
constexpr int kWholeHeld = 2;                                                       // chunks of a wavefront
constexpr int kWholeMaxN = kWholeHeld * (kWholeThreads / kWave) * kChunk;

// Sum of one value for every wavefront, sixteen at most, in the first lanes.
template <typename T>
__device__ __forceinline__ T waves_sum(T v)
{
    static_assert(kWholeThreads / kWave == 16, "one row of lanes");
    return lane_value(row16_sum(v), 0);
}

// Totals over the workgroup of M values of every wavefront, the same bits in each; at: M * waves floats of LDS, used once.
template <int M>
__device__ __forceinline__ void whole_totals(float (&v)[M], float *at, int wid, int lane, int waves)
{
#pragma unroll
    for (int m = 0; m < M; ++m) v[m] = wave_sum(v[m]);
    if (lane == 0) {
#pragma unroll
        for (int m = 0; m < M; ++m) at[m * waves + wid] = v[m];
    }
    __syncthreads();
#pragma unroll
    for (int m = 0; m < M; ++m) v[m] = waves_sum(lane < waves ? at[m * waves + lane] : 0.f);
}

struct WholeRcp {
    float fN;
    __device__ __forceinline__ float operator()(float pe) const { return __builtin_amdgcn_rcpf(fN + pe); }
};

// FUSE: the sums of every chunk go to LDS and the row is finished (q' is written only if it is asked for).
template <int PK, int QK, bool FUSE>
__global__ __launch_bounds__(kWholeThreads) void taylor_whole_kernel(const void *p, int64_t ldp, const void *q, int64_t ldq,
                                                                     const uint64_t *lane_map, const int32_t *chunk_lo,
                                                                     const int32_t *slot_of, int N, int n, float *out, int64_t ldo,
                                                                     FinalizeArgs fin)
{
    __shared__ float lds[6 * kWholeThreads / kWave];
    __shared__ __attribute__((aligned(16))) float sums[3][FUSE ? kWholeMaxN / kChunk : 1];   // of q', max(0, p - q'), min(p, q') per chunk
    __shared__ __attribute__((aligned(16))) float scratch[FUSE ? kFinishFloats : 1];
    extern __shared__ float4 blocks[];   // FUSE: the two blocks that the draws fall into
    const int64_t row = blockIdx.x;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    const int waves = blockDim.x / kWave, nchunks = (N + kChunk - 1) / kChunk;
    const void *pr = row_ptr<PK>(p, ldp, row);
    const void *qr = row_ptr<QK>(q, ldq, row);
    constexpr float kNoLogit = -INFINITY;
    uint64_t map[kWholeHeld];
    int lo[kWholeHeld], hi[kWholeHeld];
    typename RawQuad<PK>::type praw[kWholeHeld][4];
    typename RawQuad<QK>::type qraw[kWholeHeld][4];
#pragma unroll
    for (int t = 0; t < kWholeHeld; ++t) {
        const int c = wid + t * waves;
        if (c >= nchunks) break;
        map[t] = lane_map[c * kWave + lane];
        lo[t] = chunk_lo[c];
        hi[t] = chunk_lo[c + 1];
    }
#pragma unroll
    for (int t = 0; t < kWholeHeld; ++t) {
        const int c = wid + t * waves;
        if (c >= nchunks) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) praw[t][i] = raw_quad<PK>(pr, c * kChunk + 256 * i + 4 * lane, N);
    }
#pragma unroll
    for (int t = 0; t < kWholeHeld; ++t) {
        if (wid + t * waves >= nchunks) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) qraw[t][i] = raw_quad<QK>(qr, lo[t] + (int)((map[t] >> (16 + 12 * i)) & 0xFFFu), n);
    }
    // the values in id order; ids that are not kept, and those beyond N, have no weight
    float pv[kWholeHeld][4][4], qv[kWholeHeld][4][4];
    float wp = kNoLogit, wq = kNoLogit;   // largest logits of the wavefront's own chunks
#pragma unroll
    for (int t = 0; t < kWholeHeld; ++t) {
        const int c = wid + t * waves;
        if (c >= nchunks) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            row_quad_values<PK>(praw[t][i], c, i, N, PK == RDK_PROB_F32 ? 0.f : kNoLogit, pv[t][i]);
            float v[4];
            RawQuad<QK>::to(qraw[t][i], v);
            if (hi[t] > n - 4) quad_shift(v, lo[t] + (int)((map[t] >> (16 + 12 * i)) & 0xFFFu) - (n - 4));   // the row's last quad
            const uint32_t kb = (uint32_t)map[t] >> (4 * i);
            const bool b0 = kb & 1, b1 = kb & 2, b2 = kb & 4, b3 = kb & 8;
            const float s1 = b0 ? v[1] : v[0], s2 = b0 ? v[2] : v[1], s3 = b0 ? v[3] : v[2];
            const float r2 = b1 ? s2 : s1, r3 = b1 ? s3 : s2;
            const float none = QK == RDK_PROB_F32 ? 0.f : kNoLogit;
            qv[t][i][0] = b0 ? v[0] : none;
            qv[t][i][1] = b1 ? s1 : none;
            qv[t][i][2] = b2 ? r2 : none;
            qv[t][i][3] = b3 ? (b2 ? r3 : r2) : none;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (PK != RDK_PROB_F32) wp = fmaxf(wp, pv[t][i][e]);
                if (QK != RDK_PROB_F32) wq = fmaxf(wq, qv[t][i][e]);
            }
        }
    }
    // Weights of logits are formed against the wavefront's own maximum, and how far that lies below the row's comes in as one factor,
    // finely rounded: a weight is off by its distance from its reference times 6e-8, and there is no maximum of the row to wait for.
    if (PK != RDK_PROB_F32) wp = wave_max(wp);
    if (QK != RDK_PROB_F32) wq = wave_max(wq);
    const float pref = weight_reference(wp), qref = weight_reference(wq);
    float z = 0.f;
#pragma unroll
    for (int t = 0; t < kWholeHeld; ++t) {
        if (wid + t * waves >= nchunks) break;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (PK != RDK_PROB_F32) pv[t][i][e] = soft_exp(pv[t][i][e] - pref);
                if (QK != RDK_PROB_F32) qv[t][i][e] = (map[t] >> (4 * i + e)) & 1 ? soft_exp(qv[t][i][e] - qref) : 0.f;
            }
            if (PK != RDK_PROB_F32) z += (pv[t][i][0] + pv[t][i][1]) + (pv[t][i][2] + pv[t][i][3]);
        }
    }
    float *red = lds;
    float pm = 0.f, pinv = 1.f, pscale = 1.f, prest = 0.f, qm = 0.f, qscale = 1.f;   // of the row; weight of the wavefront -> of the row
    if (PK != RDK_PROB_F32 || QK != RDK_PROB_F32) {
        if (PK != RDK_PROB_F32) z = wave_sum(z);
        if (lane == 0) {
            red[wid] = wp;
            red[waves + wid] = wq;
            red[2 * waves + wid] = z;
        }
        __syncthreads();
        if (PK != RDK_PROB_F32) {
            const float m = lane < waves ? red[lane] : kNoLogit;
            pm = wave_max(m);
            // The errors that all ids share are kept out of the weights: the normaliser is added up in 64 bits, and what its reciprocal and
            // the product with the factor round off comes in as a second, small factor.  Without, the residual mass of 2500 to 12000 logits
            // was 1.1 to 1.3 times as far from 64-bit sums as the one-pass form's, with it 0.84 to 1.01 times; it costs nothing up to 512
            // rows, and 1024 rows of 1001 ids 0.3 us of 16.
            const double zt = waves_sum(lane < waves ? (double)red[2 * waves + lane] * (double)soft_exp_fine(m - pm) : 0.0);
            const float f = soft_exp_fine(wp - pm);
            pinv = 1.0f / (float)zt;
            pscale = f * pinv;
            prest = fmaf(f, pinv, -pscale) - pscale * (float)fma((double)pinv, zt, -1.0);
        }
        if (QK != RDK_PROB_F32) {
            qm = weight_reference(wave_max(lane < waves ? red[waves + lane] : kNoLogit));
            qscale = soft_exp_fine(wq - qm);
        }
        red += 3 * waves;
    }
    const float fN = (float)N;
    float s[3] = {0.f, 0.f, 0.f};   // sum q^ p, sum q^ / (N + p), sum p / (N + p)
#pragma unroll
    for (int t = 0; t < kWholeHeld; ++t) {
        if (wid + t * waves >= nchunks) break;
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                if (PK != RDK_PROB_F32) pv[t][i][e] = fmaf(pv[t][i][e], pscale, pv[t][i][e] * prest);
                const float pe = pv[t][i][e], qh = qv[t][i][e], r = __builtin_amdgcn_rcpf(fN + pe);
                s[0] += qh * pe;
                s[1] += qh * r;
                s[2] += pe * r;
            }
    }
    if (QK != RDK_PROB_F32) {
        s[0] *= qscale;
        s[1] *= qscale;
    }
    whole_totals(s, red, wid, lane, waves);
    // with the drafter row's mass Z, theta = s0 / Z and S = (N s1 + s0 s2) / Z: Z cancels in N / (Z S) and in theta / S
    const float T = fmaf(s[1], fN, s[0] * s[2]);
    const float nzs = T > 0.f ? fN / T : 0.f, ths = T > 0.f ? s[0] / T : s[0] * 0.f;   // a row without mass gives the zero row
    const float nzw = nzs * qscale;
    float *orow = out ? out + row * ldo : nullptr;
#pragma unroll
    for (int t = 0; t < kWholeHeld; ++t) {
        const int c = wid + t * waves;
        if (c >= nchunks) break;
        float sq = 0.f, sr = 0.f, sa = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int id = c * kChunk + 256 * i + 4 * lane;
            float o[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) o[e] = (nzw * qv[t][i][e] + ths * pv[t][i][e]) * __builtin_amdgcn_rcpf(fN + pv[t][i][e]);
            if (FUSE && !orow) {
            } else if ((c + 1) * kChunk <= N) {
                store4(orow + id, o[0], o[1], o[2], o[3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (id + e < N) orow[id + e] = o[e];
            }
            if (FUSE) {
                float r[4], m[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {   // beyond N both weights are zero, and so is q'
                    qv[t][i][e] = o[e];
                    r[e] = fmaxf(pv[t][i][e] - o[e], 0.f);
                    m[e] = fminf(pv[t][i][e], o[e]);
                }
                sq += (o[0] + o[1]) + (o[2] + o[3]);
                sr += (r[0] + r[1]) + (r[2] + r[3]);
                sa += (m[0] + m[1]) + (m[2] + m[3]);
            }
        }
        if (FUSE) {
            sq = wave_sum(sq);
            sr = wave_sum(sr);
            sa = wave_sum(sa);
            if (t == 0) {   // a row with a NaN or an infinity has a NaN in sum q^ p, which the minima and maxima above would hide
                sr += ths * 0.f;
                sa += ths * 0.f;
            }
            if (lane == 0) {
                sums[0][c] = sq;
                sums[1][c] = sr;
                sums[2][c] = sa;
            }
        }
    }
    if (FUSE) {
        uint32_t words[4];
        position_words(fin.d.seed, fin.d.offset + (uint64_t)row, words);
        __syncthreads();
        const WholeRcp rcp{fN};
        const Eq3Quads<QK, WholeRcp> quads{lane_map, chunk_lo, slot_of, qr, qm, nzs, ths, rcp, N};
        // The draws' blocks through LDS rather than read and redistributed again: N = 1024, 64 rows 7.85 -> 7.65 us, bf16 logits 9.25 ->
        // 8.85, N = 4000, 512 rows 10.1 -> 9.85, bf16 12.9 -> 11.85 (verify_row_kernel, which would have to form the weights again, lost
        // 0.2 to 1 us by it).
        const auto held = [&](int b0, int b1) -> const float4 * {
#pragma unroll
            for (int t = 0; t < kWholeHeld; ++t)
#pragma unroll
                for (int b = 0; b < 2; ++b) {
                    const int c = wid + t * waves;
                    if (c >= nchunks || c != (b ? b1 : b0)) continue;
                    hold_block(blocks + b * 512, pv[t], lane);
                    hold_block(blocks + b * 512 + 256, qv[t], lane);
                }
            __syncthreads();
            return blocks;
        };
        finish_row_quarters<PK, true>(scratch, sums[0], sums[1], sums[2], nchunks, fin, row, pr, pm, pinv, N, quads, words, wid, lane, held);
    }
}

// Stands in for the maximum of nothing, where -inf would make the weight of a masked id exp(-inf + inf).  Nothing finite lies
// below it: rows masked with the lowest finite value of their type keep their own maximum, and with it their weights.
constexpr float kLowest = -FLT_MAX;

// The larger of two values, neither of them a NaN that anybody would miss (fmaxf spends an instruction per operand on
// quieting NaNs).
__device__ __forceinline__ float raw_max(float a, float b)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float raw_max3(float a, float b, float c)
{
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
// Largest values of two registers over the 64 lanes, in scalar registers: the halves of the wavefront take one each.  The lane
// exchanges are part of the comparisons (two wait states before each: what it reads through another lane was just written).
__device__ __forceinline__ void wave_max2(float a, float b, float &ma, float &mb)
{
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
    float v = raw_max(__uint_as_float(r.x), __uint_as_float(r.y));
    r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
    v = raw_max(__uint_as_float(r.x), __uint_as_float(r.y));
    asm("s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
        "s_nop 1\n\t"
        "v_max_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf"
        : "+v"(v));
    ma = lane_value(v, 0);
    mb = lane_value(v, 32);
}

// Eight sums over the 64 lanes at once: lane l gets the total of v[bit reversal of l / 8].  Values are put side by side
// as they are halved (17 instructions where eight separate sums take 48).
__device__ __forceinline__ float wave_sum8(const float (&v)[8])
{
    typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
    auto pair32 = [](float a, float b) {
        const u32x2 r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(r.x) + __uint_as_float(r.y);
    };
    auto pair16 = [](float a, float b) {
        const u32x2 r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false, false);
        return __uint_as_float(r.x) + __uint_as_float(r.y);
    };
    float a = pair16(pair32(v[0], v[1]), pair32(v[2], v[3]));
    float b = pair16(pair32(v[4], v[5]), pair32(v[6], v[7]));
    a += dpp_move<0x128>(a);
    b += dpp_move<0x128>(b);
    a = (lane_id() & 8) ? b : a;
    a += dpp_move<0x141>(a);
    a += dpp_move<0xB1>(a);
    a += dpp_move<0x4E>(a);
    return a;
}

// A chunk of a target row, raw, and the raw drafter values of the first kRowAhead rounds of its run of slots [lo, hi): lane l
// the slots lo + l + 64 r.  Quads need the alignment of one element only (that is all that a global load asks for), and no load
// depends on a branch: the quads that cross the end of the row or lie past it are put right where they are used, and what lies
// past the run is left out there.  A chunk past the last one is asked for too (one line per load, never used): the number of
// loads in flight is then the same on every path, and waiting for the oldest waits for no other.
constexpr int kRowAhead = 5;
template <int PK>
struct PowerChunk {
    typename RawQuad<PK>::type p[4];
    uint64_t map;
    uint32_t q[kRowAhead];
    int lo, hi;
};
// Read-only for the kernel: scalar loads.
template <class V>
using ScalarPtr = const __attribute__((address_space(4))) V *;
template <class V>
__device__ __forceinline__ ScalarPtr<V> scalar_ptr(const V *p) { return (ScalarPtr<V>)(uintptr_t)p; }

template <int QK>
__device__ __forceinline__ uint32_t power_q_raw(const void *qr, uint32_t off)
{
    return QK == RDK_LOGIT_BF16 ? (uint32_t)*(const uint16_t *)((const char *)qr + off) : *(const uint32_t *)((const char *)qr + off);
}
template <int QK>
__device__ __forceinline__ float power_q_value(uint32_t raw) { return __uint_as_float(QK == RDK_LOGIT_BF16 ? raw << 16 : raw); }

template <int PK>
__device__ __forceinline__ void power_fetch_p(const void *pr, const uint64_t *lane_map, int c, int N, PowerChunk<PK> &b)
{
    typedef typename RawQuad<PK>::type Raw;
    constexpr uint32_t es = PK == RDK_LOGIT_BF16 ? 2 : 4;
    const uint32_t lane = (uint32_t)lane_id();
    const int at = min(c, (N - 1) / kChunk), p0 = min(at * kChunk, N - 4);
    const char *pb = (const char *)pr + (int64_t)p0 * es;
    uint32_t most = c == at ? (uint32_t)min(N - 4 - p0, kChunk) * es : 0u;
    asm("" : "+s"(most));                                  // one minimum per load, not one and a selection
    b.map = *(const uint64_t *)((const char *)(lane_map + (int64_t)at * kWave) + lane * 8);
#pragma unroll
    for (int i = 0; i < 4; ++i) b.p[i] = __builtin_nontemporal_load((const Raw *)(pb + min((4 * lane + 256 * i) * es, most)));
}
template <int PK, int QK>
__device__ __forceinline__ void power_fetch_q(const void *qr, int c, int lo, int hi, int N, int n, PowerChunk<PK> &b)
{
    constexpr uint32_t qs = QK == RDK_LOGIT_BF16 ? 2 : 4;
    const int q0 = min(lo, n - 1);
    const char *qb = (const char *)qr + (int64_t)q0 * qs;
    uint32_t most = c * kChunk < N ? (uint32_t)(n - 1 - q0) * qs : 0u;
    asm("" : "+s"(most));
#pragma unroll
    for (int r = 0; r < kRowAhead; ++r) b.q[r] = power_q_raw<QK>(qb, min(((uint32_t)lane_id() + kWave * r) * qs, most));
    b.lo = lo;
    b.hi = hi;
}

// Four target values of a lane: each goes to its slot in LDS (byte address `at`, moved on) in the lanes where the id is kept,
// into the sums of the ids that are not kept in the others.  Written on the execution mask: three vector instructions a value
// with the masks in scalar registers (kept[e]: the lanes whose id e of the quad is kept), against four where they are shifted out of
// the lane's map and eight for selecting in the sums and computing the address.
__device__ __forceinline__ void power_place(const uint64_t *kept, uint32_t &at, const float (&ev)[4], float &s1, float &s2)
{
#define RDK_PLACE(e, next)                         \
    "s_mov_b64 exec, %[k" #e "]\n\t"               \
    "ds_write_b32 %[at], %[e" #e "]\n\t" next      \
    "s_not_b64 exec, exec\n\t"                     \
    "v_add_f32 %[s1], %[e" #e "], %[s1]\n\t"       \
    "v_fmac_f32 %[s2], %[e" #e "], %[e" #e "]\n\t"
#define RDK_NEXT "v_add_u32 %[at], 4, %[at]\n\t"
    asm volatile(RDK_PLACE(0, RDK_NEXT) RDK_PLACE(1, RDK_NEXT) RDK_PLACE(2, RDK_NEXT) RDK_PLACE(3, "") "s_mov_b64 exec, -1"
                 : [at] "+v"(at), [s1] "+v"(s1), [s2] "+v"(s2)
                 : [e0] "v"(ev[0]), [e1] "v"(ev[1]), [e2] "v"(ev[2]), [e3] "v"(ev[3]), [k0] "s"(kept[0]), [k1] "s"(kept[1]),
                   [k2] "s"(kept[2]), [k3] "s"(kept[3])
                 : "scc", "memory");
#undef RDK_NEXT
#undef RDK_PLACE
}

// v with the value of one lane replaced.
template <int LANE>
__device__ __forceinline__ void lane_set(float &v, float to)
{
    asm("v_writelane_b32 %0, %1, %2" : "+v"(v) : "s"(__builtin_amdgcn_readfirstlane(__float_as_uint(to))), "n"(LANE));
}

// The target values of a chunk as floats; of a last chunk that does not fill, what lies past the row counts nothing.
template <int PK>
__device__ __forceinline__ void power_values(const PowerChunk<PK> &b, int c, int N, float (&z)[4][4])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) RawQuad<PK>::to(b.p[i], z[i]);
    if (__builtin_expect(N - c * kChunk < kChunk, 0)) {
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int left = N - (c * kChunk + 256 * i + 4 * lane_id());   // ids of the row from the lane's quad on
            quad_shift(z[i], 4 - left);
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (e >= left) z[i][e] = PK == RDK_PROB_F32 ? 0.f : -INFINITY;
        }
    }
}

// The largest logits of a chunk and of its run of drafter values, which its weights are taken relative to: the largest weight of
// a chunk is exactly 1, and how far the chunk lies below the row comes in with soft_exp_fine.
template <int PK, int QK>
__device__ __forceinline__ void power_refs(const PowerChunk<PK> &b, const float (&z)[4][4], const void *qr, float &rp, float &rq)
{
    float zm = kLowest, qm = kLowest;
    if (PK != RDK_PROB_F32) {
        float zn = raw_max3(z[1][3], z[2][0], z[2][1]);
        zm = raw_max3(z[0][0], z[0][1], z[0][2]);
        zm = raw_max3(zm, z[0][3], z[1][0]);
        zn = raw_max3(zn, z[2][2], z[2][3]);
        zm = raw_max3(zm, z[1][1], z[1][2]);
        zn = raw_max3(zn, z[3][0], z[3][1]);
        zm = raw_max3(zm, z[3][2], z[3][3]);
        zm = raw_max3(zm, zn, kLowest);
    }
    if (QK != RDK_PROB_F32) {
        auto take = [&](int r) { qm = lane_id() < b.hi - b.lo - kWave * r ? raw_max(qm, power_q_value<QK>(b.q[r])) : qm; };
        take(0);
        take(1);
        if (b.hi - b.lo > 2 * kWave) {
#pragma unroll
            for (int r = 2; r < kRowAhead; ++r) take(r);
        }
        for (int s = b.lo + kWave * kRowAhead + lane_id(); __builtin_expect(s < b.hi, 0); s += kWave)
            qm = raw_max(qm, power_q_value<QK>(power_q_raw<QK>(qr, (uint32_t)s * (QK == RDK_LOGIT_BF16 ? 2u : 4u))));
    }
    wave_max2(zm, qm, rp, rq);
}

// The power sums of a chunk, per lane (n: ids that are not kept, k: kept ones).
struct PowerSums {
    float s1n, s2n, s1k, s2k, q0, q1, q2;
};

// Forms them, e of the kept ids to LDS.
template <int PK, int QK>
__device__ __forceinline__ void power_sums(const PowerChunk<PK> &b, const float (&z)[4][4], const uint64_t (&kept)[16], int c, const void *qr,
                                           int n, float *pk, float rp, float rq, PowerSums &v)
{
    const int lane = lane_id(), lo = b.lo, hi = b.hi;
    const int run = row_run_start(lo, c);
    const uint32_t first = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float *)pk + 4 * run;
    v = PowerSums{};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        uint32_t at = first + 4 * (uint32_t)((b.map >> (16 + 12 * i)) & 0xFFFu);
        float ev[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) ev[e] = to_weight<PK>(z[i][e], rp, 1.f);   // ids beyond N: zero
        power_place(kept + 4 * i, at, ev, v.s1n, v.s2n);
    }
    // over the kept ids, in slot order, a slot a lane
    auto add = [&](float qe, float ee) {
        const float e2 = ee * ee;
        v.s1k += ee;
        v.s2k += e2;
        v.q0 += qe;
        v.q1 = fmaf(qe, ee, v.q1);
        v.q2 = fmaf(qe, e2, v.q2);
    };
    auto weight = [&](uint32_t raw) { return to_weight<QK>(power_q_value<QK>(raw), rq, 1.f); };
    auto round = [&](int r, uint32_t raw) {
        if (lane < hi - lo - kWave * r) add(weight(raw), pk[run + kWave * r + lane]);
    };
    // two rounds without a branch: selecting costs less than what a wavefront waits at the ends of short blocks (4 of 102 us).
    // What a lane past the run reads may be another run's, or lie behind them all (2 x 64 floats at most, less than the layout
    // holds there), and counts nothing.
#pragma unroll
    for (int r = 0; r < 2; ++r) {
        const bool in = lane < hi - lo - kWave * r;
        const float qe = weight(b.q[r]), ee = pk[run + kWave * r + lane];
        add(in ? qe : 0.f, in ? ee : 0.f);
    }
    if (hi - lo > 2 * kWave) {
#pragma unroll
        for (int r = 2; r < kRowAhead; ++r) round(r, b.q[r]);
    }
    for (int r = kRowAhead; __builtin_expect(lo + kWave * r < hi, 0); r += 4) {
        uint32_t more[4];
#pragma unroll
        for (int j = 0; j < 4; ++j)
            more[j] = power_q_raw<QK>(qr, (uint32_t)min(lo + kWave * (r + j) + lane, n - 1) * (QK == RDK_LOGIT_BF16 ? 2u : 4u));
        // all there before any is used: a round that is left out would leave its load to be waited for with the next chunk's
        asm volatile("s_waitcnt vmcnt(0)" : "+v"(more[0]), "+v"(more[1]), "+v"(more[2]), "+v"(more[3]));
#pragma unroll
        for (int j = 0; j < 4; ++j) round(r + j, more[j]);
    }
}

// Step A for one chunk: statistics to `stat` (arrays of nchunks floats).  lane_stat: which of them the lane writes (-1: none).
template <int PK, int QK>
__device__ __forceinline__ void row_power_chunk(const PowerChunk<PK> &b, int c, int N, const void *qr, int n, float *pk,
                                                const uint64_t *row_masks, float *stat, int nchunks, int lane_stat)
{
    uint64_t kept[16];                                 // asked for first: on their way while the maxima are found
    const ScalarPtr<uint64_t> mk = scalar_ptr(row_masks) + 16 * c;
#pragma unroll
    for (int i = 0; i < 16; ++i) kept[i] = mk[i];
    float z[4][4], rp = 0.f, rq = 0.f;
    power_values<PK>(b, c, N, z);
    if (PK != RDK_PROB_F32 || QK != RDK_PROB_F32) power_refs<PK, QK>(b, z, qr, rp, rq);
    PowerSums v;
    power_sums<PK, QK>(b, z, kept, c, qr, n, pk, rp, rq, v);
    const float all[8] = {v.s1n, v.s2n, v.s1k, v.s2k, v.q0, v.q1, v.q2, 0.f};   // in the order of the enumeration
    float out = wave_sum8(all);
    if (PK != RDK_PROB_F32) lane_set<1>(out, rp);
    if (QK != RDK_PROB_F32) lane_set<2>(out, rq);
    if (lane_stat >= 0) stat[lane_stat * nchunks + c] = out;
}

template <int PK, int QK, int T>
__global__ __launch_bounds__(T) __attribute__((amdgpu_waves_per_eu(4, 4))) void taylor_row_kernel(const void *p, int64_t ldp, const void *q, int64_t ldq,
                                                                       const uint64_t *lane_map, const uint64_t *row_masks,
                                                                       const int32_t *chunk_lo, const int32_t *item_lo, const int2 *row_items,
                                                                       int N, int n, const int32_t *slot_of,
                                                                       FinalizeArgs fin)
{
    constexpr int kW = T / kWave, kG = T / 16;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int nchunks = (N + kChunk - 1) / kChunk;
    const RowLds L = row_lds_layout(n, nchunks, kW);
    float *pk = lds + L.pk, *stat = lds + L.blk;
    int2 *il = (int2 *)(lds + L.items);
    int *ilo = (int *)(lds + L.item_lo);
    float2 *isum = (float2 *)(lds + L.items);          // an entry is read before its sums are written, by the same lanes
    const int64_t row = blockIdx.x;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    const void *pr = row_ptr<PK>(p, ldp, row);
    const void *qr = row_ptr<QK>(q, ldq, row);
    const float fN = (float)N;
    RowRcp rcp;
    rcp.invN = 1.0f / fN;
    rcp.invN2 = rcp.invN * rcp.invN;

    // ---- prologue: the table of pieces, zeros where the kept target values go, and the first two chunks of every wavefront
    // on their way meanwhile.  The table of pieces is asked for before the first chunks: loads come back
    // in the order in which they were issued, and the barrier then waits for the table alone.
    const int max_items = row_max_items(n, nchunks);
    const int nitems = item_lo[nchunks];
    int2 it0 = make_int2(0, 0), it1 = make_int2(0, 0);
    int lo0 = 0;
    if ((int)threadIdx.x < max_items) it0 = row_items[threadIdx.x];
    if ((int)threadIdx.x + T < max_items) it1 = row_items[threadIdx.x + T];
    if ((int)threadIdx.x <= nchunks) lo0 = item_lo[threadIdx.x];
    PowerChunk<PK> b0, b1, b2;
    int c = wid;
    // without a condition: a way round these loads would make the wait for the table one for everything
    const ScalarPtr<int32_t> lo_of = scalar_ptr(chunk_lo);
    const int last = nchunks - 1, ca = min(c, last), cb = min(c + kW, last), cc = min(c + 2 * kW, last);
    const int lo_a = lo_of[ca], hi_a = lo_of[ca + 1], lo_b = lo_of[cb], hi_b = lo_of[cb + 1];
    int next_lo = lo_of[cc], next_hi = lo_of[cc + 1];
    __builtin_amdgcn_sched_barrier(0);                     // the target rows' loads between the scalar loads and what waits for them
    power_fetch_p<PK>(pr, lane_map, c, N, b0);
    power_fetch_p<PK>(pr, lane_map, c + kW, N, b1);
    __builtin_amdgcn_sched_barrier(0);
    power_fetch_q<PK, QK>(qr, c, lo_a, hi_a, N, n, b0);
    power_fetch_q<PK, QK>(qr, c + kW, lo_b, hi_b, N, n, b1);
    if (threadIdx.x == 0) {                                // while the first chunks are on their way: 0.3 us more after step A
        uint32_t words[4];
        position_words(fin.d.seed, fin.d.offset + (uint64_t)row, words);
        uint32_t *fw = (uint32_t *)(lds + L.fin + kFinishFloats);
        fw[0] = words[0]; fw[1] = words[1]; fw[2] = words[2]; fw[3] = words[3];
    }
    {
        float4 *z = (float4 *)pk;
        const int quads = (L.blk - L.pk) / 4;
        for (int i = threadIdx.x; i < quads; i += T) z[i] = make_float4(0.f, 0.f, 0.f, 0.f);
        if ((int)threadIdx.x < max_items) il[threadIdx.x] = it0;
        if ((int)threadIdx.x + T < max_items) il[threadIdx.x + T] = it1;
        for (int k = threadIdx.x + 2 * T; k < max_items; k += T) il[k] = row_items[k];
        if ((int)threadIdx.x <= nchunks) ilo[threadIdx.x] = lo0;
        for (int cc = threadIdx.x + T; cc <= nchunks; cc += T) ilo[cc] = item_lo[cc];
    }
    __syncthreads();

    // ---- step A.  A lane of every eight writes one of the seven sums, the lanes 1 and 2 what else a chunk leaves behind.
    const int lane_sum = (int)(__builtin_bitreverse32((uint32_t)lane >> 3) >> 29);
    const int lane_stat = (lane & 7) == 0 ? (lane_sum < 7 ? lane_sum : -1) : lane == 1 ? kRowMax : lane == 2 ? kRowQMax : -1;
#define RDK_ROW_STEP(CUR, FREE)                                                                               \
    {                                                                                                         \
        power_fetch_q<PK, QK>(qr, c + 2 * kW, next_lo, next_hi, N, n, FREE);                                  \
        power_fetch_p<PK>(pr, lane_map, c + 2 * kW, N, FREE);                                                 \
        const int ahead = min(c + 3 * kW, last);                                                              \
        next_lo = lo_of[ahead];                                                                               \
        next_hi = lo_of[ahead + 1];                                                                           \
        row_power_chunk<PK, QK>(CUR, c, N, qr, n, pk, row_masks, stat, nchunks, lane_stat);                    \
        c += kW;                                                                                              \
    }
    if (nchunks <= 2 * kW) {
        // A short row: all of it is on its way.  What it takes then is mostly the time in which its code is fetched, and one
        // copy of it, without what looks ahead, is enough (12.4 -> 11.9 us a call for 8 rows of 16000 probabilities).
        while (c < nchunks) {
            row_power_chunk<PK, QK>(b0, c, N, qr, n, pk, row_masks, stat, nchunks, lane_stat);
            b0 = b1;
            c += kW;
        }
    }
    while (c < nchunks) {
        RDK_ROW_STEP(b0, b2)
        if (c >= nchunks) break;
        RDK_ROW_STEP(b1, b0)
        if (c >= nchunks) break;
        RDK_ROW_STEP(b2, b1)
    }
#undef RDK_ROW_STEP
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // the compiler does not count the LDS writes of power_place

    // ---- the pieces of step C: drafter values, LDS offsets and chunks of the first rounds, before the barrier
    const int grp = threadIdx.x >> 4, li = threadIdx.x & 15;
    typename RawQuad<QK>::type qh[kRowHeld];
    int pat[kRowHeld], pch[kRowHeld];
    auto piece_of = [&](int k, int &len, int &chunk) {
        const int2 it = il[k];
        len = (int)((uint32_t)it.y >> 24);
        chunk = it.y & 0x3FFFFF;
        return 4 * li < len ? L.pk + it.x - ((it.y >> 22) & 3) + 4 * chunk + 4 * li : L.zero;
    };
    auto hold = [&](int t) {
        const int k = grp + kG * t;
        int len = 0, first = 0;
        pat[t] = L.zero;
        pch[t] = 0;
        if (k < nitems) {
            pat[t] = piece_of(k, len, pch[t]);
            first = il[k].x;
        }
        qh[t] = raw_quad<QK>(qr, first + 4 * li, n);
    };
    // in steps: a short row has few pieces, and code that does nothing for it still has to be fetched
    hold(0);
    if (nitems > kG) {
        hold(1);
        hold(2);
        if (nitems > 3 * kG) {
#pragma unroll
            for (int t = 3; t < kRowHeld; ++t) hold(t);
        }
    }
    __syncthreads();

    // ---- the row maxima (every wavefront for itself), the chunk statistics relative to them, their totals
    float pm = kLowest, qm = kLowest;
    for (int cc = lane; cc < nchunks; cc += kWave) {
        pm = raw_max(pm, stat[kRowMax * nchunks + cc]);
        qm = raw_max(qm, stat[kRowQMax * nchunks + cc]);
    }
    wave_max2(pm, qm, pm, qm);
    if (PK == RDK_PROB_F32) pm = 0.f;
    if (QK == RDK_PROB_F32) qm = 0.f;
    float t5[5] = {0.f, 0.f, 0.f, 0.f, 0.f};   // sum e, e^2 over all ids; sum q^ e^k, k = 0..2
    for (int cc = threadIdx.x; cc < nchunks; cc += T) {
        float *sc = stat + cc;
        const float f = PK == RDK_PROB_F32 ? 1.f : soft_exp_fine(sc[kRowMax * nchunks] - pm), f2 = f * f;   // shared by 1024 ids
        const float fq = QK == RDK_PROB_F32 ? 1.f : soft_exp_fine(sc[kRowQMax * nchunks] - qm);
        const float s1n = sc[kRowS1n * nchunks] * f, s2n = sc[kRowS2n * nchunks] * f2;
        const float s1k = sc[kRowS1k * nchunks] * f, s2k = sc[kRowS2k * nchunks] * f2;
        const float q0 = sc[kRowQ0 * nchunks] * fq, q1 = sc[kRowQ1 * nchunks] * f * fq, q2 = sc[kRowQ2 * nchunks] * f2 * fq;
        sc[kRowS1n * nchunks] = s1n; sc[kRowS2n * nchunks] = s2n;
        sc[kRowS1k * nchunks] = s1k; sc[kRowS2k * nchunks] = s2k;
        sc[kRowQ0 * nchunks] = q0; sc[kRowQ1 * nchunks] = q1; sc[kRowQ2 * nchunks] = q2;
        sc[kRowScale * nchunks] = f;
        t5[0] += s1n + s1k; t5[1] += s2n + s2k;
        t5[2] += q0; t5[3] += q1; t5[4] += q2;
    }
    {
        const float v8[8] = {t5[0], t5[1], t5[2], t5[3], t5[4], 0.f, 0.f, 0.f};
        const float v = wave_sum8(v8);
        if ((lane & 7) == 0) lds[L.red + wid * 8 + lane_sum] = v;
    }
    __syncthreads();
#pragma unroll
    for (int j = 0; j < 5; ++j) t5[j] = 0.f;
    for (int i = 0; i < kW; ++i) {
        const float4 a4 = *(const float4 *)(lds + L.red + i * 8);
        t5[0] += a4.x; t5[1] += a4.y; t5[2] += a4.z; t5[3] += a4.w;
        t5[4] += lds[L.red + i * 8 + 4];
    }
    const float pinv = PK == RDK_PROB_F32 ? 1.f : 1.0f / t5[0];   // the row maximum itself contributes e = 1: never zero
    const float c1 = pinv / fN, c2 = c1 * c1;
    const float zq = t5[2], tn = t5[3] * pinv;
    const float an = t5[2] - t5[3] * c1 + t5[4] * c2;                  // sum q^ N / (N + p)
    const float bs = t5[0] * c1 - t5[1] * c2;                          // sum p / (N + p)
    const float inv_zq = inv_mass(zq);
    const float theta = tn * inv_zq;
    const float inv_S = inv_mass(an * inv_zq + theta * bs);
    const float nzs = fN * inv_zq * inv_S, ths = theta * inv_S;

    // ---- step C
    auto piece_sums = [&](int k, const typename RawQuad<QK>::type raw, int at, int chunk) {
        const float g = stat[kRowScale * nchunks + chunk] * pinv;       // e of this chunk -> p
        const float4 e4 = *(const float4 *)(lds + at);
        float qe[4];
        RawQuad<QK>::to(raw, qe);
        if (k >= nitems - 3) quad_shift(qe, row_items[k].x + 4 * li + 4 - n);   // a quad of the last pieces may cross the end of the row
#pragma unroll
        for (int e = 0; e < 4; ++e) qe[e] = to_weight<QK>(qe[e], qm, 1.f);
        const float pe[4] = {e4.x * g, e4.y * g, e4.z * g, e4.w * g};
        float sr = 0.f, sa = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const float v = (nzs * qe[e] + ths * pe[e]) * rcp(pe[e]);
            const float m = __builtin_amdgcn_fmed3f(pe[e], v, -INFINITY);
            sa += m;
            sr += pe[e] - m;
        }
        sr = row16_sum(sr);
        sa = row16_sum(sa);
        if (li == 0) isum[k] = make_float2(sr, sa);
    };
    auto held_sums = [&](int t) {
        const int k = grp + kG * t;
        if (k < nitems) piece_sums(k, qh[t], pat[t], pch[t]);
    };
    held_sums(0);
    if (nitems > kG) {
        held_sums(1);
        held_sums(2);
        if (nitems > 3 * kG) {
#pragma unroll
            for (int t = 3; t < kRowHeld; ++t) held_sums(t);
        }
    }
    for (int k = grp + kG * kRowHeld; k < nitems; k += kG) {
        int len, chunk;
        const int at = piece_of(k, len, chunk);
        const int first = il[k].x;
        piece_sums(k, raw_quad<QK>(qr, first + 4 * li, n), at, chunk);
    }
    __syncthreads();

    // ---- the block sums of a chunk: its pieces in order, and the closed forms from the chunk's power sums.  The three
    // results take the place of the kept values in LDS (no longer needed), the statistics are read before.
    for (int cc = grp; cc < nchunks; cc += kG) {
        const int k = ilo[cc] + li;
        const float2 f = k < ilo[cc + 1] ? isum[k] : make_float2(0.f, 0.f);
        const float sr = row16_sum(f.x), sa = row16_sum(f.y);
        if (li == 0) {
            const float *sc = stat + cc;
            const float s1n = sc[kRowS1n * nchunks];
            const float a_nk = s1n * c1 - sc[kRowS2n * nchunks] * c2;                   // sum p / (N + p), not-kept ids
            const float a_k = sc[kRowS1k * nchunks] * c1 - sc[kRowS2k * nchunks] * c2;   //                  kept ids
            float aq = sc[kRowQ0 * nchunks] - sc[kRowQ1 * nchunks] * c1 + sc[kRowQ2 * nchunks] * c2;
            aq *= rcp.invN;                                            // sum q^ / (N + p), kept ids
            const float ta = ths * a_nk;                               // sum of q' (= sum of min(p, q')) over the not-kept ids
            lds[L.sum_q + cc] = ths * (a_nk + a_k) + nzs * aq;
            lds[L.sum_a + cc] = ta + sa;
            lds[L.sum_r + cc] = (s1n * pinv - ta) + sr;
        }
    }
    __syncthreads();

    // ---- the finish of the row (draws, accept test), spread over the wavefronts
    row_finish<PK, QK, T == kRowThreads>(lds, L.fin, L.sum_q, L.sum_r, L.sum_a, fin, row, nchunks, pr, pm, pinv, qr, qm, lane_map,
                                         chunk_lo, slot_of, N, nzs, ths, rcp, wid, lane);
}

// Below these batches the two-pass kernels, which split a row over workgroups, fill the chip better.  A longer row takes longer
// in one workgroup, but gives the split form more to do on a full chip too: over 64000 to 250000 ids the two meet at 72 to 88 rows
// of probabilities, and of logits at 4 rows of 64000 ids, 28 of 100000, 36 of 128256 and 38 to 50 of 250000.  Calls, two passes -> one, probabilities: 64 / 72 / 80 / 88 rows of 128256 ids
// 25.7 -> 30.4 / 29.2 -> 30.6 / 30.6 -> 31.0 / 35.5 -> 30.4 us, 64 / 72 / 80 rows of 90000 ids 21.3 -> 24.2 / 22.1 -> 24.5 / 23.1 ->
// 24.7, of 250000 ids 35.3 -> 43.6 / 38.2 -> 44.0 / 41.2 -> 44.6.  bf16 logits, with one more launch in two passes: 24 / 32 / 40 rows
// of 100000 ids 28.1 -> 28.7 / 29.9 -> 29.0 / 30.4 -> 29.0, 32 / 40 / 64 rows of 128256 ids 30.7 -> 33.3 / 34.3 -> 33.1 / 40.6 -> 33.6,
// 32 / 40 rows of 250000 ids 39.2 -> 44.3 / 46.1 -> 44.5 (fp32 logits of 128256 ids, 32 / 40 rows, 33.5 -> 33.9 / 36.3 -> 33.6, of
// 250000 ids, 40 / 48 rows, 47.0 -> 47.9 / 47.8 -> 48.4).
constexpr int kRowMinBatch = 88, kRowMinBatchLogit = 40;
// ... unless logit rows are short: at any batch, one launch against three or four.  bf16 logits, 8 rows of 52000 ids 24.0 -> 20.7, and
// past the line, 4 / 32 rows, 56000 ids 22.8 -> 20.7 / 25.8 -> 21.4, 64000 ids 22.7 -> 22.7 / 25.5 -> 23.1 (fp32 logits: 56000 ids,
// 14000 kept, 22.6 -> 21.7, 20000 kept 24.2 -> 24.5, 64000 ids 22.4 -> 22.9).  (Short rows of probabilities are taylor_whole_kernel's.)
constexpr int kRowShortLogitN = 52 * 1024;

// LDS a workgroup may use (asked until it is told; the same on every device the library is built for).
size_t row_lds_limit()
{
    static std::atomic<size_t> limit{0};
    size_t l = limit.load(std::memory_order_relaxed);
    if (!l) {
        int dev = 0, v = 0;
        if (hipGetDevice(&dev) != hipSuccess ||
            hipDeviceGetAttribute(&v, hipDeviceAttributeMaxSharedMemoryPerBlock, dev) != hipSuccess || v <= 0)
            return 64 * 1024;
        l = (size_t)v;
        limit.store(l, std::memory_order_relaxed);
    }
    return l;
}

// ------------------------------------------------------------------------------------------------
// Identity kernel: q' scattered to the kept ids, zero elsewhere (token-level intersection, Eq. 1).
template <int QK>
__global__ __launch_bounds__(kThreads) void tli_scatter_kernel(const void *q, int64_t ldq, const int32_t *slot_of, int N, int B,
                                                               const SoftStat *qstat, float *out, int64_t ldo)
{
    for (int64_t row = blockIdx.y; row < B; row += gridDim.y) {   // positions beyond the grid's second dimension are looped over
        const void *qr = row_ptr<QK>(q, ldq, row);
        const float qm = QK == RDK_PROB_F32 ? 0.f : weight_reference(qstat[row].m), inv = inv_mass(qstat[row].s);
        for (int64_t j = (int64_t)blockIdx.x * kThreads + threadIdx.x; j < N; j += (int64_t)gridDim.x * kThreads) {
            const int s = slot_of[j];
            out[row * ldo + j] = s >= 0 ? to_weight<QK>(load1<QK>(qr, s), qm, 1.f) * inv : 0.f;
        }
    }
}

// Whether q' of a row is written by one workgroup (taylor_whole_kernel): rows that its wavefronts hold, and, of those with two chunks
// for most wavefronts, from 64 positions on; fewer leave the chip to the form that splits a row.  One call of the redistribution
// alone, two passes -> one launch, probabilities / bf16 logits, us: N = 1001, 64 rows 7.5 -> 4.1; N = 4000, 4 rows 6.6 / 11.6 -> 4.0 / 5.1,
// 256 8.0 / 13.0 -> 4.7 / 5.9; N = 16000, 64 8.4 / 13.2 -> 6.0 / 9.4, 512 23.2 / 29.9 -> 17.2 / 21.4; N = 20003, 4 7.0 / 12.2 -> 5.5 / 9.7, 256
// 16.0 / 23.3 -> 11.1 / 13.5; N = 32000, 4 6.8 / 11.7 -> 7.3 / 13.0 (not taken), 256 22.8 / 29.2 -> 14.6 / 18.6, 1024 76.5 / 70.7 -> 59.8 /
// 60.3.  The fused call that keeps q' takes the same form, for the same bits, and gains less on a full chip, where the finish of a row
// holds its registers: between 4 and 1024 rows of 4097 to 32000 ids it was faster at every size measured but one (513 bf16 rows of
// 32000 ids, +4 %).  Beyond 1024 rows the two meet (redistribution alone / fused with q'): logits at 8192 ids (8192 bf16 rows of 8003
// ids 154 -> 108 / 225 -> 174, 4096 of 12000 102 -> 75 / 145 -> 173), probabilities not below 32768 (4096 of 32000 363 -> 220 / 398 -> 267);
// beyond 2048 rows also at two chunks of ids, below which the finish is most of the call (4096 rows of probabilities, 3001 ids 36 -> 21 /
// 69 -> 55, 1001 20.7 -> 11.0 / 51.5 -> 54.3, 200 16.5 -> 6.1 / 43.2 -> 48.7).
constexpr int kWholeAnyBatchN = 24 * kChunk, kWholeLeastRows = 64;
constexpr int kWholeManyRows = 4 * kComputeUnits, kWholeManyLogitN = 8 * kChunk, kWholeMostRows = 8 * kComputeUnits, kWholeMostLeastN = 2 * kChunk;
bool taylor_in_one(const KernelHandle &h, int32_t B, bool prob)
{
    if (h.N < 4 || h.n < 4) return false;
    if (B <= kWholeManyRows) return h.N <= (B < kWholeLeastRows ? kWholeAnyBatchN : kWholeMaxN);
    return h.N <= (prob ? kWholeMaxN : kWholeManyLogitN) && (B <= kWholeMostRows || h.N >= kWholeMostLeastN);
}

// The same for the fused call without q', beside taylor_row_kernel.  That one reads the tables of a kernel, keeps the kept target
// values in LDS and goes through the kept slots again; this one holds everything in registers and has less to do after its sums, but
// every id carries a drafter value (and the exponential of one), and beyond 8192 ids its wavefronts leave no room for a second
// row on a compute unit.  Fused calls, taylor_row_kernel -> this, probabilities / fp32 logits, us: N = 1001, 64 positions 11.5 / 22.3
// (logits below 1024 ids: four launches) -> 7.5 / 8.8, 1024 18.8 / 26.0 -> 13.7 / 15.9, 4096 70.9 / 61.4 -> 48.5 / 55.6; N = 4096, 8192 133 /
// 148 -> 91 / 112; N = 8003, 4 10.8 / 11.7 -> 7.8 / 9.8, 512 14.1 / 15.7 -> 11.9 / 15.2, 4096 77 / 84 -> 58 / 75 (but logits of 8192 ids with
// 819 kept, 1300 rows +8 %); N = 12000, 16 11.9 / 13.2 -> 9.4 / 12.0, 256 13.3 / 14.6 -> 10.6 / 13.2, 384 16.0 / 18.1 -> 17.3 / 22.5; N = 14003,
// 16 12.2 / 13.4 -> 10.1 / 14.3; N = 20003, 64 13.3 / 14.7 -> 10.9 / 14.9; N = 32003, 4 13.5 / 15.2 -> 12.5 / 17.9, 256 17.6 / 19.6 -> 16.9 /
// 22.6.
constexpr int kWholeLogitN = 12 * kChunk;
bool taylor_finished_in_one(const KernelHandle &h, int32_t B, rdk_input_kind_t p_kind)
{
    if (h.N < 4 || h.n < 4) return false;
    const bool prob = p_kind == RDK_PROB_F32;
    if (B <= kComputeUnits) return h.N <= (prob ? kWholeMaxN : kWholeLogitN);
    return h.N <= (prob || B <= 2 * kComputeUnits ? kFinishWaves : kFinishWaves / 2) * kChunk;
}

// c == nullptr: plain Eq. 3 into `out`.  Otherwise the fused call: verification sums per block, then the finish.
template <int PK, int QK>
rdk_status_t run_taylor(const KernelHandle &h, RowInput p, RowInput q, int32_t B, float *out, int64_t ldo, void *ws,
                        const FusedCall *c, hipStream_t st)
{
    LinearWs w = carve(h, B, ws);
    rdk_status_t rc;
    // the fused call: three block sums per 1024 ids and row, one record per row for the per-sequence scan
    const int nchunks = (h.N + kChunk - 1) / kChunk;
    const size_t per = align_up((size_t)B * nchunks * sizeof(float), 256);
    char *fused_ws = (char *)ws + taylor_workspace_bytes(h, B);
    uint64_t *seq_rec = (uint64_t *)(fused_ws + 3 * per);
    if (out ? taylor_in_one(h, B, PK == RDK_PROB_F32 && QK == RDK_PROB_F32) : taylor_finished_in_one(h, B, p.kind)) {
        // q' has the same bits in the call that only writes it and in the fused one
        FinalizeArgs fa{};
        int waves = nchunks < kWholeThreads / kWave ? nchunks : kWholeThreads / kWave;
        if (c) {
            fa.d = c->d;
            fa.draft_ids = c->draft_ids; fa.accept = c->accept; fa.alpha = c->alpha; fa.resid_mass = c->resid_mass;
            fa.resid_ids = c->resid_ids; fa.n_accepted = c->n_accepted; fa.out_tokens = c->out_tokens;
            // The scan of a sequence by its last row, or, with more than four rows for every compute unit, in a launch of its own: 1024 rows
            // of 4000 probabilities 2.1 us more than without a scan against 2.5 for the launch, 2048 4.5 : 2.5, 6144 11.2 : 2.6.
            if (B <= kWholeManyRows) set_scan(fa, seq_rec);
            if (waves < kFinishWaves) waves = kFinishWaves;
        }
#define RDK_WHOLE_LAUNCH(FUSE, LDS)                                                                                           \
    RDK_TIMED_LAUNCH("taylor_whole_kernel", (taylor_whole_kernel<PK, QK, FUSE>), dim3((unsigned)B), dim3(waves * kWave), LDS, st, \
                     p.ptr, p.ld, q.ptr, q.ld, h.lane_map, h.chunk_lo, h.slot_of, h.N, h.n, out, ldo, fa)
        if (c) {
            static LdsGrant grant;
            rc = grant((const void *)taylor_whole_kernel<PK, QK, true>, kHeldQuads * sizeof(float4));
            if (rc != RDK_OK) return rc;
            RDK_WHOLE_LAUNCH(true, kHeldQuads * sizeof(float4));
        } else {
            RDK_WHOLE_LAUNCH(false, 0);
        }
#undef RDK_WHOLE_LAUNCH
        RDK_LAUNCH_CHECK("taylor_whole_kernel");
        return c ? scan_if_left(fa, st) : RDK_OK;
    }
    {
        // the fused call without q': one pass over the target rows, one workgroup per position, when the kept target
        // values of a row fit the LDS of a compute unit and there are enough positions to fill the chip, or the rows are so
        // short that splitting them saves less than the extra launches cost (from the vocabulary size on at which the series of
        // the chunk sums are exact to fp32 rounding)
        size_t lds_bytes = (size_t)row_lds_layout(h.n, nchunks, kRowWaves).total * sizeof(float);
        const bool fits = h.N >= kRowMaskMinN && h.n >= 4 && lds_bytes <= row_lds_limit();
        const bool pays = PK == RDK_PROB_F32 ? B >= kRowMinBatch : B >= kRowMinBatchLogit || h.N <= kRowShortLogitN;
        if (c && !out && fits && pays) {
            // More rows than compute units: workgroups of half the size, two on a unit where their LDS allows it, so that
            // one streams while the other is at its barriers and its finish.
            bool halves = false;
            if (B > kComputeUnits) {
                const size_t half_bytes = (size_t)row_lds_layout(h.n, nchunks, kRowWaves / 2).total * sizeof(float);
                halves = 2 * align_up(half_bytes, 2048) <= row_lds_limit();
                if (halves) lds_bytes = half_bytes;
            }
            FinalizeArgs fa{};                // the block sums stay in the workgroup's LDS
            fa.d = c->d;
            fa.p = p.ptr; fa.ldp = p.ld;
            fa.pstat = w.pstat; fa.p_splits = w.p_splits;
            fa.nblk = nchunks;
            fa.draft_ids = c->draft_ids; fa.accept = c->accept; fa.alpha = c->alpha; fa.resid_mass = c->resid_mass;
            fa.resid_ids = c->resid_ids; fa.n_accepted = c->n_accepted; fa.out_tokens = c->out_tokens;
            // with more positions than compute units the workgroups take turns, and each would add its round trips to the
            // chain of its unit: the scan is a launch of its own then
            if (B <= kComputeUnits) set_scan(fa, seq_rec);
#define RDK_ROW_LAUNCH(THREADS)                                                                                              \
    {                                                                                                                       \
        static LdsGrant grant;                                                                                              \
        rc = grant((const void *)taylor_row_kernel<PK, QK, THREADS>, row_lds_limit());                                      \
        if (rc != RDK_OK) return rc;                                                                                        \
        RDK_TIMED_LAUNCH("taylor_row_kernel", (taylor_row_kernel<PK, QK, THREADS>), dim3((unsigned)B), dim3(THREADS),       \
                         lds_bytes, st, p.ptr, p.ld, q.ptr, q.ld, h.lane_map, h.row_masks, h.chunk_lo, h.item_lo, h.row_items, \
                         h.N, h.n, h.slot_of, fa);                                                                          \
    }
            if (halves) RDK_ROW_LAUNCH(kRowThreads / 2)
            else RDK_ROW_LAUNCH(kRowThreads)
#undef RDK_ROW_LAUNCH
            RDK_LAUNCH_CHECK("taylor_row_kernel");
            return scan_if_left(fa, st);
        }
    }
    // logit target rows of a large vocabulary: the first pass of Eq. 3 also delivers the softmax statistics
    const bool onepass = PK != RDK_PROB_F32 && h.N >= kOnePassMinN;
    if (PK != RDK_PROB_F32 && !onepass) {
        rc = launch_row_stats<PK>(p, h.N, B, w.p_splits, w.pstat, st);
        if (rc != RDK_OK) return rc;
    }
    if (QK != RDK_PROB_F32) {
        rc = launch_row_stats<QK>(q, h.n, B, 1, w.qstat, st);
        if (rc != RDK_OK) return rc;
    }
    TaylorArgs a;
    a.p = p.ptr; a.q = q.ptr; a.ldp = p.ld; a.ldq = q.ld;
    a.slot_of = h.slot_of; a.kept = h.kept_ids; a.chunk_lo = h.chunk_lo; a.N = h.N; a.n = h.n; a.splits = w.t_splits;
    a.onepass = onepass;
    a.w = w;
    // first pass: one-pass or two-pass statistics; in the fused call (c != NULL) it leaves the target rows cacheable
    const dim3 grid((unsigned)B * w.t_splits);
#define RDK_LAUNCH_STATS(KERNEL)                                                                                         \
    RDK_TIMED_LAUNCH("taylor_stats_kernel", KERNEL, grid, dim3(kThreads), 0, st, p.ptr, p.ld, q.ptr, q.ld, h.kept_ids,  \
                     h.chunk_lo, h.N, h.n, w.t_splits, w)
    bool launched = false;
    if constexpr (PK != RDK_PROB_F32) {
        if (onepass) {
            if (c) RDK_LAUNCH_STATS((taylor_stats_onepass_kernel<PK, QK, true>));
            else RDK_LAUNCH_STATS((taylor_stats_onepass_kernel<PK, QK, false>));
            launched = true;
        }
    }
    if (!launched) {
        if (c) RDK_LAUNCH_STATS((taylor_stats_kernel<PK, QK, true>));
        else RDK_LAUNCH_STATS((taylor_stats_kernel<PK, QK, false>));
    }
#undef RDK_LAUNCH_STATS
    RDK_LAUNCH_CHECK("taylor_stats_kernel");
    if (!c) {
        {
            RDK_TIMED_LAUNCH("taylor_write_kernel", (taylor_write_kernel<PK, QK, false>), grid, dim3(kThreads), 0, st, a,
                             out, ldo, (float *)nullptr, (float *)nullptr, (float *)nullptr);
        }
        RDK_LAUNCH_CHECK("taylor_write_kernel");
        return RDK_OK;
    }
    float *part_q = (float *)fused_ws, *part_r = (float *)(fused_ws + per), *part_a = (float *)(fused_ws + 2 * per);
    {
        RDK_TIMED_LAUNCH("taylor_write_kernel", (taylor_write_kernel<PK, QK, true>), grid, dim3(kThreads), 0, st, a, out,
                         ldo, part_q, part_r, part_a);
    }
    RDK_LAUNCH_CHECK("taylor_write_kernel");
    FinalizeArgs fa{};
    fa.d = c->d;
    fa.p = p.ptr; fa.ldp = p.ld;
    fa.pstat = w.pstat; fa.p_splits = w.p_splits;
    fa.part_q = part_q; fa.part_r = part_r; fa.part_a = part_a;
    fa.nblk = nchunks;
    fa.draft_ids = c->draft_ids; fa.accept = c->accept; fa.alpha = c->alpha; fa.resid_mass = c->resid_mass;
    fa.resid_ids = c->resid_ids; fa.n_accepted = c->n_accepted; fa.out_tokens = c->out_tokens;
    return launch_finalize<PK, 1024, true, QpTaylor<PK, QK>>(fa, QpTaylor<PK, QK>{a}, seq_rec, st);
}

template <int QK>
rdk_status_t run_tli(const KernelHandle &h, RowInput q, int32_t B, float *out, int64_t ldo, void *ws, hipStream_t st)
{
    LinearWs w = carve(h, B, ws);
    rdk_status_t rc = launch_row_stats<QK>(q, h.n, B, 1, w.qstat, st);
    if (rc != RDK_OK) return rc;
    const int bx = (h.N + kThreads * 4 - 1) / (kThreads * 4);
    {
        RDK_TIMED_LAUNCH("tli_scatter_kernel", (tli_scatter_kernel<QK>), dim3(bx, B < 32768 ? B : 32768), dim3(kThreads), 0, st, q.ptr,
                         q.ld, h.slot_of, h.N, B, w.qstat, out, ldo);
    }
    RDK_LAUNCH_CHECK("tli_scatter_kernel");
    return RDK_OK;
}

}  // namespace

size_t taylor_workspace_bytes(const KernelHandle &h, int32_t B)
{
    const int splits = row_splits(B, h.N, kWaves);
    return align_up((size_t)B * splits * sizeof(SoftStat), 256) + align_up((size_t)B * sizeof(SoftStat), 256) +
           align_up((size_t)B * splits * 8 * sizeof(float), 256);
}

size_t taylor_fused_workspace_bytes(const KernelHandle &h, int32_t B)
{
    const int nchunks = (h.N + kChunk - 1) / kChunk;
    return taylor_workspace_bytes(h, B) + 3 * align_up((size_t)B * nchunks * sizeof(float), 256) +
           align_up((size_t)B * 2 * sizeof(uint64_t), 256);
}

rdk_status_t launch_taylor(const KernelHandle &h, RowInput p, RowInput q, int32_t B, float *out, int64_t ldo, void *ws,
                           const FusedCall *c, hipStream_t st)
{
#define RDK_T(PK, QK) \
    if (p.kind == PK && q.kind == QK) return run_taylor<PK, QK>(h, p, q, B, out, ldo, ws, c, st);
    RDK_T(RDK_PROB_F32, RDK_PROB_F32)
    RDK_T(RDK_PROB_F32, RDK_LOGIT_F32)
    RDK_T(RDK_PROB_F32, RDK_LOGIT_BF16)
    RDK_T(RDK_LOGIT_F32, RDK_PROB_F32)
    RDK_T(RDK_LOGIT_F32, RDK_LOGIT_F32)
    RDK_T(RDK_LOGIT_F32, RDK_LOGIT_BF16)
    RDK_T(RDK_LOGIT_BF16, RDK_PROB_F32)
    RDK_T(RDK_LOGIT_BF16, RDK_LOGIT_F32)
    RDK_T(RDK_LOGIT_BF16, RDK_LOGIT_BF16)
#undef RDK_T
    return RDK_ERR_DTYPE;
}

rdk_status_t launch_tli_scatter(const KernelHandle &h, RowInput q, int32_t B, float *out, int64_t ldo, void *ws, hipStream_t st)
{
    switch (q.kind) {
        case RDK_PROB_F32: return run_tli<RDK_PROB_F32>(h, q, B, out, ldo, ws, st);
        case RDK_LOGIT_F32: return run_tli<RDK_LOGIT_F32>(h, q, B, out, ldo, ws, st);
        case RDK_LOGIT_BF16: return run_tli<RDK_LOGIT_BF16>(h, q, B, out, ldo, ws, st);
    }
    return RDK_ERR_DTYPE;
}

}  // namespace rdk
