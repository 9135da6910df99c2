// Verification of a batch of positions: Alg. 4 of the paper, steps 2 and 4-10, given the target
// rows p and the redistributed drafter rows q' (both over the N target ids).
//
// Short rows: one launch (verify_row_kernel).  Otherwise two (three when p arrives as logits):
//   [row_softstats]   running (max, sum exp) of the logits, a few partials per row
//   verify_stream     one pass over p and q': per 1024-id block the sums of q', of max(0, p - q')
//                     and of min(p, q')  (Def. 2.1 and the residual of step 8)
//   verify_finalize   per row: totals, Philox uniforms, the two inverse-CDF draws (block located from
//                     the partial sums, then re-read), the accept test, and the per-sequence scan
// The streaming pass is bound by HBM: 8 bytes per (position, id), nothing is written but 12 bytes
// per 1024 ids.
#include <mutex>

#include "rdk_finalize.hpp"

namespace rdk {

namespace {

constexpr int kStreamThreads = 256;
constexpr int kWavesPerBlock = kStreamThreads / kWave;

struct VerifyWs {
    float *part_q, *part_r, *part_a;  // [B, nchunks]
    SoftStat *pstat;                  // [B, stat_splits] (logit input only)
    uint64_t *seq_rec;                // [B, 2] records of the per-sequence scan; NULL where the scratch has no room for them
    int nchunks, stat_splits;
};

__host__ __device__ inline int chunks_of(int64_t N) { return (int)((N + kChunk - 1) / kChunk); }

size_t seq_rec_bytes(const rdk_verify_desc_t &d)
{
    return d.gamma > 0 && d.gamma <= kScanMaxGamma ? align_up((size_t)d.B * 2 * sizeof(uint64_t), 256) : 0;
}

VerifyWs carve(const rdk_verify_desc_t &d, void *ws, size_t ws_bytes)
{
    VerifyWs w;
    w.nchunks = chunks_of(d.N);
    w.stat_splits = row_splits(d.B, d.N, kWavesPerBlock);
    char *p = (char *)ws;
    size_t per = align_up((size_t)d.B * w.nchunks * sizeof(float), 256);
    w.part_q = (float *)p; p += per;
    w.part_r = (float *)p; p += per;
    w.part_a = (float *)p; p += per;
    w.pstat = (SoftStat *)p; p += align_up((size_t)d.B * w.stat_splits * sizeof(SoftStat), 256);
    w.seq_rec = seq_rec_bytes(d) && ws_bytes >= verify_workspace_bytes(d) ? (uint64_t *)p : nullptr;
    return w;
}

// ------------------------------------------------------------------------------------------------
template <int KIND, bool HAS_Q>
__global__ __launch_bounds__(kStreamThreads) void verify_stream_kernel(const void *p, int64_t ldp, const float *q, int64_t ldq,
                                                                       int N, int splits, VerifyWs w)
{
    const int64_t row = blockIdx.x / splits;
    const int split = blockIdx.x % splits;
    const int cpw = (w.nchunks + splits - 1) / splits;
    const int c_begin = split * cpw, c_end = min(w.nchunks, c_begin + cpw);
    const void *pr = row_ptr<KIND>(p, ldp, row);
    const float *qr = HAS_Q ? q + row * ldq : nullptr;
    const int wid = threadIdx.x / kWave, lane = lane_id();
    float m = 0.f, inv = 1.f;
    if (KIND != RDK_PROB_F32) {
        const SoftStat rs = merged_row_stat<KIND>(w.pstat, w.stat_splits, row);
        m = rs.m;
        inv = 1.0f / rs.s;
    }
    const float pfill = KIND == RDK_PROB_F32 ? 0.f : -INFINITY;

    for (int c = c_begin + wid; c < c_end; c += kWavesPerBlock) {
        float4 pv[4], qv[4];
        load_chunk<KIND>(pr, (int64_t)c * kChunk, N, pfill, pv);
        if (HAS_Q) load_chunk<RDK_PROB_F32>(qr, (int64_t)c * kChunk, N, 0.f, qv);
        float sq = 0.f, sr = 0.f, sa = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const float pe[4] = {to_weight<KIND>(pv[i].x, m, inv), to_weight<KIND>(pv[i].y, m, inv),
                                 to_weight<KIND>(pv[i].z, m, inv), to_weight<KIND>(pv[i].w, m, inv)};
            if (HAS_Q) {
                const float qe[4] = {qv[i].x, qv[i].y, qv[i].z, qv[i].w};
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    sq += qe[e];
                    sr += fmaxf(pe[e] - qe[e], 0.f);
                    sa += fminf(pe[e], qe[e]);
                }
            } else {
                sr += (pe[0] + pe[1]) + (pe[2] + pe[3]);
            }
        }
        sr = wave_sum(sr);
        if (HAS_Q) {
            sq = wave_sum(sq);
            sa = wave_sum(sa);
        }
        if (lane == 0) {
            const int64_t o = row * w.nchunks + c;
            w.part_r[o] = sr;
            if (HAS_Q) {
                w.part_q[o] = sq;
                w.part_a[o] = sa;
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------
// The whole verification of a position by one workgroup: softmax statistics (logit rows), block sums in LDS, finish and
// scan, in one launch where the split form takes two (three for logits).  The chunks of 1024 ids are dealt to the wavefronts
// in turn; two chunks of both rows are on their way at a time, asked for before anything else, and a logit row whose chunks
// are all among them (N <= 32768 with sixteen wavefronts) is read once; a longer one is read a second time, out of L2.  Sums
// and draws are those of the split form, bit for bit with probability rows.
// What bounds it: the chain of dependent steps of one position (N = 1000: 7.3 us of GPU time, a launch included); for the
// longest rows the rate at which one compute unit reads (N = 32000, 64 rows: 11.4 us).
constexpr int kRowMaxChunks = 64;   // of the block sums in LDS

template <int KIND>
struct RowPair {
    typename RawQuad<KIND>::type p[4];
    typename RawQuad<RDK_PROB_F32>::type q[4];
};

template <int KIND>
__device__ __forceinline__ void row_fetch(const void *row, int c, int N, typename RawQuad<KIND>::type (&v)[4])
{
#pragma unroll
    for (int i = 0; i < 4; ++i) v[i] = raw_quad<KIND>(row, c * kChunk + 256 * i + 4 * lane_id(), N);
}

template <int KIND>
__device__ __forceinline__ void row_stat_chunk(const typename RawQuad<KIND>::type (&raw)[4], int c, int N, SoftStat &st)
{
    float v[4][4];
    float mx = st.m;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        row_quad_values<KIND>(raw[i], c, i, N, -INFINITY, v[i]);
        mx = fmaxf(mx, fmaxf(fmaxf(v[i][0], v[i][1]), fmaxf(v[i][2], v[i][3])));
    }
    if (mx > -INFINITY) {
        float s = st.s == 0.f ? 0.f : st.s * soft_exp(st.m - mx);
#pragma unroll
        for (int i = 0; i < 4; ++i)
            s += (soft_exp(v[i][0] - mx) + soft_exp(v[i][1] - mx)) + (soft_exp(v[i][2] - mx) + soft_exp(v[i][3] - mx));
        st.m = mx;
        st.s = s;
    }
}

template <int KIND, int T>
__global__ __launch_bounds__(T) void verify_row_kernel(const void *p, int64_t ldp, const float *q, int64_t ldq, int N,
                                                                 int nchunks, FinalizeArgs fin)
{
    constexpr int kRowWaves = T / kWave;
    __shared__ __attribute__((aligned(16))) float sums[3][kRowMaxChunks];   // of q', max(0, p - q'), min(p, q') per chunk
    __shared__ __attribute__((aligned(16))) float scratch[kFinishFloats];
    __shared__ SoftStat sh_stat[kRowWaves];
    const int64_t row = blockIdx.x;
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    const void *pr = row_ptr<KIND>(p, ldp, row);
    const float *qr = q + row * ldq;
    RowPair<KIND> buf[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
        const int c = min(wid + t * kRowWaves, nchunks - 1);
        row_fetch<KIND>(pr, c, N, buf[t].p);
        row_fetch<RDK_PROB_F32>(qr, c, N, buf[t].q);
    }
    uint32_t words[4];
    position_words(fin.d.seed, fin.d.offset + (uint64_t)row, words);
    float pm = 0.f, pinv = 1.f;
    if (KIND != RDK_PROB_F32) {
        SoftStat st{-INFINITY, 0.f};
#pragma unroll
        for (int t = 0; t < 2; ++t)
            if (wid + t * kRowWaves < nchunks) row_stat_chunk<KIND>(buf[t].p, wid + t * kRowWaves, N, st);
        for (int c = wid + 2 * kRowWaves; c < nchunks; c += kRowWaves) {
            typename RawQuad<KIND>::type v[4];
            row_fetch<KIND>(pr, c, N, v);
            row_stat_chunk<KIND>(v, c, N, st);
        }
        st = wave_soft_merge(st);
        if (lane == 0) sh_stat[wid] = st;
        __syncthreads();
        // a lane for every wavefront: one after the other took 1 us of a call (bf16 logits, N = 1024, 64 rows 9.7 -> 8.75 us, N = 20003,
        // 256 rows 14.7 -> 13.3, N = 32000, 64 rows 14.2 -> 13.1)
        st = wave_soft_merge(lane < kRowWaves ? sh_stat[lane] : SoftStat{-INFINITY, 0.f});
        pm = st.m;
        pinv = 1.0f / st.s;
    }
    auto chunk_sums = [&](const RowPair<KIND> &b, int c) {
        float sq = 0.f, sr = 0.f, sa = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            float pe[4], qe[4];
            row_quad_values<KIND>(b.p[i], c, i, N, KIND == RDK_PROB_F32 ? 0.f : -INFINITY, pe);
            row_quad_values<RDK_PROB_F32>(b.q[i], c, i, N, 0.f, qe);
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const float w = to_weight<KIND>(pe[e], pm, pinv);
                sq += qe[e];
                sr += fmaxf(w - qe[e], 0.f);
                sa += fminf(w, qe[e]);
            }
        }
        sr = wave_sum(sr);
        sq = wave_sum(sq);
        sa = wave_sum(sa);
        if (lane == 0) {
            sums[0][c] = sq;
            sums[1][c] = sr;
            sums[2][c] = sa;
        }
    };
    for (int c = wid; c < nchunks; c += 2 * kRowWaves) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            const int cc = c + t * kRowWaves, next = cc + 2 * kRowWaves;
            if (cc >= nchunks) break;
            chunk_sums(buf[t], cc);
            if (next < nchunks) {
                row_fetch<KIND>(pr, next, N, buf[t].p);
                row_fetch<RDK_PROB_F32>(qr, next, N, buf[t].q);
            }
        }
    }
    __syncthreads();
    const QpMemory::Row qrow{qr, N};
    const PolicyQuads<QpMemory::Row, QpMemory::kStages> quads{qrow};
    finish_row_quarters<KIND, true>(scratch, sums[0], sums[1], sums[2], nchunks, fin, row, pr, pm, pinv, N, quads, words, wid, lane);
}

}  // namespace

// Per-sequence scan as a launch of its own (sequences longer than one workgroup's waves).
__global__ void sequence_scan_kernel(int S, int gamma, const int32_t *draft_ids, const uint8_t *accept,
                                     const int32_t *resid_ids, int32_t *n_accepted, int32_t *out_tokens)
{
    const int s = blockIdx.x * blockDim.x + threadIdx.x;
    if (s >= S) return;
    const int64_t b0 = (int64_t)s * gamma;
    // flags are read eight at a time so that the loads of a group are in flight together (one round trip per group
    // instead of one per draft position)
    int j = gamma;
    for (int g0 = 0; g0 < gamma && j == gamma; g0 += 8) {
        uint8_t f[8];
#pragma unroll
        for (int t = 0; t < 8; ++t) f[t] = g0 + t < gamma ? accept[b0 + g0 + t] : (uint8_t)0;
#pragma unroll
        for (int t = 7; t >= 0; --t)
            if (g0 + t < gamma && !f[t]) j = g0 + t;   // the lowest rejected position of the group wins
    }
    if (n_accepted) n_accepted[s] = j;
    if (out_tokens) {
        int32_t *o = out_tokens + (int64_t)s * (gamma + 1);
        const int32_t resid = j < gamma ? resid_ids[b0 + j] : -1;
        for (int i0 = 0; i0 <= gamma; i0 += 8) {
            int32_t d[8];
#pragma unroll
            for (int t = 0; t < 8; ++t) d[t] = i0 + t < j ? draft_ids[b0 + i0 + t] : -1;
#pragma unroll
            for (int t = 0; t < 8; ++t)
                if (i0 + t <= gamma) o[i0 + t] = i0 + t < j ? d[t] : (i0 + t == j && j < gamma) ? resid : -1;
        }
    }
}

namespace {

__global__ void philox_words_kernel(uint64_t seed, uint64_t offset, int count, uint32_t *words)
{
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= count) return;
    uint32_t w[4];
    position_words(seed, offset + (uint64_t)i, w);
    for (int j = 0; j < 4; ++j) words[(int64_t)i * 4 + j] = w[j];
}

// Whether a position is verified by one workgroup in one launch.  The split form spreads a row over the chip, which pays
// for its extra launches where there are few long rows.  Measured in GPU time of a call, split form -> one launch:
//   probabilities   N = 1000:  4 rows 9.2 -> 7.3 us, 512 rows 12.1 -> 9.1;   N = 16000:  64 rows 11.2 -> 10.1, 256 rows 15.4 -> 12.3;
//                   N = 24000: 4 rows 9.4 -> 8.9;   N = 32000: 4 rows 9.1 -> 10.0, 64 rows 11.9 -> 11.4, 512 rows 32.2 -> 30.1;
//                   N = 64000: 96 rows 17.0 -> 20.3, 300 rows 35.5 -> 38.9;   N = 1000, 1024 rows (a second turn of workgroups) 14.5 -> 15.8
//   bf16 logits     N = 1000:  4 rows 14.1 -> 10.7;   N = 4001: 512 rows 22.5 -> 13.9;   N = 24000: 4 rows 14.2 -> 13.3, 1024 rows
//                   49.3 -> 43.8;   N = 32000: 4 rows 13.7 -> 15.4, 64 rows 16.8 -> 15.9;   N = 64000: 96 rows 21.7 -> 22.9,
//                   256 rows 37.6 -> 31.2, 1024 rows 100.2 -> 86.7;   N = 128256: 300 rows 65.1 -> 72.4
template <int KIND>
bool row_in_one(const rdk_verify_desc_t &d)
{
    if (d.N < 4 || (KIND == RDK_PROB_F32 && d.B > 2 * kComputeUnits)) return false;
    const int limit = d.B < 48 ? 24 : KIND == RDK_PROB_F32 || d.B < 128 ? 32 : kRowMaxChunks;
    return d.N <= limit * kChunk;
}

template <int KIND, bool HAS_Q>
rdk_status_t run_verify(const rdk_verify_desc_t &d, RowInput p, const float *q, int64_t ldq, int32_t *draft_ids,
                        uint8_t *accept, float *alpha, float *resid_mass, int32_t *resid_ids, int32_t *n_accepted,
                        int32_t *out_tokens, void *ws, size_t ws_bytes, hipStream_t st)
{
    VerifyWs w = carve(d, ws, ws_bytes);
    FinalizeArgs fa{};
    fa.d = d;
    fa.p = p.ptr; fa.ldp = p.ld;
    fa.pstat = w.pstat; fa.p_splits = w.stat_splits;
    fa.part_q = w.part_q; fa.part_r = w.part_r; fa.part_a = w.part_a;
    fa.nblk = w.nchunks;
    fa.draft_ids = draft_ids; fa.accept = accept; fa.alpha = alpha; fa.resid_mass = resid_mass;
    fa.resid_ids = resid_ids; fa.n_accepted = n_accepted; fa.out_tokens = out_tokens;
    if constexpr (HAS_Q) {
        if (row_in_one<KIND>(d)) {
            set_scan(fa, w.seq_rec);
            // more rows than compute units: workgroups of half the size, two on a unit (512 rows of 1000 ids 14.1 -> 9.1 us)
            if (d.B <= kComputeUnits)
                RDK_TIMED_LAUNCH("verify_stream_kernel", (verify_row_kernel<KIND, 1024>), dim3((unsigned)d.B), dim3(1024), 0, st, p.ptr, p.ld,
                                 q, ldq, d.N, w.nchunks, fa);
            else
                RDK_TIMED_LAUNCH("verify_stream_kernel", (verify_row_kernel<KIND, 512>), dim3((unsigned)d.B), dim3(512), 0, st, p.ptr, p.ld, q,
                                 ldq, d.N, w.nchunks, fa);
            RDK_LAUNCH_CHECK("verify_row_kernel");
            return scan_if_left(fa, st);
        }
    }
    const int splits = row_splits(d.B, d.N, kWavesPerBlock);
    if (KIND != RDK_PROB_F32) {
        rdk_status_t rc = launch_row_stats<KIND>(p, d.N, d.B, w.stat_splits, w.pstat, st);
        if (rc != RDK_OK) return rc;
    }
    {
        RDK_TIMED_LAUNCH("verify_stream_kernel", (verify_stream_kernel<KIND, HAS_Q>), dim3((unsigned)d.B * splits),
                         dim3(kStreamThreads), 0, st, p.ptr, p.ld, q, ldq, d.N, splits, w);
    }
    RDK_LAUNCH_CHECK("verify_stream_kernel");
    QpMemory qp{q, ldq, d.N};
    return launch_finalize<KIND, 1024, HAS_Q, QpMemory>(fa, qp, w.seq_rec, st);
}

// Sums of each 1024-id block of materialised rows (the draft draw from a q' that sits in memory).
__global__ __launch_bounds__(kStreamThreads) void row_block_sums_kernel(const float *q, int64_t ldq, int N, int nchunks, int splits,
                                                                        float *part_q)
{
    const int64_t row = blockIdx.x / splits;
    const int split = blockIdx.x % splits;
    const int cpw = (nchunks + splits - 1) / splits;
    const int c_begin = split * cpw, c_end = min(nchunks, c_begin + cpw);
    const float *qr = q + row * ldq;
    const int wid = threadIdx.x / kWave, lane = lane_id();
    for (int c = c_begin + wid; c < c_end; c += kWavesPerBlock) {
        float4 qv[4];
        load_chunk<RDK_PROB_F32>(qr, (int64_t)c * kChunk, N, 0.f, qv);
        float sq = 0.f;
#pragma unroll
        for (int i = 0; i < 4; ++i) sq += (qv[i].x + qv[i].y) + (qv[i].z + qv[i].w);
        sq = wave_sum(sq);
        if (lane == 0) part_q[row * nchunks + c] = sq;
    }
}

}  // namespace

size_t draft_rows_workspace_bytes(int32_t B, int32_t N) { return align_up((size_t)B * chunks_of(N) * sizeof(float), 256); }

rdk_status_t launch_draft_from_rows(const float *q_prime, int64_t ldq, int32_t B, int32_t N, uint64_t seed, uint64_t offset,
                                    int32_t *draft_ids, float *q_draft, void *ws, hipStream_t st)
{
    const int nchunks = chunks_of(N);
    const int splits = row_splits(B, N, kWavesPerBlock);
    float *part_q = (float *)ws;
    RDK_TIMED_LAUNCH("row_block_sums_kernel", row_block_sums_kernel, dim3((unsigned)B * splits), dim3(kStreamThreads), 0, st,
                     q_prime, ldq, N, nchunks, splits, part_q);
    RDK_LAUNCH_CHECK("row_block_sums_kernel");
    DraftArgs a{B, N, seed, offset, part_q, nchunks, draft_ids, q_draft};
    return launch_draft_finalize<1024, QpMemory>(a, QpMemory{q_prime, ldq, N}, st);
}

size_t verify_sums_bytes(const rdk_verify_desc_t &d)
{
    const int nchunks = chunks_of(d.N);
    const size_t per = align_up((size_t)d.B * nchunks * sizeof(float), 256);
    return 3 * per + align_up((size_t)d.B * row_splits(d.B, d.N, kWavesPerBlock) * sizeof(SoftStat), 256);
}

size_t verify_workspace_bytes(const rdk_verify_desc_t &d) { return verify_sums_bytes(d) + seq_rec_bytes(d); }

rdk_status_t launch_verify(const rdk_verify_desc_t &d, RowInput p, const float *q_prime, int64_t ldq, int32_t *draft_ids,
                           uint8_t *accept, float *alpha, float *resid_mass, int32_t *resid_ids, int32_t *n_accepted,
                           int32_t *out_tokens, void *ws, size_t ws_bytes, hipStream_t st)
{
#define RDK_VERIFY_CASE(K)                                                                                                  \
    case K:                                                                                                                 \
        return q_prime ? run_verify<K, true>(d, p, q_prime, ldq, draft_ids, accept, alpha, resid_mass, resid_ids,           \
                                             n_accepted, out_tokens, ws, ws_bytes, st)                                      \
                       : run_verify<K, false>(d, p, q_prime, ldq, draft_ids, accept, alpha, resid_mass, resid_ids,          \
                                              n_accepted, out_tokens, ws, ws_bytes, st);
    switch (p.kind) {
        RDK_VERIFY_CASE(RDK_PROB_F32)
        RDK_VERIFY_CASE(RDK_LOGIT_F32)
        RDK_VERIFY_CASE(RDK_LOGIT_BF16)
    }
#undef RDK_VERIFY_CASE
    return RDK_ERR_DTYPE;
}

// ---- verification without a caller workspace: the scratch of the two kernels lives in a device array of this
// library, one copy per GPU, held until the process ends.
constexpr size_t kStaticScratchBytes = (size_t)4 << 20;
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

size_t verify_static_scratch_limit() { return kStaticScratchBytes; }

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void *g_scratch_ptr[kMaxDevices];   // device address of `scratch` on each GPU, looked up once per GPU
}  // namespace

rdk_status_t launch_verify_static(const rdk_verify_desc_t &d, RowInput p, const float *q_prime, int64_t ldq, int32_t *draft_ids,
                                  uint8_t *accept, float *alpha, float *resid_mass, int32_t *resid_ids, int32_t *n_accepted,
                                  int32_t *out_tokens, hipStream_t st)
{
    if (verify_sums_bytes(d) > kStaticScratchBytes) return RDK_ERR_WORKSPACE;
    int dev = -1;
    RDK_HIP(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) return RDK_ERR_UNSUPPORTED;
    void *ptr = nullptr;
    {
        std::lock_guard<std::mutex> lock(g_scratch_mutex);
        if (!g_scratch_ptr[dev]) {
            // the array's name is a host-side handle, not a device address: every use below goes through `ptr`
            void *sym = nullptr;
            RDK_HIP(hipGetSymbolAddress(&sym, HIP_SYMBOL(scratch)));
            if (!sym) return RDK_ERR_HIP;
            g_scratch_ptr[dev] = sym;
        }
        ptr = g_scratch_ptr[dev];
    }
    // nothing in the scratch has to start at zero: the streaming pass writes every block sum the finish step reads
    return launch_verify(d, p, q_prime, ldq, draft_ids, accept, alpha, resid_mass, resid_ids, n_accepted, out_tokens, ptr,
                         kStaticScratchBytes, st);
}

rdk_status_t launch_sequence_scan(const rdk_verify_desc_t &d, const int32_t *draft_ids, const uint8_t *accept,
                                  const int32_t *resid_ids, int32_t *n_accepted, int32_t *out_tokens, hipStream_t st)
{
    const int S = d.B / d.gamma;
    {
        RDK_TIMED_LAUNCH("sequence_scan_kernel", sequence_scan_kernel, dim3((S + 63) / 64), dim3(64), 0, st, S, d.gamma,
                         draft_ids, accept, resid_ids, n_accepted, out_tokens);
    }
    RDK_LAUNCH_CHECK("sequence_scan_kernel");
    return RDK_OK;
}

rdk_status_t launch_philox_words(uint64_t seed, uint64_t offset, int32_t count, uint32_t *words, hipStream_t st)
{
    hipLaunchKernelGGL(philox_words_kernel, dim3((count + 255) / 256), dim3(256), 0, st, seed, offset, count, words);
    RDK_LAUNCH_CHECK("philox_words_kernel");
    return RDK_OK;
}

}  // namespace rdk
