// Alg. 1, step 2 with the top-k sparse kernel, gathers served out of LDS: the form for small batches and small vocabularies.
//
// A workgroup holds the drafter row of one position in LDS and walks a share of the target ids: the neighbour pairs of a
// pruned id are streamed from L2 (eight lanes per id, 16 bytes per lane: whole 1 KB pieces of the table), each lane gathers
// its two neighbours' values from LDS, and the eight lanes of an id are added up in registers.  The row is read in its own
// layout (no transposed copy), and its normaliser (Eq. 1; row maximum and softmax sum for logits) comes out of the pass that
// fills LDS, so the call needs no launch before this one (one for the softmax statistics of logit target rows that are
// split over workgroups).
//
// What bounds it: the table, read once per position (80 GB/s per compute unit when it does not fit the L2 of an XCD, 137 GB/s
// when it does), where the position-minor form (rdk_sparse.hip) reads it once per 32 positions; below that, the launches and
// the chain of dependent reads of one position.  Where one workgroup holds a whole row it also takes the softmax statistics
// of the target row and finishes the row, so that the call is one launch: N = 1024, n = 256, 16 positions 20.4 -> 8.7 us,
// with bf16 logits 29.5 -> 10.1; N = 4000, k = 16, 8 positions 20.8 -> 11.8; N = 128256, 8 positions over 32 workgroups each
// 34.4 -> 18.1, with bf16 logits 44.9 -> 22.4.
#include "rdk_slab.hpp"

namespace rdk {

namespace {

constexpr int kSlabThreads = 1024;
constexpr int kSlabWaves = kSlabThreads / kWave;
constexpr int kTile = 256;                          // target ids of a wavefront's tile at most
constexpr int kQuads = 9;                           // quads of slots a thread holds while LDS is filled
constexpr size_t kLdsBytes = (size_t)160 * 1024;    // of a compute unit
constexpr int kFinishRegs = 8;                      // block sums a lane keeps in registers in the finish
constexpr int kFinishMaxBlocks = kFinishRegs * kWave;

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x4 __attribute__((ext_vector_type(4)));

// LDS: [0, slots) the drafter weights, then the staged tiles, the reductions, and the block sums of a finished row
__host__ __device__ inline int slab_slots(int n) { return (n + 3) / 4 * 4; }
constexpr int kRedFloats = 6 * kSlabWaves;
inline size_t slab_lds_bytes(int n, int nblk_finish)
{
    return ((size_t)slab_slots(n) + (size_t)kSlabWaves * kTile + kRedFloats + 3 * (size_t)nblk_finish) * sizeof(float);
}

struct SlabArgs {
    const void *q;
    int64_t ldq;
    SparseTables t;
    const int32_t *pruned_ids, *kept_ids;
    int n, B;
    int splits, tiles, tiles_per_split;   // workgroups per row, wavefront tiles per row and per workgroup
    SoftStat *qrow;
    float *out;
    int64_t ldo;
};

__device__ __forceinline__ void wave_lds_sync()
{
    // LDS operations of one wavefront execute in order: only the compiler has to be kept from moving them
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// Number of pruned ids below target id j, the same for the whole wavefront (j may be N or more).  Read through the scalar
// cache: as a vector load its wait would drain the pairs that are on their way.
__device__ __forceinline__ int pruned_below(const int32_t *slot_of, int j, int N, int n)
{
    typedef const __attribute__((address_space(4))) int32_t *scalar_ptr;
    const int s = ((scalar_ptr)(uintptr_t)slot_of)[min(j, N - 1)];
    return j >= N ? N - n : s < 0 ? -s - 1 : j - s;
}

// Maximum / sum over the workgroup, the same bits in every thread; `red`: kSlabWaves floats that nothing else uses meanwhile.
__device__ __forceinline__ float block_max(float v, float *red)
{
    v = wave_max(v);
    if (lane_id() == 0) red[threadIdx.x / kWave] = v;
    __syncthreads();
    float m = red[0];
    for (int i = 1; i < kSlabWaves; ++i) m = fmaxf(m, red[i]);
    return m;
}

__device__ __forceinline__ float block_sum(float v, float *red)
{
    v = wave_sum(v);
    if (lane_id() == 0) red[threadIdx.x / kWave] = v;
    __syncthreads();
    float s = red[0];
    for (int i = 1; i < kSlabWaves; ++i) s += red[i];
    return s;
}

__device__ __forceinline__ float max4(float4 v) { return fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w)); }

// The drafter row on its way to LDS, a quad per thread and round.  bf16 values stay as they lie in memory until all are there (their
// maximum is what the workgroup waits for first, so they are also asked for before the pairs: one sequence of 8 drafts at N =
// 128256 24.4 -> 23.4 us a call; rows of fp32 lost 0.3 us by either).
template <int QK>
struct SlabRow {
    static constexpr bool kPacked = QK == RDK_LOGIT_BF16;
    typedef typename std::conditional<kPacked, uint2, float4>::type Quad;
    Quad quad[kQuads];

    __device__ __forceinline__ void request(const SlabArgs &a, const void *qr)
    {
        const float fill = QK == RDK_PROB_F32 ? 0.f : -INFINITY;
#pragma unroll
        for (int v = 0; v < kQuads; ++v) {
            const int s = slot(v);
            if constexpr (kPacked) {
                if (v * kSlabThreads * 4 >= a.n) continue;           // behind the end of the row: not looked at either
                const uint16_t *r = (const uint16_t *)qr + s;
                constexpr uint32_t kNone = 0xFF80u;                  // -infinity
                quad[v] = make_uint2(kNone | kNone << 16, kNone | kNone << 16);
                if (s + 3 < a.n) quad[v] = make_uint2(((const u32x2_any *)r)->x, ((const u32x2_any *)r)->y);
                else if (s < a.n)
                    quad[v] = make_uint2(r[0] | (s + 1 < a.n ? r[1] : kNone) << 16, (s + 2 < a.n ? r[2] : kNone) | (s + 3 < a.n ? r[3] : kNone) << 16);
            } else {
                quad[v] = make_float4(fill, fill, fill, fill);
                if (s < a.n) quad[v] = load4<QK>(qr, s, a.n, fill);
            }
        }
    }
    static __device__ __forceinline__ int slot(int v) { return (int)(threadIdx.x + v * kSlabThreads) * 4; }
    __device__ __forceinline__ float4 values(int v) const
    {
        if constexpr (kPacked)
            return make_float4(__uint_as_float(quad[v].x << 16), __uint_as_float(quad[v].x & 0xFFFF0000u), __uint_as_float(quad[v].y << 16),
                               __uint_as_float(quad[v].y & 0xFFFF0000u));
        else
            return quad[v];
    }
};

// Fills the slab with the unnormalised drafter weights of the requested row of n slots; qmax = the row maximum (logits), zinv = 1 /
// mass.  The last barrier inside leaves the slab ready.
template <int QK>
__device__ __forceinline__ void slab_fill(int n, const SlabRow<QK> &row, float *slab, float *red, float &qmax, float &zinv)
{
    qmax = 0.f;
    if (QK != RDK_PROB_F32) {
        float m = -INFINITY;
#pragma unroll
        for (int v = 0; v < kQuads; ++v)
            if (!SlabRow<QK>::kPacked || v * kSlabThreads * 4 < n) m = fmaxf(m, max4(row.values(v)));
        qmax = weight_reference(block_max(m, red));
    }
    float z = 0.f;
#pragma unroll
    for (int v = 0; v < kQuads; ++v) {
        const int s = SlabRow<QK>::slot(v);
        if (s < n) {
            const float4 x = row.values(v);
            const float4 w = make_float4(to_weight<QK>(x.x, qmax, 1.f), to_weight<QK>(x.y, qmax, 1.f), to_weight<QK>(x.z, qmax, 1.f),
                                         to_weight<QK>(x.w, qmax, 1.f));
            z += (w.x + w.y) + (w.z + w.w);
            *(float4 *)(slab + s) = w;
        }
    }
    zinv = inv_mass(block_sum(z, red + kSlabWaves));
}

// Softmax maximum and normaliser of a whole logit target row, by the workgroup (the row comes from L2 a second time later).
template <int KIND>
__device__ __forceinline__ SoftStat row_soft_stat(const void *pr, int N, float *red)
{
    float m = -INFINITY;
    for (int j = threadIdx.x * 4; j < N; j += kSlabThreads * 4) m = fmaxf(m, max4(load4<KIND>(pr, j, N, -INFINITY)));
    m = block_max(m, red);
    float s = 0.f;
    for (int j = threadIdx.x * 4; j < N; j += kSlabThreads * 4) {
        const float4 x = load4<KIND>(pr, j, N, -INFINITY);
        s += (soft_exp(x.x - m) + soft_exp(x.y - m)) + (soft_exp(x.z - m) + soft_exp(x.w - m));
    }
    return SoftStat{m, block_sum(s, red + kSlabWaves)};
}

// Sum over the 8 lanes of an aligned group, in every one of them.
__device__ __forceinline__ float oct_total(float v)
{
    v += dpp_move<0xB1>(v);
    v += dpp_move<0x4E>(v);
    v += dpp_move<0x141>(v);
    return v;
}

// The drafter weights as the finish inside this kernel finds them.
struct LdsColumn {
    const float *slab;
    float inv_z;
    __device__ __forceinline__ float operator()(int s) const { return slab[s]; }
};

// FIN: one workgroup holds the whole row and finishes it.  T: target ids of one tile of a wavefront, 256 (four per lane) or 64
// (one per lane: a small vocabulary then reaches all wavefronts).
template <int PK, int QK, bool FIN, int T>
__global__ __launch_bounds__(kSlabThreads) void slab_product_kernel(SlabArgs a, FuseArgs f, FinalizeArgs fin, DraftArgs draft)
{
    constexpr bool FUSE = PK >= 0, SUMS = PK != -1;
    constexpr int PKIND = FUSE ? PK : RDK_PROB_F32;
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    const int N = a.t.N;
    float *slab = lds;
    float *stage = lds + slab_slots(a.n) + wid * kTile;
    float *red = lds + slab_slots(a.n) + kSlabWaves * kTile;
    float *blocks = red + kRedFloats;                        // FIN: three block sums per 64 ids
    const int b = FIN ? blockIdx.x : blockIdx.x / a.splits, split = FIN ? 0 : blockIdx.x % a.splits;
    const int nblk = (N + kSumTile - 1) / kSumTile * (kSumTile / kSubIds);
    const int o = lane & 7, i = lane >> 3;
    const int rounds = a.t.kk / 16;
    const int t_end = min(a.tiles, (split + 1) * a.tiles_per_split);
    const void *pr = FUSE ? row_ptr<PKIND>(f.p, f.ldp, b) : nullptr;
    const float pfill = PKIND == RDK_PROB_F32 ? 0.f : -INFINITY;

    // the tile being worked on: its pruned ids [u_lo, u_hi) (pruned slots), its target values; and the bounds of the next
    int tile = split * a.tiles_per_split + wid, ub = 0, rd = 0;
    int u_lo = 0, u_hi = 0, next_lo = 0, next_hi = 0;
    float4 praw = make_float4(pfill, pfill, pfill, pfill);
    int kept_c = 0;           // the first 64 kept ids of the tile, one per lane: id and diagonal weight
    float kept_w = 0.f;
    i32x4 ev_a[8], ev_b[8];   // zeros: an item without ids is worked on like any other (slot 0, weight 0)
    int c_a = 0, c_b = 0;
#pragma unroll
    for (int g = 0; g < 8; ++g) ev_a[g] = ev_b[g] = i32x4{0, 0, 0, 0};
    // byte offsets of 32 bits (slab_taken bounds the table), one addition and one minimum per load: 64-bit addresses per load
    // took as many vector instructions as everything else
    const uint32_t row_bytes = (uint32_t)a.t.kk * 8u;
    auto request = [&](i32x4 (&ev)[8], int &c, int first, int round, int hi) {
        const uint32_t in_row = (uint32_t)round * 128u + 16u * o;
        const uint32_t at = (uint32_t)(first + i) * row_bytes + in_row, last = (uint32_t)(hi - 1) * row_bytes + in_row;
#pragma unroll
        for (int g = 0; g < 8; ++g)
            ev[g] = *(const i32x4 *)((const char *)a.t.nbr + min(at + (uint32_t)g * 8u * row_bytes, last));
        c = a.pruned_ids[(uint32_t)min(first + 8 * o + i, hi - 1)];
    };
    auto begin_tile = [&](int t, int lo, int hi) {
        u_lo = lo;
        u_hi = hi;
        if (FUSE) {
            if (T == 256) praw = load4<PKIND>(pr, t * T + 4 * lane, N, pfill);
            else praw.x = t * T + lane < N ? load1<PKIND>(pr, t * T + lane) : pfill;
        }
        const int s = min(min(t * T, N) - lo + lane, a.n - 1);
        kept_c = a.kept_ids[s];
        kept_w = a.t.self_w[s];
        next_lo = pruned_below(a.t.slot_of, (t + kSlabWaves) * T, N, a.n);
        next_hi = pruned_below(a.t.slot_of, (t + kSlabWaves) * T + T, N, a.n);
    };
    const void *qr = row_ptr<QK>(a.q, a.ldq, b);
    SlabRow<QK> qraw;
    if (SlabRow<QK>::kPacked) qraw.request(a, qr);
    if (tile < t_end) {
        const int lo = pruned_below(a.t.slot_of, tile * T, N, a.n), hi = pruned_below(a.t.slot_of, tile * T + T, N, a.n);
        begin_tile(tile, lo, hi);
        ub = lo;
        if (lo < hi) request(ev_a, c_a, lo, 0, hi);
    }

    SoftStat pstat{-INFINITY, 0.f};   // this lane's partial of the target row's statistics
    static_assert(kMaxSplits <= kWave, "one partial per lane");
    if (FUSE && PKIND != RDK_PROB_F32 && !FIN && lane < f.p_splits) pstat = f.pstat[(int64_t)b * f.p_splits + lane];
    if (!SlabRow<QK>::kPacked) qraw.request(a, qr);

    float qmax, zinv;
    slab_fill<QK>(a.n, qraw, slab, red, qmax, zinv);
    if (!FIN && split == 0 && threadIdx.x == 0) a.qrow[b] = SoftStat{qmax, zinv};
    float pm = 0.f, pinv = 1.f;
    if (FUSE && PKIND != RDK_PROB_F32) {
        const SoftStat rs = FIN ? row_soft_stat<PKIND>(pr, N, red + 2 * kSlabWaves) : wave_soft_merge(pstat);
        pm = rs.m;
        pinv = 1.0f / rs.s;
        if (!FIN && split == 0 && threadIdx.x == 0) f.pmerged[b] = rs;
    }

    // the staged tile in id order: the kept ids join in, then q' is stored and the sums of the tile's blocks are taken
    auto finish_tile = [&]() {
        const int j0 = tile * T, jl = T == 256 ? j0 + 4 * lane : j0 + lane;
        const int s_lo = min(j0, N) - u_lo, s_hi = min(j0 + T, N) - u_hi;
        if (s_lo + lane < s_hi) stage[kept_c - j0] = kept_w * slab[s_lo + lane];
        for (int s = s_lo + kWave + lane; s < s_hi; s += kWave) stage[a.kept_ids[s] - j0] = a.t.self_w[s] * slab[s];
        wave_lds_sync();
        float qv[4] = {0.f, 0.f, 0.f, 0.f};
        if (T == 256) {
            const float4 sv = *(const float4 *)(stage + 4 * lane);
            qv[0] = jl + 0 < N ? sv.x * zinv : 0.f; qv[1] = jl + 1 < N ? sv.y * zinv : 0.f;
            qv[2] = jl + 2 < N ? sv.z * zinv : 0.f; qv[3] = jl + 3 < N ? sv.w * zinv : 0.f;
        } else {
            qv[0] = jl < N ? stage[lane] * zinv : 0.f;
        }
        wave_lds_sync();   // the next tile is staged over this one
        if (a.out != nullptr) {
            float *dst = a.out + (int64_t)b * a.ldo + jl;
            if (T == 256 && jl + 3 < N) {
                const f32x4_any v = {qv[0], qv[1], qv[2], qv[3]};
                __builtin_nontemporal_store(v, (f32x4_any *)dst);
            } else {
#pragma unroll
                for (int e = 0; e < (T == 256 ? 4 : 1); ++e)
                    if (jl + e < N) dst[e] = qv[e];
            }
        }
        if (SUMS) {
            float sq = 0.f, sr = 0.f, sa = 0.f;
            if (FUSE) {
                const float p4[4] = {praw.x, praw.y, praw.z, praw.w};
#pragma unroll
                for (int e = 0; e < (T == 256 ? 4 : 1); ++e) {
                    const float pe = to_weight<PKIND>(p4[e], pm, pinv);
                    sq += qv[e];
                    sr += fmaxf(pe - qv[e], 0.f);
                    sa += fminf(pe, qv[e]);
                }
            } else {
                sq = ((qv[0] + qv[1]) + qv[2]) + qv[3];   // the order of the fused form: same block sums, same drafts
            }
            sq = T == 256 ? row16_sum(sq) : wave_sum(sq);
            if (FUSE) {
                sr = T == 256 ? row16_sum(sr) : wave_sum(sr);
                sa = T == 256 ? row16_sum(sa) : wave_sum(sa);
            }
            const bool writes = T == 256 ? (lane & 15) == 0 : lane == 0;
            const int at = tile * (T / kSubIds) + (T == 256 ? lane >> 4 : 0);
            if (writes && at < nblk) {
                if (FIN) {
                    blocks[at] = sq;
                    if (FUSE) {
                        blocks[nblk + at] = sr;
                        blocks[2 * nblk + at] = sa;
                    }
                } else {
                    const int64_t g = (int64_t)b * nblk + at;
                    f.part_q[g] = sq;
                    if (FUSE) {
                        f.part_r[g] = sr;
                        f.part_a[g] = sa;
                    }
                }
            }
        }
    };

    // ---- a wavefront's work is a list of items: 16 neighbours (one round) of 64 pruned ids.  lane = 8 i + o takes of id i of
    // each of eight groups of eight ids the neighbours 2 o and 2 o + 1; the pairs of an item are requested while the item
    // before it is worked on.  Lanes past the last pruned id of a tile repeat it.
    float acc[8];
    auto item = [&](const i32x4 (&cur)[8], int cu, i32x4 (&nxt)[8], int &ncu) {
        // the item after this one
        int n_tile = tile, n_ub = ub, n_rd = rd + 1;
        const bool ids_done = n_rd == rounds, tile_done = ids_done && ub + 64 >= u_hi;
        if (ids_done) {
            n_rd = 0;
            n_ub = ub + 64;
        }
        int n_lo = u_lo, n_hi = u_hi;
        if (tile_done) {
            n_tile = tile + kSlabWaves;
            n_lo = next_lo;
            n_hi = next_hi;
            n_ub = n_lo;
        }
        // the gathers of this item first: they wait for its pairs, and with them for everything requested before; only then
        // the pairs of the next item, so that no later wait of this item has to cover them
        float x[8], y[8];
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            x[g] = slab[cur[g].x];
            y[g] = slab[cur[g].z];
        }
        __builtin_amdgcn_sched_barrier(0);
        if (n_tile < t_end && n_ub < n_hi) request(nxt, ncu, n_ub, n_rd, n_hi);
        if (rd == 0) {
#pragma unroll
            for (int g = 0; g < 8; ++g) acc[g] = 0.f;
        }
#pragma unroll
        for (int g = 0; g < 8; ++g) {
            acc[g] = fmaf(__int_as_float(cur[g].y), x[g], acc[g]);
            acc[g] = fmaf(__int_as_float(cur[g].w), y[g], acc[g]);
        }
        if (ids_done) {
            float res = 0.f;                                 // lane (i, o) is left with the product of id i of group o
#pragma unroll
            for (int g = 0; g < 8; ++g) {
                const float t = oct_total(acc[g]);
                if (o == g) res = t;
            }
            if (ub + 8 * o + i < u_hi) stage[cu - tile * T] = res;
        }
        if (tile_done) {
            finish_tile();
            if (n_tile < t_end) begin_tile(n_tile, n_lo, n_hi);
        }
        tile = n_tile;
        ub = n_ub;
        rd = n_rd;
    };
    if (tile < t_end) {
        for (;;) {
            item(ev_a, c_a, ev_b, c_b);
            if (tile >= t_end) break;
            item(ev_b, c_b, ev_a, c_a);
            if (tile >= t_end) break;
        }
    }
    if (FIN && SUMS) {
        __syncthreads();
        WideScratch &sh = *(WideScratch *)red;               // the reductions are over
        const SparseRow<LdsColumn> row{a.t.slot_of, a.t.nbr, a.t.self_w, a.t.kk, N, LdsColumn{slab, zinv}};
        auto setup = [&]() { return FinishSetup<SparseRow<LdsColumn>>{row, pm, pinv}; };
        if (FUSE) finish_row_wide<PKIND, kFinishRegs>(fin, setup, b, pr, blocks, blocks + nblk, blocks + 2 * nblk, sh, wid, lane);
        else if (wid == 0) draft_row<kSubIds, kFinishRegs, 3>(draft, row, b, blocks);
    }
}

struct SlabPlan {
    int tile, splits, tiles, tiles_per_split;
    bool finishes;
};

SlabPlan slab_plan(const KernelHandle &h, int32_t B)
{
    SlabPlan p;
    // Giving a row to several workgroups costs a finish in a launch of its own (about 5 us) and, for logit target rows, one
    // more for their statistics.  One workgroup per row up to 1 MB of table: 0.77 MB (N = 8000, k = 16) takes 16.5 us
    // either way with probabilities, 18.9 us against 22.6 with logits; 1.5 MB 24.5 us against 21.6.
    const int64_t table = (int64_t)(h.N - h.n) * h.kk * 8;
    const int nblk = sparse_blocks(h.N);
    const bool whole = nblk <= kFinishMaxBlocks && slab_lds_bytes(h.n, nblk) <= kLdsBytes;
    int splits = B >= kComputeUnits || (whole && table <= 1000000) ? 1 : kComputeUnits / B;
    p.tile = 256;
    p.tiles = nblk * kSubIds / p.tile;
    const int most = (p.tiles + kSlabWaves - 1) / kSlabWaves;    // every wavefront gets a tile
    if (splits > most) splits = most;
    p.tiles_per_split = (p.tiles + splits - 1) / splits;
    p.splits = (p.tiles + p.tiles_per_split - 1) / p.tiles_per_split;
    if (p.splits == 1 && p.tiles < kSlabWaves) {
        p.tile = 64;
        p.tiles_per_split = p.tiles = nblk;
    }
    p.finishes = p.splits == 1 && whole;
    return p;
}

template <int PK, int QK, bool FIN, int T>
rdk_status_t launch_one(const SlabArgs &a, const FuseArgs &f, const FinalizeArgs &fin, const DraftArgs &draft, hipStream_t st)
{
    static LdsGrant grant;
    const rdk_status_t rc = grant((const void *)slab_product_kernel<PK, QK, FIN, T>, kLdsBytes);
    if (rc != RDK_OK) return rc;
    RDK_TIMED_LAUNCH("sparse_product_kernel", (slab_product_kernel<PK, QK, FIN, T>), dim3((unsigned)a.B * a.splits), dim3(kSlabThreads),
                     slab_lds_bytes(a.n, FIN ? sparse_blocks(a.t.N) : 0), st, a, f, fin, draft);
    RDK_LAUNCH_CHECK("sparse_product_kernel");
    return RDK_OK;
}

template <int QK>
rdk_status_t launch_kind(int kind, const SlabPlan &p, const SlabArgs &a, const FuseArgs &f, const FinalizeArgs &fin, const DraftArgs &draft,
                         hipStream_t st)
{
    // rows that are finished in place exist for both tiles; a row that is split, or only written, has no use for the small one
#define RDK_SLAB(PK)                                                                      \
    case PK:                                                                              \
        if (!p.finishes) return launch_one<PK, QK, false, 256>(a, f, fin, draft, st);     \
        return p.tile == 64 ? launch_one<PK, QK, true, 64>(a, f, fin, draft, st)          \
                            : launch_one<PK, QK, true, 256>(a, f, fin, draft, st);
    switch (kind) {
        case -1:
            return p.tile == 64 ? launch_one<-1, QK, false, 64>(a, f, fin, draft, st) : launch_one<-1, QK, false, 256>(a, f, fin, draft, st);
        RDK_SLAB(-2)
        RDK_SLAB(RDK_PROB_F32)
        RDK_SLAB(RDK_LOGIT_F32)
        RDK_SLAB(RDK_LOGIT_BF16)
    }
#undef RDK_SLAB
    return RDK_ERR_DTYPE;
}

}  // namespace

// The table is read once per position here and once per 32 positions in the position-minor form, which pays with a
// transposition, a finish and (logits) up to two statistics passes in launches of their own.  The line lies at 288 MiB of
// table reads per call.  Kernels with a step table leave this form earlier (rdk_steps.hip), so it parts the two for longer drafter
// rows; fused calls, this -> position-minor, probabilities / bf16 logits, us: N = 128256, n = 32064, 16 / 24 positions (187 / 281
// MiB) 25.9 -> 34.0 / 34.8 -> 35.3 (bf16 32.2 -> 45.1 / 40.1 -> 46.7); N = 60000, n = 24000, 48 / 64 (210 / 281) 29.9 -> 32.9 / 33.0 ->
// 33.3 (bf16 35.3 -> 45.5 / 38.3 -> 46.1); N = 128256, n = 25000, k = 32, 8 / 11 (201 / 277) 27.3 -> 41.7 / 46.7 -> 41.9 (bf16 32.5 ->
// 54.4 / 52.6 -> 55.1).  Below 288 MiB a byte offset into the table fits 32 bits.
bool slab_taken(const KernelHandle &h, int32_t B)
{
    if (h.n > kQuads * 4 * kSlabThreads || slab_lds_bytes(h.n, 0) > kLdsBytes) return false;
    return (int64_t)B * (h.N - h.n) * h.kk * 8 <= (int64_t)288 << 20;
}

bool slab_finishes(const KernelHandle &h, int32_t B) { return slab_plan(h, B).finishes; }

rdk_status_t launch_slab_product(const KernelHandle &h, RowInput q, int32_t B, float *out, int64_t ldo, SoftStat *qrow, int kind,
                                 const FuseArgs &f, const FinalizeArgs &fin, const DraftArgs &draft, hipStream_t st)
{
    const SlabPlan p = slab_plan(h, B);
    SlabArgs a{};
    a.q = q.ptr; a.ldq = q.ld;
    a.t = tables_of(h);
    a.pruned_ids = h.pruned_ids; a.kept_ids = h.kept_ids;
    a.n = h.n; a.B = B;
    a.splits = p.splits; a.tiles = p.tiles; a.tiles_per_split = p.tiles_per_split;
    a.qrow = qrow;
    a.out = out; a.ldo = ldo;
    switch (q.kind) {
        case RDK_PROB_F32: return launch_kind<RDK_PROB_F32>(kind, p, a, f, fin, draft, st);
        case RDK_LOGIT_F32: return launch_kind<RDK_LOGIT_F32>(kind, p, a, f, fin, draft, st);
        case RDK_LOGIT_BF16: return launch_kind<RDK_LOGIT_BF16>(kind, p, a, f, fin, draft, st);
    }
    return RDK_ERR_DTYPE;
}

}  // namespace rdk
