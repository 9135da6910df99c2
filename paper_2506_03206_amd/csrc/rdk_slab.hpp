// The top-k sparse product out of LDS (rdk_slab.hip), and what it shares with the position-minor form (rdk_sparse.hip).
#pragma once
#include "rdk_finalize.hpp"

namespace rdk {

constexpr int kSubIds = 64;        // ids per block of verification sums in the sparse forms
constexpr int kSumTile = 256;      // the number of blocks of a row is rounded up to whole tiles of this many ids

inline int sparse_blocks(int32_t N) { return (N + kSumTile - 1) / kSumTile * (kSumTile / kSubIds); }

struct SparseTables {
    const int32_t *slot_of;
    const int2 *nbr;
    const float *self_w;
    int kk, N;
};

inline SparseTables tables_of(const KernelHandle &h) { return SparseTables{h.slot_of, h.nbr, h.self_w, h.kk, h.N}; }

// q' of one position re-computed from the sparse kernel (the finish of a row needs two blocks of 64 ids of it).
template <class Col>
struct SparseRow {
    const int32_t *slot_of;
    const int2 *nbr;
    const float *self_w;
    int kk, N;
    Col col;   // drafter weight of a slot; col.inv_z = 1 / mass of the row
    __device__ __forceinline__ float value(int j) const
    {
        if (j >= N) return 0.f;
        const int s = slot_of[j];
        if (s >= 0) return self_w[s] * col(s) * col.inv_z;
        const int64_t u = -s - 1;
        float acc = 0.f;
        for (int t0 = 0; t0 < kk; t0 += 2) {
            const int4 ev = *(const int4 *)(nbr + u * kk + t0);
            acc += __int_as_float(ev.y) * col(ev.x);
            acc += __int_as_float(ev.w) * col(ev.z);
        }
        return acc * col.inv_z;
    }
    // One id per lane (blocks of 64 ids): the slot, then the first sixteen table entries, then their gathers; a kept
    // id is a row whose entries all point at its own slot, the first with the diagonal weight.
    struct Pending1 {
        int se;
        int ii[16];
        float ww[16], gg[16];
    };
    template <int K>
    __device__ __forceinline__ void stage1(Pending1 &t, int64_t idx) const
    {
        if (K == 0) {
            t.se = idx < N ? slot_of[idx] : 0;   // beyond N: computed, discarded
        } else if (K == 1) {
            const int s = t.se;
            const bool kept = s >= 0;
            const int64_t u = kept ? 0 : -s - 1;
#pragma unroll
            for (int x = 0; x < 16; x += 2) {
                const int4 ev = *(const int4 *)(nbr + u * kk + x);
                t.ii[x] = ev.x; t.ww[x] = __int_as_float(ev.y);
                t.ii[x + 1] = ev.z; t.ww[x + 1] = __int_as_float(ev.w);
            }
            const float sw = self_w[max(s, 0)];
            if (kept) {
#pragma unroll
                for (int x = 0; x < 16; ++x) {
                    t.ii[x] = s;
                    t.ww[x] = x == 0 ? sw : 0.f;
                }
            }
        } else {
#pragma unroll
            for (int x = 0; x < 16; ++x) t.gg[x] = col(t.ii[x]);
        }
    }
    __device__ __forceinline__ float result1(Pending1 &t, int64_t idx) const
    {
        float acc = 0.f;
#pragma unroll
        for (int x = 0; x < 16; ++x) acc += t.ww[x] * t.gg[x]; 
        const bool kept = t.se >= 0;
        const int64_t u = kept ? 0 : -t.se - 1;
        for (int x0 = 16; x0 < kk; x0 += 16) {
#pragma unroll
            for (int x = 0; x < 16; x += 2) {
                const int4 ev = *(const int4 *)(nbr + u * kk + x0 + x);
                t.ii[x] = kept ? t.se : ev.x; t.ww[x] = kept ? 0.f : __int_as_float(ev.y);
                t.ii[x + 1] = kept ? t.se : ev.z; t.ww[x + 1] = kept ? 0.f : __int_as_float(ev.w);
            }
#pragma unroll
            for (int x = 0; x < 16; ++x) t.gg[x] = col(t.ii[x]);
#pragma unroll
            for (int x = 0; x < 16; ++x) acc += t.ww[x] * t.gg[x];
        }
        return idx < N ? acc * col.inv_z : 0.f;
    }
    __device__ __forceinline__ float load1(int j) const { return value(j); }
};

template <class Column>
struct QpSparse {
    static constexpr bool kSpreadRows = true;
    static constexpr int kStages = 3;
    SparseTables a;
    Column col;
    typedef SparseRow<typename Column::Row> Row;
    __device__ __forceinline__ Row row(int64_t b) const { return Row{a.slot_of, a.nbr, a.self_w, a.kk, a.N, col.row(b)}; }
};

// What the fused form adds to the product: the target rows, and where the per-block sums go.
struct FuseArgs {
    const void *p;
    int64_t ldp;
    const SoftStat *pstat;             // softmax statistics of logit target rows, p_splits partials per row
    int p_splits;
    SoftStat *pmerged;                 // [B]: the merged pair of each row, written by the product out of LDS
    float *part_q, *part_r, *part_a;   // [B, sparse_blocks(N)]: one entry per 64-id block
};

// The product out of LDS (rdk_slab.hip): whether it is taken for a batch of B positions, and whether it finishes the rows
// itself (draws, accept test, per-sequence scan) because one workgroup holds all of a row.
bool slab_taken(const KernelHandle &h, int32_t B);
bool slab_finishes(const KernelHandle &h, int32_t B);

// kind: what else the product does.  -1: nothing (out is required); -2: sums of q' per block (the finish: the draft draw
// `draft`); an input kind: fused with the verification sums against target rows of that kind (the finish: `fin`).
// qrow [B]: receives maximum (logits) and 1 / mass of the drafter rows.  out: q' [B, ldo], or NULL.
rdk_status_t launch_slab_product(const KernelHandle &h, RowInput q, int32_t B, float *out, int64_t ldo, SoftStat *qrow, int kind,
                                 const FuseArgs &f, const FinalizeArgs &fin, const DraftArgs &draft, hipStream_t st);

}  // namespace rdk
