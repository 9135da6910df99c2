// Alg. 1, step 2 with the top-k sparse kernel, P positions at a time, gathers served out of LDS: the form for larger batches of
// drafter rows of up to 20320 slots (P = 4 up to 10144, else 2).
//
// A workgroup holds the drafter rows of P positions side by side in LDS and streams a table past them that is laid out for it: a
// row of the table is 64 consecutive target ids, one per lane, and a step is one entry of every lane, so a lane reads its own
// slots and weights (16 bytes at a time), gathers P values with one LDS read per entry and keeps its id's P sums in registers: no
// exchange between lanes, and q' leaves in id order.  An entry is six bytes (slot 16 bits, weight 32).  The order of an id's
// entries is chosen when the table is built so that the reads that LDS serves together touch different banks: 1.9 instead of
// 3.1 turns per group of sixteen lanes (P = 4, 16 entries), 2.0 instead of 3.6 (P = 2).
//
// What bounds it: per 64 ids, entry and position the position-minor form (rdk_sparse.hip) takes two 128-byte lines through the
// vector L1, this one 3 / P; the vector L1 hands out about 0.34 lines a clock either way.  At P = 2 that is still the bound
// (counters, N = 151936, n = 16384, k = 32, 1024 positions: 0.31-0.33 lines a clock, vector ALU 53 % and LDS 40 % busy), at P = 4
// the vector ALU is 70 % busy, LDS 45 %.  How far ahead the table is requested hardly matters (one to six units: within 8 %).
// Measured, position-minor -> this, probabilities / bf16 logits, whole fused calls in us: N = 151936, n = 16384, k = 32, 1024
// positions 866 / 921 -> 697 / 709 (bf16 702 to 724 on other rows and kept ids); N = 100000, n = 10000, k = 32, 512 positions 302 /
// 308 -> 169 / 172; N = 32000, n = 8000, k = 16, 1024 positions 119 / 139 -> 85 / 88 and 128 positions 33 / 43 -> 25 / 30; N =
// 16000, n = 4000, 256 positions 28 / 43 -> 23 / 30.
// Larger rows would have to come to LDS in windows that take turns, with sums kept between them: measured at n = 16384 with four
// positions (820-1060 us) and at n = 32064 with two (147 us against 122), the refills, the entries that do not divide evenly
// over the windows and the kept sums cost more than the lines saved.
#include "rdk_steps.hpp"

#include <limits.h>

namespace rdk {

namespace {

constexpr int kThreads = 1024;
constexpr int kWaves = kThreads / kWave;
constexpr size_t kLdsBytes = (size_t)160 * 1024;   // of a compute unit
constexpr int kRedBytes = 1024;                    // of it for the row masses and statistics
constexpr int kZeroSlots = 32;                     // slots of weight zero behind the row, one per bank: where padding points
constexpr int kUnitSteps = 8;                      // steps (one entry of every lane each) of a unit
constexpr uint32_t kUnitBytes = 3072;              // 64 x 8 slots of 16 bits, 64 x 4 weights, 64 x 4 weights
constexpr int kRing = 2;                           // units on their way to a wavefront
constexpr int most_lot_rows(int P) { return P == 4 ? 4 : 8; }   // rows that a wavefront takes at a time
constexpr int kLeastLot = 2;                           // ... a multiple of this, whose units fill whole rounds of the ring

constexpr int most_slots(int P) { return (int)((kLdsBytes - kRedBytes) / (4 * P) / 32 * 32 - kZeroSlots); }
__host__ __device__ constexpr int zero_slot(int n) { return (n + 31) / 32 * 32; }

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

template <class T>
__device__ __forceinline__ T scalar_load(const T *p)
{
    return *(const __attribute__((address_space(4))) T *)(uintptr_t)p;
}

// ------------------------------------------------------------------------------------------------ the table
struct StepBuild {
    const int32_t *slot_of;
    const int2 *nbr;
    const float *self_w;
    int N, n, k, kk;
    StepTable t;
};

struct Entries {   // of one target id: its neighbours, or a kept id's own slot
    const int2 *row;
    int count, self;
    float w;
    __device__ __forceinline__ int slot(int e) const { return row ? row[e].x : self; }
    __device__ __forceinline__ float weight(int e) const { return row ? __int_as_float(row[e].y) : w; }
};

__device__ __forceinline__ Entries entries_of(const StepBuild &b, int id)
{
    Entries x{nullptr, 0, 0, 0.f};
    if (id >= b.N) return x;
    const int s = b.slot_of[id];
    if (s >= 0) {
        x.count = 1;
        x.self = s;
        x.w = b.self_w[s];
    } else {
        x.count = b.k;
        x.row = b.nbr + (int64_t)min(-s - 1, b.N - b.n - 1) * b.kk;
    }
    return x;
}

// First unit of every row of 64 ids: as many units as its longest id takes, numbered by one workgroup.
__global__ __launch_bounds__(1024) void step_rows_kernel(StepBuild b)
{
    __shared__ uint32_t total[1024 / kWave], carry;
    const StepTable &t = b.t;
    const int tid = threadIdx.x, lane = lane_id(), wid = tid / kWave;
    const uint32_t full = (uint32_t)(b.k + kUnitSteps - 1) / kUnitSteps;
    if (tid == 0) carry = 0;
    __syncthreads();
    for (int base = 0; base <= t.rows; base += 1024) {
        const int r = base + tid;
        uint32_t v = 0;
        if (r < t.rows) {
            v = 1;
            for (int j = r * kWave; j < min((r + 1) * kWave, b.N); ++j)
                if (b.slot_of[j] < 0) v = full;
        }
        const uint32_t lot = v + __shfl_xor(v, 1, kWave);
        static_assert(kLeastLot == 2, "the rows of the smallest lot");
        if (r < t.rows && r % kLeastLot == kLeastLot - 1) v += (kRing - lot % kRing) % kRing;
        uint32_t incl = v;
        for (int o = 1; o < kWave; o <<= 1) {
            const uint32_t y = __shfl_up(incl, o, kWave);
            if (lane >= o) incl += y;
        }
        if (lane == kWave - 1) total[wid] = incl;
        __syncthreads();
        incl += carry;
        for (int w = 0; w < wid; ++w) incl += total[w];
        if (r <= t.rows) t.first[r] = incl - v;
        __syncthreads();
        if (tid == 1023) carry = incl;
        __syncthreads();
    }
}

// The lanes whose reads LDS serves together (measured): for 8 bytes a half of the wavefront, for 16 bytes two patterns in
// each half.  Lane i of group g.
template <int P>
__device__ __forceinline__ int served_lane(int g, int i)
{
    if (P == 2) return g * 32 + i;
    const int l = g & 1 ? (i < 8 ? 4 + i : i < 12 ? 8 + i : 16 + i) : (i < 4 ? i : i < 8 ? 8 + i : 12 + i);
    return (g & 2) * 16 + l;
}

__device__ __forceinline__ int wave_min(int v)
{
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) v = min(v, __shfl_xor(v, off, kWave));
    return v;
}

// The entries: one wavefront per row and group of lanes that LDS serves together, step by step.  Every lane of the group takes of its
// remaining entries one whose bank the fewest of this step's reads touch, of several the bank with the most reads still to come
// (the threads of the wavefront look at one candidate each).
template <int P>
__global__ __launch_bounds__(kWave) void step_entries_kernel(StepBuild b)
{
    constexpr int kGroups = P, kGroup = kWave / kGroups, kBanks = kGroup;
    __shared__ int2 entry[kGroup][kWave];
    __shared__ uint64_t left[kGroup];
    __shared__ int read[kBanks], todo[kBanks];
    const StepTable &t = b.t;
    const int g = blockIdx.x % kGroups, r = blockIdx.x / kGroups, lane = threadIdx.x;
    const uint32_t first = t.first[r];
    const int steps = (int)(t.first[r + 1] - first) * kUnitSteps, zero = zero_slot(b.n);
    if (lane < kBanks) todo[lane] = 0;
    __syncthreads();
    for (int i = 0; i < kGroup; ++i) {
        const Entries x = entries_of(b, r * kWave + served_lane<P>(g, i));
        if (lane < x.count) {
            entry[i][lane] = make_int2(x.slot(lane), __float_as_int(x.weight(lane)));
            atomicAdd(&todo[x.slot(lane) % kBanks], 1);
        }
        if (lane == 0) left[i] = x.count >= 64 ? ~(uint64_t)0 : ((uint64_t)1 << x.count) - 1;
    }
    for (int step = 0; step < steps; ++step) {
        char *unit = (char *)t.body + (size_t)(first + step / kUnitSteps) * kUnitBytes;
        const int st = step % kUnitSteps;
        __syncthreads();
        if (lane < kBanks) read[lane] = 0;
        for (int i = 0; i < kGroup; ++i) {
            const int li = (i * 5 + step * 7) % kGroup, l = served_lane<P>(g, li);
            __syncthreads();
            const uint64_t m = left[li];
            int2 mine = make_int2(0, 0);
            int key = INT_MAX;
            if ((m >> lane) & 1) {
                mine = entry[li][lane];
                key = read[mine.x % kBanks] << 20 | (4095 - min(todo[mine.x % kBanks], 4095)) << 8 | lane;
            }
            key = wave_min(key);
            int2 chosen;
            const bool later = key >> 20 > 0 && __popcll(m) < steps - step;   // a bank that is taken, and room in a later step
            if (m != 0 && !later) {
                const int e = key & 255;
                chosen = make_int2(lane_value(mine.x, e), lane_value(mine.y, e));
                if (lane == 0) {
                    left[li] = m & ~((uint64_t)1 << e);
                    --todo[chosen.x % kBanks];
                }
            } else {
                const int bank = wave_min(lane < kBanks ? read[lane] << 8 | lane : INT_MAX) & 255;
                chosen = make_int2(zero + bank, 0);
            }
            if (lane == 0) {
                ++read[chosen.x % kBanks];
                *(uint16_t *)(unit + l * 16 + st * 2) = (uint16_t)chosen.x;
                *(int *)(unit + 1024 + (st / 4) * 1024 + l * 16 + (st % 4) * 4) = chosen.y;
            }
        }
    }
}

// ------------------------------------------------------------------------------------------------ the product
struct StepArgs {
    const void *q;
    int64_t ldq;
    int qkind;
    int N, n, B;
    StepTable t;
    int groups, parts;    // of P positions; workgroups that share the rows of a group
    int lot;              // rows that a wavefront takes at a time
    bool by_xcd;
    SoftStat *qrow;
    float *out;
    int64_t ldo;
};

// LDS address of the slot in one half of a word: one instruction (the compiler takes two or three).
template <int HALF, int P>
__device__ __forceinline__ uint32_t lds_at(uint32_t pair, uint32_t base)
{
    uint32_t r;
    if (HALF) asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(r) : "v"(pair), "n"(4 * P), "v"(base));
    else asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(r) : "v"(pair), "n"(4 * P), "v"(base));
    return r;
}

// The P drafter rows into LDS, side by side: qm = their maxima (logits), z = the sums of their weights.  Every request is made; a
// quad that crosses the end of the row, or lies behind it, is the row's last.  red: 2 kWaves P floats; the caller's barrier
// follows.
template <int QK, int P>
__device__ __forceinline__ void fill_rows(const char *const (&row)[P], int n, float *slab, float *red, float (&qm)[P])
{
    const int wid = threadIdx.x / kWave, lane = lane_id();
    constexpr int kIter = (most_slots(P) / 4 + kThreads - 1) / kThreads;
    typename RawQuad<QK>::type raw[kIter][P];
#pragma unroll
    for (int v = 0; v < kIter; ++v)
#pragma unroll
        for (int p = 0; p < P; ++p) raw[v][p] = raw_quad<QK>(row[p], (int)(threadIdx.x + v * kThreads) * 4, n);
#pragma unroll
    for (int p = 0; p < P; ++p) {
        qm[p] = 0.f;
        if (QK != RDK_PROB_F32) {
            float m = -INFINITY;   // what is read twice does not change a maximum
#pragma unroll
            for (int v = 0; v < kIter; ++v) {
                float x[4];
                RawQuad<QK>::to(raw[v][p], x);
                m = fmaxf(m, fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3])));
            }
            m = wave_max(m);
            if (lane == 0) red[wid * P + p] = m;
        }
    }
    if (QK != RDK_PROB_F32) {
        __syncthreads();
#pragma unroll
        for (int p = 0; p < P; ++p) qm[p] = weight_reference(wave_max(red[lane % kWaves * P + p]));
    }
    float z[P];
#pragma unroll
    for (int p = 0; p < P; ++p) z[p] = 0.f;
#pragma unroll
    for (int v = 0; v < kIter; ++v) {
        const int i = (int)(threadIdx.x + v * kThreads) * 4;
        if (i >= n) continue;
        float w[4][P];
#pragma unroll
        for (int p = 0; p < P; ++p) {
            float x[4];
            RawQuad<QK>::to(raw[v][p], x);
            const int past = i - (n - 4);
            if (past > 0) {
                quad_shift(x, past);
#pragma unroll
                for (int e = 0; e < 4; ++e) x[e] = i + e < n ? x[e] : QK == RDK_PROB_F32 ? 0.f : -INFINITY;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) w[e][p] = to_weight<QK>(x[e], qm[p], 1.f);
            z[p] += (w[0][p] + w[1][p]) + (w[2][p] + w[3][p]);
        }
        if (P == 2) {
            *(f32x4 *)(slab + i * P) = f32x4{w[0][0], w[0][1], w[1][0], w[1][1]};
            *(f32x4 *)(slab + i * P + 4) = f32x4{w[2][0], w[2][1], w[3][0], w[3][1]};
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e) *(f32x4 *)(slab + (i + e) * P) = f32x4{w[e][0], w[e][1], w[e][2 % P], w[e][3 % P]};
        }
    }
    if (threadIdx.x < kZeroSlots * P) slab[zero_slot(n) * P + threadIdx.x] = 0.f;
#pragma unroll
    for (int p = 0; p < P; ++p) {
        z[p] = wave_sum(z[p]);
        if (lane == 0) red[(kWaves + wid) * P + p] = z[p];
    }
}

// One instruction each (the compiler guards against signalling NaNs with one or two more).
__device__ __forceinline__ float min_of(float x, float y)
{
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}
__device__ __forceinline__ float max_of(float x, float y)
{
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}

// Totals over the wavefront of M values, a few lanes each: lane 16 h + i is left with value 4 i + {0, 2, 1, 3}[h].
template <int M>
__device__ __forceinline__ float spread_totals(const float (&v)[M], int lane)
{
    constexpr int kRegs = (M + 3) / 4;
    float t[kRegs];
#pragma unroll
    for (int i = 0; i < kRegs; ++i) {
        float h[2];
#pragma unroll
        for (int j = 0; j < 2; ++j) {
            const int at = 4 * i + 2 * j;
            const float x = at < M ? v[at < M ? at : 0] : 0.f, y = at + 1 < M ? v[at + 1 < M ? at + 1 : 0] : 0.f;
            const auto two = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
            h[j] = __uint_as_float(two[0]) + __uint_as_float(two[1]);
        }
        const auto two = __builtin_amdgcn_permlane16_swap(__float_as_uint(h[0]), __float_as_uint(h[1]), false, false);
        t[i] = row16_sum(__uint_as_float(two[0]) + __uint_as_float(two[1]));
    }
    float r = t[0];
#pragma unroll
    for (int i = 1; i < kRegs; ++i) r = (lane & 15) == i ? t[i] : r;
    return r;
}

// A unit's data on its way: the slots and weights of eight steps.
struct UnitData {
    uint4 slots;
    f32x4 w0, w1;
};

template <int PK, int P>
__global__ __launch_bounds__(kThreads) void steps_product_kernel(StepArgs a, FuseArgs f)
{
    constexpr bool FUSE = PK >= 0, SUMS = PK != -1;
    constexpr int PKIND = FUSE ? PK : RDK_PROB_F32;
    constexpr int kSums = FUSE ? 3 * P : P;
    constexpr int kHold = most_lot_rows(P);
    constexpr uint32_t kPBytes = PKIND == RDK_LOGIT_BF16 ? 2 : 4;
    typedef float V __attribute__((ext_vector_type(P)));
    extern __shared__ __attribute__((aligned(16))) float lds[];
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    const int N = a.N, rows = a.t.rows;
    float *red = lds;                      // [2][kWaves][P] maxima and masses
    float *stats = red + 2 * kWaves * P;   // [P] maxima and [P] 1 / normalisers of the target rows
    int *taken = (int *)(stats + 2 * P);   // lots given out
    float *slab = lds + kRedBytes / sizeof(float);
    typedef const __attribute__((address_space(3))) V LdsV;
    const uint32_t slab_at = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) float *)slab;

    int group, part;
    if (a.by_xcd) {
        const int per = (a.groups + 7) / 8, rank = blockIdx.x / 8;
        part = rank / per;
        group = rank % per * 8 + blockIdx.x % 8;
    } else {
        group = blockIdx.x / a.parts;
        part = blockIdx.x % a.parts;
    }
    if (group >= a.groups) return;
    const int b0 = group * P;
    const char *qrow[P], *prow[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        const int64_t b = min(b0 + p, a.B - 1);
        qrow[p] = (const char *)(a.qkind == RDK_LOGIT_BF16 ? row_ptr<RDK_LOGIT_BF16>(a.q, a.ldq, b) : row_ptr<RDK_PROB_F32>(a.q, a.ldq, b));
        prow[p] = FUSE ? (const char *)row_ptr<PKIND>(f.p, f.ldp, b) : nullptr;
    }
    // softmax statistics of logit target rows: one wavefront per row
    if (FUSE && PKIND != RDK_PROB_F32 && wid < P) {
        const SoftStat s = merged_row_stat<RDK_LOGIT_F32>(f.pstat, f.p_splits, min(b0 + wid, a.B - 1));
        if (lane == 0) {
            stats[wid] = s.m;
            stats[wid + P] = 1.0f / s.s;
            if (part == 0 && b0 + wid < a.B) f.pmerged[b0 + wid] = s;
        }
    }
    if (threadIdx.x == 0) *taken = kWaves;
    float qm[P];
    if (a.qkind == RDK_PROB_F32) fill_rows<RDK_PROB_F32, P>(qrow, a.n, slab, red, qm);
    else if (a.qkind == RDK_LOGIT_F32) fill_rows<RDK_LOGIT_F32, P>(qrow, a.n, slab, red, qm);
    else fill_rows<RDK_LOGIT_BF16, P>(qrow, a.n, slab, red, qm);
    __syncthreads();
    float zinv[P], pm[P], pinv[P];
#pragma unroll
    for (int p = 0; p < P; ++p) {
        zinv[p] = inv_mass(wave_sum(lane < kWaves ? red[(kWaves + lane) * P + p] : 0.f));
        pm[p] = FUSE && PKIND != RDK_PROB_F32 ? stats[p] : 0.f;
        pinv[p] = FUSE && PKIND != RDK_PROB_F32 ? stats[P + p] : 1.f;
        if (part == 0 && threadIdx.x == 0 && b0 + p < a.B) a.qrow[b0 + p] = SoftStat{qm[p], zinv[p]};
    }
    // where the sums of a row go: the lane that spread_totals leaves a value with, and its entry of the first row
    float *sum_to = nullptr;
    if (SUMS) {
        const int h = lane >> 4, v = 4 * (lane & 15) + (h == 1 ? 2 : h == 2 ? 1 : h), p = v % P, kind = v / P;
        if (v < kSums && b0 + p < a.B) sum_to = (kind == 0 ? f.part_q : kind == 1 ? f.part_r : f.part_a) + (int64_t)(b0 + p) * rows;
    }

    // lots of kHold rows, to whichever wavefront is free: the older wavefronts of a SIMD get more of its issue slots
    const int hold = a.lot, lots = (rows + hold - 1) / hold, lot_stop = (int)((int64_t)lots * (part + 1) / a.parts);
    int lot = (int)((int64_t)lots * part / a.parts) + wid;
    if (lot >= lot_stop) return;
    uint32_t at = scalar_load(a.t.first + lot * hold);
    const char *src = (const char *)a.t.body + (size_t)at * kUnitBytes;
    uint32_t ask = at, ask_end = scalar_load(a.t.first + min((lot + 1) * hold, rows));   // what is requested next
    int next_lot = lot;
    uint32_t next_at = at, next_end = ask_end;
    UnitData data[kRing];
    auto request = [&](UnitData &d) {
        // every request is made, past the end of the work for the last unit again: the number of requests on their way is then
        // the same on every path, and a wait covers no more than it has to
        if (ask == ask_end) {
            ask = next_at;
            ask_end = next_end;
            src = (const char *)a.t.body + (size_t)ask * kUnitBytes;
        }
        uint32_t lane16 = (uint32_t)lane * 16u;
        asm volatile("" : "+v"(lane16));   // a 32-bit offset beside a scalar base, not a 64-bit address kept in registers
        d.slots = *(const uint4 *)(src + lane16);
        d.w0 = *(const f32x4 *)(src + 1024 + lane16);
        d.w1 = *(const f32x4 *)(src + 2048 + lane16);
        src += kUnitBytes;
        ++ask;
        __builtin_amdgcn_sched_barrier(0);
    };
    auto take = [&]() {   // the lot after this one; none: this one again, which is not worked on
        int n = 0;
        if (lane == 0) n = atomicAdd(taken, 1);
        next_lot = __builtin_amdgcn_readfirstlane(n) + (int)((int64_t)lots * part / a.parts);
        const int l = next_lot < lot_stop ? next_lot : lot;
        next_at = scalar_load(a.t.first + l * hold);
        next_end = scalar_load(a.t.first + min((l + 1) * hold, rows));
    };
    take();
#pragma unroll
    for (int d = 0; d < kRing; ++d) request(data[d]);
    for (;;) {
        const int r0 = lot * hold, r1 = min(r0 + hold, rows);
        uint32_t row_end = scalar_load(a.t.first + r0 + 1), row_end2 = scalar_load(a.t.first + r0 + 2);
        uint32_t row_end3 = scalar_load(a.t.first + min(r0 + 3, rows));
        const uint32_t end = scalar_load(a.t.first + r1);
        uint32_t praw[FUSE ? kHold : 1][P];
        if (FUSE) {
#pragma unroll
            for (int x = 0; x < kHold; ++x) {
                const int base = min(min(r0 + x, r1 - 1) * kWave, N - 1);
                const uint32_t off = (uint32_t)min(lane, N - 1 - base) * kPBytes;
#pragma unroll
                for (int p = 0; p < P; ++p) {
                    if (PKIND == RDK_LOGIT_BF16) praw[x][p] = __builtin_nontemporal_load((const uint16_t *)(prow[p] + (size_t)base * kPBytes + off));
                    else praw[x][p] = __builtin_nontemporal_load((const uint32_t *)(prow[p] + (size_t)base * kPBytes + off));
                }
            }
        }
        typedef float HeldVec __attribute__((ext_vector_type(kHold * P)));
        HeldVec held = (HeldVec)(0.f);
        int i = 0;
        float acc[P];
#pragma unroll
        for (int p = 0; p < P; ++p) acc[p] = 0.f;
        do {
#pragma unroll
            for (int d = 0; d < kRing; ++d) {
                const UnitData &u = data[d];
                V g[4], h[4];
                g[0] = *(LdsV *)lds_at<0, P>(u.slots.x, slab_at);
                g[1] = *(LdsV *)lds_at<1, P>(u.slots.x, slab_at);
                g[2] = *(LdsV *)lds_at<0, P>(u.slots.y, slab_at);
                g[3] = *(LdsV *)lds_at<1, P>(u.slots.y, slab_at);
                h[0] = *(LdsV *)lds_at<0, P>(u.slots.z, slab_at);
                h[1] = *(LdsV *)lds_at<1, P>(u.slots.z, slab_at);
                h[2] = *(LdsV *)lds_at<0, P>(u.slots.w, slab_at);
                h[3] = *(LdsV *)lds_at<1, P>(u.slots.w, slab_at);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int p = 0; p < P; ++p) acc[p] = fmaf(u.w0[e], g[e][p], acc[p]);
#pragma unroll
                for (int e = 0; e < 4; ++e)
#pragma unroll
                    for (int p = 0; p < P; ++p) acc[p] = fmaf(u.w1[e], h[e][p], acc[p]);
                if (++at == row_end) {
#pragma unroll
                    for (int p = 0; p < P; ++p) {
                        held[p * kHold + i] = acc[p];
                        acc[p] = 0.f;
                    }
                    ++i;
                    row_end = row_end2;
                    row_end2 = row_end3;
                    row_end3 = scalar_load(a.t.first + min(r0 + i + 3, rows));
                }
                request(data[d]);
            }
        } while (at != end);

        // q' itself, and its sums
#pragma unroll
        for (int x = 0; x < kHold; ++x) {
            const int r = r0 + x, id = r * kWave + lane;
            if (r >= r1) break;
            float sums[kSums];
#pragma unroll
            for (int p = 0; p < P; ++p) {
                const float qv = held[p * kHold + x] * zinv[p];
                if (a.out != nullptr && id < N && b0 + p < a.B) __builtin_nontemporal_store(qv, a.out + (int64_t)(b0 + p) * a.ldo + id);
                if (SUMS) sums[p] = qv;
                if (FUSE) {
                    const float raw = PKIND == RDK_LOGIT_BF16 ? __uint_as_float(praw[x][p] << 16) : __uint_as_float(praw[x][p]);
                    float pe = to_weight<PKIND>(raw, pm[p], pinv[p]);
                    if ((r + 1) * kWave > N) pe = id < N ? pe : 0.f;
                    sums[P + p] = max_of(pe - qv, 0.f);
                    sums[2 * P + p] = min_of(pe, qv);
                }
            }
            if (SUMS) {
                const float total = spread_totals<kSums>(sums, lane);
                if (sum_to) sum_to[r] = total;
            }
        }
        if (next_lot >= lot_stop) break;
        lot = next_lot;
        at = next_at;
        take();
    }
}

template <int PK, int P>
rdk_status_t launch_one(const StepArgs &a, const FuseArgs &f, hipStream_t st)
{
    static LdsGrant grant;
    const rdk_status_t rc = grant((const void *)steps_product_kernel<PK, P>, kLdsBytes);
    if (rc != RDK_OK) return rc;
    const int grid = (a.by_xcd ? (a.groups + 7) / 8 * 8 : a.groups) * a.parts;
    const size_t lds = kRedBytes + ((size_t)zero_slot(a.n) + kZeroSlots) * P * sizeof(float);
    RDK_TIMED_LAUNCH("sparse_product_kernel", (steps_product_kernel<PK, P>), dim3((unsigned)grid), dim3(kThreads), lds, st, a, f);
    RDK_LAUNCH_CHECK("sparse_product_kernel");
    return RDK_OK;
}

template <int P>
rdk_status_t launch_kind(int kind, const StepArgs &a, const FuseArgs &f, hipStream_t st)
{
    switch (kind) {
        case -2: return launch_one<-2, P>(a, f, st);
        case -1: return launch_one<-1, P>(a, f, st);
        case RDK_PROB_F32: return launch_one<RDK_PROB_F32, P>(a, f, st);
        case RDK_LOGIT_F32: return launch_one<RDK_LOGIT_F32, P>(a, f, st);
        case RDK_LOGIT_BF16: return launch_one<RDK_LOGIT_BF16, P>(a, f, st);
    }
    return RDK_ERR_DTYPE;
}

}  // namespace

StepTable step_table_plan(int32_t N, int32_t n, int32_t k, size_t *bytes)
{
    StepTable t{};
    *bytes = 0;
    // none for a kernel of which no batch of a thousand positions or two would read enough to take this form (steps_taken)
    if (k < 1 || n < 4 || n > most_slots(2) || (int64_t)(N - n) * ((k + 15) / 16 * 16) * 8 < (int64_t)128 << 10) return t;
    t.P = n <= most_slots(4) ? 4 : 2;
    t.rows = sparse_blocks(N);
    const size_t units = (size_t)t.rows * ((k + kUnitSteps - 1) / kUnitSteps) + (size_t)t.rows / kLeastLot * (kRing - 1);
    size_t off = 0;
    t.off_body = off; off += align_up(units * kUnitBytes, 256);
    t.off_first = off; off += align_up((size_t)(t.rows + 1) * 4, 256);
    *bytes = off;
    return t;
}

void step_table_place(StepTable &t, char *base)
{
    t.body = base + t.off_body;
    t.first = (uint32_t *)(base + t.off_first);
}

rdk_status_t launch_step_table(const KernelHandle &h, hipStream_t st)
{
    const StepBuild b{h.slot_of, h.nbr, h.self_w, h.N, h.n, h.k, h.kk, h.steps};
    if (h.steps.P == 0) return RDK_OK;
    hipLaunchKernelGGL(step_rows_kernel, dim3(1), dim3(1024), 0, st, b);
    RDK_LAUNCH_CHECK("step_rows_kernel");
    const dim3 grid((unsigned)h.steps.rows * h.steps.P);
    if (h.steps.P == 2) hipLaunchKernelGGL((step_entries_kernel<2>), grid, dim3(kWave), 0, st, b);
    else hipLaunchKernelGGL((step_entries_kernel<4>), grid, dim3(kWave), 0, st, b);
    RDK_LAUNCH_CHECK("step_entries_kernel");
    return RDK_OK;
}

// The table is read once per P positions here, once per position in the product out of LDS one row at a time (rdk_slab.hip), which
// reads it in 16 neighbours and 8 bytes each, and finishes a row in the same launch where one workgroup holds it.  The line to
// that form lies at 180 MiB of its table reads.  Fused calls, one row at a time -> this, probabilities / bf16 logits, us:
//   above it  N = 32000, n = 8000, 63 positions (184 MiB) 21.9 / 27.9 -> 19.7 / 24.8; N = 16000, n = 4000, 128 (187) 20.9 / 27.2 ->
//             18.3 / 24.6; N = 64000, n = 16000, 32 (187) 23.3 / 29.4 -> 22.9 / 26.2; N = 250000, n = 20000, k = 8, 7 (196) 44.1 /
//             51.1 -> 22.5 / 27.9; N = 100000, n = 20000, 24 (234) 29.3 / 35.2 -> 29.4 / 34.6; N = 100000, n = 10000, 20 (219) 24.8 /
//             31.2 -> 25.3 / 31.2, the one that loses of seventeen measured there
//   below it  N = 32000, n = 8000, 32 / 40 / 48 positions (93 / 117 / 140 MiB) 16.5 -> 18.7 / 18.0 -> 18.9 / 20.4 -> 19.1 (bf16 22.2 ->
//             24.2 / 24.3 -> 24.5 / 26.2 -> 24.5); N = 64000, n = 16000, 24 (140) 22.0 / 28.0 -> 23.2 / 27.4; N = 100000, n = 10000, 12 /
//             16 (131 / 175) 26.4 -> 20.8 / 21.1 -> 22.2; N = 250000, n = 10144, 6 (175) 40.7 / 46.5 -> 25.6 / 31.7
// What decides is how the positions of a batch divide over the compute units in either form more than the bytes: between 120 MiB
// and the line this form is already the faster one for most shapes, above the line for all but that one.  A row that is finished in
// place stays there while every row has a compute unit of its own, which pays for logits: N = 8000, n = 2000, 256 positions (187
// MiB) 17.8 / 19.8 -> 17.5 / 24.4, N = 12000, n = 3000, 256 positions (281 MiB) 24.2 / 24.8 -> 20.5 / 26.9; with more rows than
// units, N = 4000, n = 1000, 512 positions (187 MiB), 23.2 / 26.8 -> 19.2 / 25.8.  Beyond 288 MiB (where the position-minor form is
// the other one) this is never the slower.
bool steps_taken(const KernelHandle &h, int32_t B)
{
    if (h.steps.P == 0 || (int64_t)B * (h.N - h.n) * h.kk * 8 <= (int64_t)180 << 20) return false;
    return !(slab_taken(h, B) && slab_finishes(h, B) && B <= kComputeUnits);
}

rdk_status_t launch_steps_product(const KernelHandle &h, RowInput q, int32_t B, float *out, int64_t ldo, SoftStat *qrow, int kind,
                                 const FuseArgs &f, hipStream_t st)
{
    StepArgs a{};
    a.q = q.ptr; a.ldq = q.ld;
    a.qkind = q.kind;
    a.N = h.N; a.n = h.n; a.B = B;
    a.t = h.steps;
    a.groups = (B + a.t.P - 1) / a.t.P;
    a.by_xcd = a.groups >= 32;
    const int padded = a.by_xcd ? (a.groups + 7) / 8 * 8 : a.groups;
    // a workgroup per compute unit, and lots that keep its wavefronts busy to the end
    a.parts = padded >= kComputeUnits ? 1 : kComputeUnits / padded;
    const int most = (a.t.rows / kLeastLot + kWaves - 1) / kWaves;
    if (a.parts > most) a.parts = most;
    a.lot = most_lot_rows(a.t.P);
    while (a.lot > kLeastLot && a.t.rows / a.parts < a.lot * kWaves * 4) a.lot /= 2;
    a.qrow = qrow;
    a.out = out; a.ldo = ldo;
    return a.t.P == 2 ? launch_kind<2>(kind, a, f, st) : launch_kind<4>(kind, a, f, st);
}

}  // namespace rdk
