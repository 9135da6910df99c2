// Exact redistribution (Alg. 1, step 2):  P'[b, j] = sum_s Q'[b, s] M[s, j]  with a dense kernel M.
//   fp32 kernel:  both operands split into three bf16 parts each, six part products per term on the bf16 matrix
//                 cores (v_mfma_f32_32x32x16_bf16) with fp32 accumulation; M read straight from its row-major
//                 rows, split over the kept slots, fixed-order reduction.
//   bf16 kernel:  M rounded to bf16, the drafter rows to eleven significant bits; both held as scaled fp16 numbers,
//                 fp32 accumulation on the matrix cores (v_mfma_f32_32x32x16_f16), rows rescaled so that they sum to one.
// Step 1 (Eq. 1) is folded in: rows of Q' are the drafter rows divided by their sums.
#include <algorithm>

#include "rdk_rowstats.hpp"

namespace rdk {

namespace {

// ------------------------------------------------------------------------------------------------ fp32
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kRowGroup = 64;    // positions per wavefront tile: two 32-row MFMA blocks
constexpr int kColSet = 128;     // target ids per wavefront tile

// At 64 positions the product needs 2 n N flop against 4 n N bytes of M: 32 flop per byte, more than the fp32 matrix
// unit delivers per HBM byte (157 TFLOP/s : 8 TB/s = 20).  The bf16 matrix instruction is sixteen times as fast, and
// an fp32 number is the exact sum of three bf16 numbers (its leading, middle and trailing eight significant bits), so
// the product of two fp32 numbers is taken from the six largest products of their parts, all accumulated in fp32 by
// the MFMA:
//   x y = xh yh + (xh ym + xm yh) + (xh yl + xl yh + xm ym) + terms below 2^-24 |x y|.
// Every part product is exact in fp32, so the result carries the rounding of an fp32 dot product.  With six bf16
// MFMAs in place of sixteen fp32 ones per sixteen slots the path is bound by reading M, not by the matrix rate.
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kSplitStep = 16;   // kept slots per bf16 MFMA
constexpr int kSplitRing = 3;     // slot blocks in the load ring (all but one ahead of the MFMAs; deeper rings gain nothing)

// Upper halves of h, m, l hold the three bf16 parts of x (x = h + m + l exactly, for normal numbers).
__device__ __forceinline__ void split3(float x, uint32_t &h, uint32_t &m, uint32_t &l)
{
    h = __float_as_uint(x) & 0xFFFF0000u;
    const float r = x - __uint_as_float(h);      // exact: at most sixteen significant bits are left
    m = __float_as_uint(r) & 0xFFFF0000u;
    l = __float_as_uint(r - __uint_as_float(m)); // exact, at most eight significant bits: already a bf16 number
}

// two bf16 numbers given in the upper halves of a and b, packed as (a, b) = (low half, high half)
__device__ __forceinline__ uint32_t pack_upper(uint32_t a, uint32_t b) { return (a >> 16) | (b & 0xFFFF0000u); }

// ---- The drafter rows are brought into operand form by one workgroup per row, which also takes the row's statistics: a
// launch for the statistics alone cost 3 us, and loads of single values more (fp32 path, N = 2000, n = 500, one position: 19.9
// -> 17.5 us a call; 16-bit path, N = 8000, n = 2000, 16 positions 24.1 -> 20.2, N = 32000, n = 8000, 64 positions 119.7 -> 111.3).
constexpr int kPrepThreads = 512;
constexpr int kPrepWaves = kPrepThreads / kWave;

// The raw values of slots s .. s + 7 of a row, `fill` past its end.
template <int QK>
__device__ __forceinline__ void load8(const void *qr, int s, int n, float fill, float (&v)[8])
{
    if (s + 8 <= n) {
        float lo[4], hi[4];
        const typename RawQuad<QK>::type a = raw_quad<QK>(qr, s, n), b = raw_quad<QK>(qr, s + 4, n);
        RawQuad<QK>::to(a, lo);
        RawQuad<QK>::to(b, hi);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[e] = lo[e];
            v[4 + e] = hi[e];
        }
    } else {
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = s + e < n ? load1<QK>(qr, s + e) : fill;
    }
}

// What a logit row's weights are formed against, in every thread (0 for probabilities).
template <int QK>
__device__ __forceinline__ float prep_row_max(const void *qr, int n, float *sh)
{
    if (QK == RDK_PROB_F32) return 0.f;
    float m = -INFINITY;
    for (int s = threadIdx.x * 8; s < n; s += kPrepThreads * 8) {
        float v[8];
        load8<QK>(qr, s, n, -INFINITY, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) m = fmaxf(m, v[e]);
    }
    m = wave_max(m);
    if (lane_id() == 0) sh[threadIdx.x / kWave] = m;
    __syncthreads();
    m = sh[0];
    for (int i = 1; i < kPrepWaves; ++i) m = fmaxf(m, sh[i]);
    __syncthreads();
    return weight_reference(m);
}

// Sum over the workgroup, in every thread.
template <typename T>
__device__ __forceinline__ T prep_row_sum(T v, T *sh)
{
    v = wave_sum(v);
    if (lane_id() == 0) sh[threadIdx.x / kWave] = v;
    __syncthreads();
    v = sh[0];
    for (int i = 1; i < kPrepWaves; ++i) v += sh[i];
    return v;
}

// A records of this form: for row block rb (32 positions) and slot block kb (16 slots) three consecutive 1 KB
// records, part p = 0 (leading), 1, 2; lane l = 32 g + r holds part p of the unnormalised drafter weights of
// position 32 rb + r at slots 16 kb + 8 g + e, e = 0..7 -- the A operand of one 32x32x16 MFMA.  Zero beyond B and n.
// One workgroup per row (blockIdx.x, whole row groups); qstat[b] receives the row's maximum (logits) and mass.
template <int QK>
__global__ __launch_bounds__(kPrepThreads) void prep_a_split_kernel(const void *q, int64_t ldq, SoftStat *qstat, int n, int B, int KB,
                                                                    uint16_t *Ap)
{
    __shared__ float sh[kPrepWaves];
    const int b = blockIdx.x;
    const void *qr = row_ptr<QK>(q, ldq, min(b, B - 1));
    const float fill = QK == RDK_PROB_F32 ? 0.f : -INFINITY;
    const float qm = prep_row_max<QK>(qr, n, sh);
    float z = 0.f;
    for (int c = threadIdx.x; c < KB * 2; c += kPrepThreads) {   // eight consecutive slots
        uint32_t h[8], m[8], lo[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) h[e] = m[e] = lo[e] = 0u;
        if (b < B && c * 8 < n) {
            float v[8];
            load8<QK>(qr, c * 8, n, fill, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const float x = to_weight<QK>(v[e], qm, 1.f);
                z += x;
                split3(x, h[e], m[e], lo[e]);
            }
        }
        uint4 *dst = (uint4 *)Ap + (((int64_t)(b / 32) * KB + c / 2) * 3) * kWave + (c % 2) * 32 + b % 32;
        dst[0] = make_uint4(pack_upper(h[0], h[1]), pack_upper(h[2], h[3]), pack_upper(h[4], h[5]), pack_upper(h[6], h[7]));
        dst[kWave] = make_uint4(pack_upper(m[0], m[1]), pack_upper(m[2], m[3]), pack_upper(m[4], m[5]), pack_upper(m[6], m[7]));
        dst[2 * kWave] = make_uint4(pack_upper(lo[0], lo[1]), pack_upper(lo[2], lo[3]), pack_upper(lo[4], lo[5]), pack_upper(lo[6], lo[7]));
    }
    z = prep_row_sum(z, sh);
    if (threadIdx.x == 0 && b < B) qstat[b] = SoftStat{qm, z};
}

// The same for long rows: a thread per 16 bytes of the records, in their order.  Workgroups that own a row write 16 bytes of a
// 128-byte line each, three times per eight slots.  The records of logits need the row's maximum: that costs more than the
// launch for it from about 5000 slots on (one launch against two, a call of 16 positions: n = 2000 29.7 us against 32.4, 4000 56.9 :
// 58.4, 5000 76.2 : 76.3, 8000 198.3 : 196.1).  Those of probabilities need nothing of their row, whose mass is taken by the first B
// workgroups of the same launch: one workgroup a row -> this, the product's calls, n = 2000, one position 24.0 -> 23.8, 256 52.9 ->
// 51.9, n = 4000, one 49.0 -> 45.6, 256 158.9 -> 154.8; n = 600 either way the same.  With a launch for the mass: n = 6000, 5 positions
// 80.0 -> 76.9, n = 12001, 256 1414 -> 1405.
constexpr int kPrepRowMax = 4096, kPrepRowMaxProb = 2048;
template <int QK>
__global__ __launch_bounds__(kStatThreads) void prep_a_records_kernel(const void *q, int64_t ldq, SoftStat *qstat, int n, int B, int KB,
                                                                      int64_t records, uint16_t *Ap)
{
    const int mass_rows = QK == RDK_PROB_F32 ? B : 0;
    if ((int)blockIdx.x < mass_rows) {
        row_stats<QK>(row_ptr<QK>(q, ldq, blockIdx.x), n, 0, (n + kChunk - 1) / kChunk, qstat + blockIdx.x);
        return;
    }
    const int64_t idx = (int64_t)(blockIdx.x - mass_rows) * blockDim.x + threadIdx.x;
    if (idx >= records * kWave) return;
    const int l = (int)(idx % kWave);
    const int64_t rec = idx / kWave;
    const int kb = (int)(rec % KB);
    const int b = (int)(rec / KB) * 32 + l % 32, g = l / 32;
    uint32_t h[8], m[8], lo[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) h[e] = m[e] = lo[e] = 0u;
    if (b < B) {
        const void *qr = row_ptr<QK>(q, ldq, b);
        const float qm = QK == RDK_PROB_F32 ? 0.f : weight_reference(qstat[b].m);
        const int s = kb * kSplitStep + g * 8;
        if (s < n) {
            float v[8];
            load8<QK>(qr, s, n, QK == RDK_PROB_F32 ? 0.f : -INFINITY, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) split3(to_weight<QK>(v[e], qm, 1.f), h[e], m[e], lo[e]);
        }
    }
    uint4 *dst = (uint4 *)(Ap + ((rec * 3) * kWave + l) * 8);
    dst[0] = make_uint4(pack_upper(h[0], h[1]), pack_upper(h[2], h[3]), pack_upper(h[4], h[5]), pack_upper(h[6], h[7]));
    dst[kWave] = make_uint4(pack_upper(m[0], m[1]), pack_upper(m[2], m[3]), pack_upper(m[4], m[5]), pack_upper(m[6], m[7]));
    dst[2 * kWave] = make_uint4(pack_upper(lo[0], lo[1]), pack_upper(lo[2], lo[3]), pack_upper(lo[4], lo[5]), pack_upper(lo[6], lo[7]));
}

// One wavefront per (128 target ids, 64 positions, one split of the slot blocks), one wavefront per SIMD.  The B
// operand of the 32x32x16 MFMA wants from lane l = 32 g + c the eight slots 8 g .. 8 g + 7 of column c.  Column c of
// MFMA e (e = 0..3) is given the target id j0 + 4 c + e, so the lane reads M[s][j0 + 4c .. + 3] for its eight slots
// s = 16 kb + 8 g + i with eight 16-byte loads of the row-major M -- no packing of M -- splits the 32 values
// in registers and feeds four MFMA columns; the four results of a lane are again four consecutive ids.  Loads run
// two slot blocks ahead through a ring of three register sets; the split length is a multiple of three blocks (A is
// zero beyond n, rows of M are clamped to the last one).  Tiles of 64 ids at two wavefronts per SIMD were slower
// (0.26 ms against 0.22 ms): every wavefront reads all drafter records of its split.
//
// What bounds it: reading M (N = 32000, n = 8000, 64 positions: 1 GB in 180 us, 5.7 TB/s, where a bare read stream reaches
// 6.9), and the matrix unit for several row groups.  A lone wavefront has to keep both busy from one instruction stream, so the
// parts of a pair of columns are taken one unit ahead of their products and every MFMA is followed by five vector instructions
// and now and then one load: eight loads at once fill the queue of the vector memory pipe, and the wavefront waits there
// without issuing MFMAs.  The barrier keeps the wavefronts of a workgroup in step: they read neighbouring pieces of the same
// rows of M, and drift apart otherwise (N = 64000, n = 16000, one position: 680 us a call without it, 640 with it).  The row
// groups of a tile run side by side on one XCD, whose L2 then reads M once for all of them.
// Whole calls (product and verification), loads and products in turn -> this: N = 32000, n = 8000, 64 positions 226 -> 211 us;
// N = 64000, n = 16000, one 713 -> 640; N = 30000, n = 12000, 100 539 -> 481; N = 40000, n = 5000, 256 754 -> 651; N = 5000, n =
// 1000, five 26.0 -> 24.9.  The drafter records through LDS instead, once per workgroup: 1-2 % slower everywhere.
constexpr int kSplitWaves = 4;   // wavefronts per workgroup: neighbouring id tiles

// M is loaded non-temporally where it is read once and is larger than the memory-side cache (213 -> 209 us at 1 GB); a smaller one
// may still lie there from the call before (N = 5000, n = 1000: 26.7 us non-temporally, 24.8 without).
constexpr size_t kLastLevelBytes = (size_t)256 << 20;

// Issue order of a unit: its 24 MFMAs spread over the vector instructions and loads.
#define RDK_INTERLEAVE(LOADS)                                                                                        \
    {                                                                                                                \
        _Pragma("unroll") for (int i_ = 0; i_ < 24; ++i_) {                                                          \
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);                                                       \
            __builtin_amdgcn_sched_group_barrier(0x002, 5, 0);                                                       \
            if (i_ * (LOADS) / 24 != (i_ + 1) * (LOADS) / 24) __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);     \
        }                                                                                                            \
        __builtin_amdgcn_sched_barrier(0);                                                                           \
    }
template <bool STREAM>
__global__ __launch_bounds__(kSplitWaves * kWave) __attribute__((amdgpu_waves_per_eu(1, 1))) void exact_f32_split_kernel(
    const uint16_t *Ap, const float *M, int64_t ldm, int n, int N, int B, int KB, int blocks_per_split, int row_groups, int splits,
    const SoftStat *qstat, float *dst, int64_t ldd, int64_t split_stride, bool scale_here)
{
    const int lane = lane_id(), c = lane % 32, g = lane / 32;
    // The row groups of a tile run at the same time on the same XCD: consecutive workgroups go round the XCDs, so each XCD is given a
    // share of the list of (split, tile, row group) of its own, equal ones, because all workgroups are to be resident at once.  (Whole
    // tiles dealt out to the XCDs left some of them with more workgroups than compute units: N = 10729, n = 2067, 235 positions
    // 122 us a call, this way 88.)
    const int tile_groups = (N + kSplitWaves * kColSet - 1) / (kSplitWaves * kColSet), share = gridDim.x / 8;
    const int item = row_groups > 1 ? blockIdx.x % 8 * share + blockIdx.x / 8 : blockIdx.x;
    const int rg = item % row_groups, tile_group = item / row_groups % tile_groups, split = item / row_groups / tile_groups;
    if (split >= splits) return;   // a whole workgroup
    const int j0 = (tile_group * kSplitWaves + threadIdx.x / kWave) * kColSet, col = j0 + 4 * c;
    const int kb0 = split * blocks_per_split, kb_last = kb0 + blocks_per_split - 1;
    const bool full = col + 3 < N;
    const int lcol = col < N ? col : 0;   // lanes beyond N read column 0 (never stored): no branch around the loads
    f32x16 acc[2][4];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int e = 0; e < 4; ++e)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[rb][e][v] = 0.f;
    const bf16x8 *a_rec[2];
#pragma unroll
    for (int rb = 0; rb < 2; ++rb) a_rec[rb] = (const bf16x8 *)Ap + ((int64_t)(rg * 2 + rb) * KB) * 3 * kWave + lane;

    bf16x8 a_ring[kSplitRing][2][3], parts[2][2][3];
    float4 b_ring[kSplitRing][8];
    auto load_a = [&](bf16x8 (&slot)[2][3], int kbi) {
        const int kb = min(kbi, kb_last);
#pragma unroll
        for (int rb = 0; rb < 2; ++rb)
#pragma unroll
            for (int pt = 0; pt < 3; ++pt) slot[rb][pt] = a_rec[rb][((int64_t)kb * 3 + pt) * kWave];
    };
    auto load_half = [&](float4 (&slot)[8], int kbi, int half) {
        const int kb = min(kbi, kb_last);
#pragma unroll
        for (int i = 4 * half; i < 4 * half + 4; ++i) {
            const int s = min(kb * kSplitStep + 8 * g + i, n - 1);
            const u32x4 *src = (const u32x4 *)(M + (int64_t)s * ldm + lcol);
            slot[i] = __builtin_bit_cast(float4, STREAM ? __builtin_nontemporal_load(src) : *src);
        }
    };
    // the three parts of the eight values of columns e and e + 1, as operands
    auto split_pair = [&](bf16x8 (&out)[2][3], const float4 (&slot)[8], int e) {
#pragma unroll
        for (int ee = 0; ee < 2; ++ee) {
            uint32_t h[8], m[8], l[8];
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const float x = e + ee == 0 ? slot[i].x : e + ee == 1 ? slot[i].y : e + ee == 2 ? slot[i].z : slot[i].w;
                split3(x, h[i], m[i], l[i]);
            }
            const u32x4 hv = {pack_upper(h[0], h[1]), pack_upper(h[2], h[3]), pack_upper(h[4], h[5]), pack_upper(h[6], h[7])};
            const u32x4 mv = {pack_upper(m[0], m[1]), pack_upper(m[2], m[3]), pack_upper(m[4], m[5]), pack_upper(m[6], m[7])};
            const u32x4 lv = {pack_upper(l[0], l[1]), pack_upper(l[2], l[3]), pack_upper(l[4], l[5]), pack_upper(l[6], l[7])};
            out[ee][0] = __builtin_bit_cast(bf16x8, hv);
            out[ee][1] = __builtin_bit_cast(bf16x8, mv);
            out[ee][2] = __builtin_bit_cast(bf16x8, lv);
        }
    };
    // the six part products of two columns, smallest first, alternating between the four accumulators involved
    auto products = [&](const bf16x8 (&af)[2][3], const bf16x8 (&bf)[2][3], int e) {
        constexpr int kPart[6][2] = {{1, 1}, {2, 0}, {0, 2}, {1, 0}, {0, 1}, {0, 0}};
#pragma unroll
        for (int x = 0; x < 6; ++x)
#pragma unroll
            for (int ee = 0; ee < 2; ++ee)
#pragma unroll
                for (int rb = 0; rb < 2; ++rb)
                    acc[rb][e + ee] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[rb][kPart[x][0]], bf[ee][kPart[x][1]], acc[rb][e + ee], 0, 0, 0);
    };
#pragma unroll
    for (int t = 0; t < kSplitRing; ++t) {
        if (t + 1 < kSplitRing) load_a(a_ring[t], kb0 + t);
        load_half(b_ring[t], kb0 + t, 0);
        if (t + 1 < kSplitRing) load_half(b_ring[t], kb0 + t, 1);
        __builtin_amdgcn_sched_barrier(0);
    }
    split_pair(parts[0], b_ring[0], 0);
    __builtin_amdgcn_sched_barrier(0);
    // A unit is half of a block: the products of two columns, and in their shade the parts of the next two columns and the loads
    // of the block whose registers fell free last.
    for (int kb = kb0; kb <= kb_last; kb += kSplitRing) {
#pragma unroll
        for (int t = 0; t < kSplitRing; ++t) {   // ring entries are compile-time constants after unrolling
            constexpr int kAhead = kSplitRing - 1;
            load_a(a_ring[(t + kAhead) % kSplitRing], kb + t + kAhead);
            load_half(b_ring[(t + kAhead) % kSplitRing], kb + t + kAhead, 1);
            split_pair(parts[1], b_ring[t], 2);
            products(a_ring[t], parts[0], 0);
            RDK_INTERLEAVE(10)
            load_half(b_ring[t], kb + t + kSplitRing, 0);
            split_pair(parts[0], b_ring[(t + 1) % kSplitRing], 0);
            products(a_ring[t], parts[1], 2);
            RDK_INTERLEAVE(4)
        }
        __builtin_amdgcn_s_barrier();
    }
#undef RDK_INTERLEAVE
    // D layout of a 32x32 tile: lane l holds column l % 32 and rows 8 * (v / 4) + 4 * (l / 32) + v % 4, v = 0..15
    float *base = dst + (int64_t)split * split_stride;
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            const int b = rg * kRowGroup + rb * 32 + 8 * (v / 4) + 4 * g + (v % 4);
            if (b >= B) continue;
            const float sc = scale_here ? inv_mass(qstat[b].s) : 1.f;
            const float o[4] = {acc[rb][0][v] * sc, acc[rb][1][v] * sc, acc[rb][2][v] * sc, acc[rb][3][v] * sc};
            float *drow = base + (int64_t)b * ldd + col;
            if (full) {
                store4(drow, o[0], o[1], o[2], o[3]);
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (col + e < N) drow[e] = o[e];
            }
        }
}

// Sum of the split partials in split order, times the row's scale (fp32 path: 1 / drafter row sum, Eq. 1).  Four ids a
// thread and four partials in flight, which come out of the memory-side cache: a thread that walked single ids paid that
// latency once per partial (fp32 path, N = 8000, n = 2000, fourteen splits: 8 positions 40.4 -> 31.5 us a call, 64: 46.3 -> 37.2).
__global__ __launch_bounds__(256) void exact_reduce_kernel(const float *part, int64_t ldd, int64_t split_stride, int splits,
                                                           const SoftStat *qstat, const float *out_scale, int N, int B, float *out,
                                                           int64_t ldo)
{
    for (int b = blockIdx.y; b < B; b += gridDim.y) {   // positions beyond the grid's second dimension are looped over
        const float sc = out_scale ? out_scale[b] : inv_mass(qstat[b].s);
        const int j = (blockIdx.x * blockDim.x + threadIdx.x) * 4;
        if (j >= N) return;
        const float *src = part + (int64_t)b * ldd + j;     // rows of partials are padded to whole quads
        float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int z0 = 0; z0 < splits; z0 += 4) {
            float4 v[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = *(const float4 *)(src + (int64_t)min(z0 + t, splits - 1) * split_stride);
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                if (z0 + t >= splits) break;
                s.x += v[t].x; s.y += v[t].y; s.z += v[t].z; s.w += v[t].w;
            }
        }
        float *dst = out + (int64_t)b * ldo + j;
        const float o[4] = {s.x * sc, s.y * sc, s.z * sc, s.w * sc};
        if (j + 3 < N) {
            store4(dst, o[0], o[1], o[2], o[3]);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (j + e < N) dst[e] = o[e];
        }
    }
}

// ------------------------------------------------------------------------------------------------ bf16

constexpr int kKStep = 16;          // kept slots per MFMA (32x32x16)
constexpr int kColBlock = 32;       // target ids per MFMA tile
constexpr int kColBlocksPerWg = 4;  // 128 target ids per workgroup

__device__ __forceinline__ uint16_t f32_to_bf16_rne(float x)
{
    uint32_t u = __float_as_uint(x);
    if ((u & 0x7F800000u) == 0x7F800000u) return (uint16_t)(u >> 16);   // inf / nan pass through
    u += 0x7FFFu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

// The 16-bit operands of the dense product.  A bf16 number keeps eight significant bits: rounding a peaked drafter row
// to it moves single outputs by up to 2^-8, twice the tolerance this path states (2e-3).  The matrix cores run fp16
// at the same rate, and fp16 keeps eleven bits, so both operands are held as fp16 numbers scaled by 2^15:
//   * an entry of M is first rounded to bf16 (the format the kernel is specified in) and that value, times 2^15, is
//     an fp16 number exactly as long as it is at least 2^-29;
//   * an entry of a normalised drafter row is rounded to eleven significant bits (relative error at most 2^-12).
// Values whose scaled magnitude is below the smallest normal fp16 number (2^-14, i.e. below 2^-29 = 1.9e-9 unscaled)
// are stored as zero, whatever the denormal mode of the hardware; the products carry the factor 2^30, taken out
// again by the row scale.
constexpr float kOperandScale = 32768.0f;                 // 2^15
constexpr float kOperandUnscale = 1.0f / 32768.0f;
constexpr float kHalfMinNormal = 6.103515625e-05f;        // 2^-14

__device__ __forceinline__ uint16_t f32_to_operand(float x)   // x >= 0, at most 1
{
    const float y = x * kOperandScale;
    if (!(y >= kHalfMinNormal)) return 0;
    return __builtin_bit_cast(uint16_t, (_Float16)y);   // round to nearest even
}

__device__ __forceinline__ float operand_to_f32(uint16_t h) { return (float)__builtin_bit_cast(_Float16, h) * kOperandUnscale; }

// an entry of M as stored: rounded to bf16, then held as a scaled fp16 number
__device__ __forceinline__ uint16_t kernel_entry(float m) { return f32_to_operand(bf16_to_f32(f32_to_bf16_rne(m))); }

// Packed layout of the bf16 kernel: for column block jb (32 ids) and slot block kb (16 slots) one
// contiguous 1 KB record holding, for lane l = 32 * g + c (g = 0..1, c = 0..31), the eight values
// M[kb*16 + g*8 + e, jb*32 + c], e = 0..7 -- exactly the B operand of one 32x32x16 MFMA, so that a
// wavefront fetches it with a single 16-byte-per-lane load.  Records of one jb are consecutive in kb.
__global__ void pack_bf16_kernel(const float *M, int64_t ldm, int n, int N, int KB, uint16_t *packed)
{
    const int jb = blockIdx.x, lane = threadIdx.x;
    const int g = lane / 32, c = lane % 32;
    const int j = jb * kColBlock + c;
    for (int kb = blockIdx.y; kb < KB; kb += gridDim.y) {
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 8; e += 2) {
            const int s = kb * kKStep + g * 8 + e;
            const float v0 = (s < n && j < N) ? M[(int64_t)s * ldm + j] : 0.f;
            const float v1 = (s + 1 < n && j < N) ? M[(int64_t)(s + 1) * ldm + j] : 0.f;
            w[e / 2] = (uint32_t)kernel_entry(v0) | ((uint32_t)kernel_entry(v1) << 16);
        }
        *(uint4 *)(packed + (((int64_t)jb * KB + kb) * 64 + lane) * 8) = make_uint4(w[0], w[1], w[2], w[3]);
    }
}

// fp32 sums of the rows of M as stored (needed to rescale output rows to unit mass).
__global__ void rounded_row_sum_kernel(const float *M, int64_t ldm, int N, float *row_sum)
{
    const int s = blockIdx.x;
    double sum = 0.0;
    for (int j = threadIdx.x; j < N; j += blockDim.x)
        sum += (double)operand_to_f32(kernel_entry(M[(int64_t)s * ldm + j]));
    sum = wave_sum(sum);
    __shared__ double sh[4];
    if (lane_id() == 0) sh[threadIdx.x / kWave] = sum;
    __syncthreads();
    if (threadIdx.x == 0) row_sum[s] = (float)((sh[0] + sh[1]) + (sh[2] + sh[3]));
}

__global__ void unpack_bf16_kernel(const uint16_t *packed, int n, int N, int KB, float *M, int64_t ldm)
{
    const int jb = blockIdx.x, lane = threadIdx.x;
    const int g = lane / 32, c = lane % 32;
    const int j = jb * kColBlock + c;
    if (j >= N) return;
    for (int kb = blockIdx.y; kb < KB; kb += gridDim.y) {
        const uint16_t *rec = packed + (((int64_t)jb * KB + kb) * 64 + lane) * 8;
        for (int e = 0; e < 8; ++e) {
            const int s = kb * kKStep + g * 8 + e;
            if (s < n) M[(int64_t)s * ldm + j] = operand_to_f32(rec[e]);
        }
    }
}

// A operand: TLI-normalised drafter rows as 16-bit operands (see f32_to_operand), packed like M: for row block rb (32 positions) and
// slot block kb (16 slots) one 1 KB record holding, for lane l = 32 * g + r, the eight values
// q'[rb*32 + r, kb*16 + g*8 + e], e = 0..7 -- the A operand of one 32x32x16 MFMA.  Also per row the factor
// 2^-30 / sum_s rounded(q'_s) * row_sum[s]: it takes the operand scales out and makes the output row sum to one.
// One workgroup per position.
template <int QK>
__global__ __launch_bounds__(kPrepThreads) void prep_a_bf16_kernel(const void *q, int64_t ldq, const float *row_sum, int n, int KB, int B,
                                                                   uint16_t *Ap, float *out_scale)
{
    __shared__ float sh[kPrepWaves];
    __shared__ double shd[kPrepWaves];
    const int b = blockIdx.x;
    const int rb = b / 32, r = b % 32;
    const float fill = QK == RDK_PROB_F32 ? 0.f : -INFINITY;
    const void *qr = row_ptr<QK>(q, ldq, min(b, B - 1));
    // the row is normalised before it is rounded: its mass comes out of a pass of its own (the others hit the caches)
    const float qm = prep_row_max<QK>(qr, n, sh);
    float z = 0.f;
    for (int s = threadIdx.x * 8; s < n; s += kPrepThreads * 8) {
        float v[8];
        load8<QK>(qr, s, n, fill, v);
#pragma unroll
        for (int e = 0; e < 8; ++e) z += to_weight<QK>(v[e], qm, 1.f);
    }
    const float inv = inv_mass(prep_row_sum(z, sh));
    double mass = 0.0;
    for (int c = threadIdx.x; c < KB * 2; c += kPrepThreads) {   // chunk of 8 consecutive slots
        const int kb = c / 2, g = c % 2;
        uint32_t w[4] = {0u, 0u, 0u, 0u};
        if (b < B && c * 8 < n) {
            float v[8], ms[8];
            load8<QK>(qr, c * 8, n, fill, v);
            load8<RDK_PROB_F32>(row_sum, c * 8, n, 0.f, ms);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const uint16_t h = f32_to_operand(to_weight<QK>(v[e], qm, 1.f) * inv);
                mass += (double)operand_to_f32(h) * (double)ms[e];
                w[e / 2] |= (uint32_t)h << (16 * (e % 2));
            }
        }
        *(uint4 *)(Ap + (((int64_t)rb * KB + kb) * 64 + g * 32 + r) * 8) = make_uint4(w[0], w[1], w[2], w[3]);
    }
    const double total = prep_row_sum(mass, shd);
    if (threadIdx.x == 0 && b < B)
        out_scale[b] = total > 0.0 ? (float)((double)kOperandUnscale * (double)kOperandUnscale / total) : 0.f;
}

// P'[512 x 128] per workgroup: W wavefronts, wavefront w owns RB row blocks (32 positions each) and all four
// column blocks (32 target ids each) of the workgroup's column group, i.e. RB x 4 accumulator tiles of
// 32 x 32 fp32.  The kept slots are walked in stages of 64 (four MFMA steps):
//   * A records come straight from global memory (L2-resident: every workgroup walks the slots at the same pace),
//   * the 16 B records of a stage are fetched once per workgroup, parked in LDS (three buffers in turn) and read by all
//     wavefronts: the vector memory pipe of a CU could not feed every wavefront its own copy;
//   * requests run two (A) and three (B) stages ahead of the MFMAs; large batches use one wavefront per SIMD with
//     the whole register file (accumulators in the AGPR half), which halves the LDS reads per MFMA.
// With requests in one go at the head of a stage, and the stage's LDS writes, barrier and first reads at its end, the matrix pipe was
// busy 70 % of the clocks; spread between the MFMAs, with the barrier in mid-stage, 80 % (N = 256000, n = 32000, 512 positions: 11.55 ->
// 10.0 M clocks under the counters, at 1.60 -> 1.45 GHz: 7114 -> 6755 us a call of two).  The clock follows the power from here on.
// M is streamed from HBM exactly once when all positions fit one row of workgroups (B <= 512).
// Where there are fewer column groups than the chip has compute units, be it in the whole call or in its last round, the slots are
// split over blockIdx.z, in whole turns of six stages, and the partial products of the groups from group0 on go to `out` without
// their scale (split_stride apart).
// A record of M: read exactly once per launch, so it is loaded non-temporally and leaves the L2 to the A records,
// which every workgroup of an XCD reads again.
typedef unsigned u32x4_t __attribute__((ext_vector_type(4)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
__device__ __forceinline__ f16x8 load_once(const f16x8 *p)
{
    return __builtin_bit_cast(f16x8, __builtin_nontemporal_load((const u32x4_t *)p));
}

template <int W, int RB, bool SPLIT>
__global__ __launch_bounds__(W * 64) void exact_bf16_kernel(const uint16_t *Ap, const uint16_t *Mp, int KB, int KB_split, int group0,
                                                            int N, int B, const float *out_scale, float *out, int64_t ldo,
                                                            int64_t split_stride)
{
    constexpr int RPW = 16 / W;   // B records a wavefront fetches per stage
    __shared__ f16x8 bbuf[3][16][64];
    const int wid = __builtin_amdgcn_readfirstlane(threadIdx.x / kWave), lane = lane_id();
    const int jb0 = (group0 + blockIdx.x) * kColBlocksPerWg;
    const int rb0 = (blockIdx.y * W + wid) * RB;
    const int n_jb = (N + kColBlock - 1) / kColBlock;
    const int kb_first = blockIdx.z * KB_split;
    const int stages = min(KB_split, KB - kb_first) / 4;
    if (SPLIT) out += (int64_t)blockIdx.z * split_stride;
    f32x16 acc[RB][kColBlocksPerWg];
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < kColBlocksPerWg; ++c)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[r][c][v] = 0.f;

    const f16x8 *a_ptr[RB];   // the same for every lane, which adds its own place in a record
#pragma unroll
    for (int r = 0; r < RB; ++r) a_ptr[r] = (const f16x8 *)Ap + ((int64_t)(rb0 + r) * KB + kb_first) * 64;
    const f16x8 *b_src[RPW];
    int b_rec[RPW];
#pragma unroll
    for (int i = 0; i < RPW; ++i) {
        b_rec[i] = wid * RPW + i;                               // record = jb * 4 + kb within the stage
        const int jb = min(jb0 + b_rec[i] / 4, n_jb - 1);       // surplus column blocks recompute the last one
        b_src[i] = (const f16x8 *)Mp + ((int64_t)jb * KB + kb_first + b_rec[i] % 4) * 64;
    }
    // Loads return to a wavefront in issue order, so every load inherits the latency of the slowest one before
    // it.  The B records come from HBM: they are requested three stages ahead and kept in a ring of registers.
    // The A records (L2) are requested two stages ahead, block by block as their registers fall free; the only
    // B request older than an A record at the time it is needed is then two whole stages old.
    // The first requests are issued in the order the stages keep afterwards (A by slot block, at least as many
    // requests behind every record as in the steady state): the wait counts the compiler derives for the first stages
    // of the loop are the minimum over both ways into them, and a different order here would tighten them for good.
    f16x8 a_even[RB][4], a_odd[RB][4], b_ring[3][RPW];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
#pragma unroll
        for (int r = 0; r < RB; ++r) a_even[r][kb] = a_ptr[r][kb * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int i = 0; i < RPW; ++i) b_ring[t][i] = load_once(b_src[i] + (int64_t)min(t, stages - 1) * 4 * 64 + lane);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kb = 0; kb < (RB > 1 ? 3 : 4); ++kb)
#pragma unroll
        for (int r = 0; r < RB; ++r) a_odd[r][kb] = a_ptr[r][((int64_t)min(1, stages - 1) * 4 + kb) * 64 + lane];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < RPW; ++i) bbuf[0][b_rec[i]][lane] = b_ring[0][i];
    __syncthreads();
    f16x8 bq[4];   // B fragments are read from LDS two MFMA groups ahead
    bq[0] = bbuf[0][0][lane];
    bq[1] = bbuf[0][4][lane];

    // One stage: sixteen groups f = kb * 4 + c of RB MFMAs, and between the MFMAs of a group at most one request of each kind, so
    // that it is issued while an MFMA runs.  The registers of slot block kb fall free with its last group; they take the request
    // for the same block TWO stages ahead during the next slot block (those of the last one during the next stage: APREV), so
    // even and odd stages own one register set each.  SLOT = s % 3 is the ring entry free for the B request three stages ahead, and
    // the LDS buffer of this stage.  The next stage's B records go to LDS in the third slot block, the barrier that makes
    // them visible stands before the last one, and the first two fragments of the next stage are read behind it: no wavefront
    // waits for LDS between two stages.  All indices are clamped: no branches.
#define RDK_STAGE(SLOT, ACUR, APREV)                                                                                 \
    {                                                                                                                \
        const int64_t sp = (int64_t)min(s + 1, stages - 1) * 256, sa = (int64_t)min(s + 2, stages - 1) * 256;        \
        const int64_t sb = (int64_t)min(s + 3, stages - 1) * 256;                                                    \
        if (RB == 1) _Pragma("unroll") for (int i = 0; i < RPW; ++i) b_ring[SLOT][i] = load_once(b_src[i] + sb + lane); \
        __builtin_amdgcn_sched_barrier(0);                                                                           \
        _Pragma("unroll") for (int f = 0; f < 16; ++f) {                                                             \
            const int kb = f / 4, c = f % 4, nf = (f + 2) % 16;                                                      \
            if (f == 12) __syncthreads();                                                                            \
            _Pragma("unroll") for (int r = 0; r < RB; ++r) {                                                         \
                acc[r][c] = __builtin_amdgcn_mfma_f32_32x32x16_f16(ACUR[r][kb], bq[f % 4], acc[r][c], 0, 0, 0);     \
                __builtin_amdgcn_sched_barrier(0);                                                                   \
                if (r == 0) bq[(f + 2) % 4] = bbuf[f + 2 < 16 ? SLOT : (SLOT + 1) % 3][(nf % 4) * 4 + nf / 4][lane]; \
                if (RB == 1 && c == 3) ACUR[0][kb] = a_ptr[0][sa + kb * 64 + lane];                                  \
                if (RB > 1 && r == RB / 4 && c < RB) {                                                                   \
                    if (kb == 0) APREV[c][3] = a_ptr[c][sp + 3 * 64 + lane];                                         \
                    else ACUR[c][(kb + 3) % 4] = a_ptr[c][sa + (kb - 1) * 64 + lane];                                \
                }                                                                                                    \
                if (RB > 1 && r == RB / 2 && c == 2 && kb < RPW) b_ring[SLOT][kb % RPW] = load_once(b_src[kb % RPW] + sb + lane); \
                if (r == RB - 1 && kb == 2)                                                                          \
                    _Pragma("unroll") for (int i = c; i < RPW; i += 4) bbuf[(SLOT + 1) % 3][b_rec[i]][lane] = b_ring[(SLOT + 1) % 3][i]; \
                __builtin_amdgcn_sched_barrier(0);                                                                   \
            }                                                                                                        \
        }                                                                                                            \
        ++s;                                                                                                         \
    }
    // the number of stages is a multiple of six (the slot count is padded for it): six stages of straight-line code
    for (int s = 0; s < stages;) {
        RDK_STAGE(0, a_even, a_odd)
        RDK_STAGE(1, a_odd, a_even)
        RDK_STAGE(2, a_even, a_odd)
        RDK_STAGE(0, a_odd, a_even)
        RDK_STAGE(1, a_even, a_odd)
        RDK_STAGE(2, a_odd, a_even)
    }
#undef RDK_STAGE
    // D layout of the 32x32 tile: lane l holds column l % 32 and rows 8 * (v / 4) + 4 * (l / 32) + v % 4, v = 0..15
#pragma unroll
    for (int r = 0; r < RB; ++r)
#pragma unroll
        for (int c = 0; c < kColBlocksPerWg; ++c) {
            const int j = (jb0 + c) * kColBlock + (lane % 32);
            if (jb0 + c >= n_jb || j >= N) continue;
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int b = (rb0 + r) * 32 + 8 * (v / 4) + 4 * (lane / 32) + (v % 4);
                if (b >= B) continue;
                if (SPLIT) out[(int64_t)b * ldo + j - group0 * (kColBlocksPerWg * kColBlock)] = acc[r][c][v];
                else out[(int64_t)b * ldo + j] = acc[r][c][v] * out_scale[b];
            }
        }
}

// How the 16-bit product is cut: wavefronts per workgroup, row blocks per wavefront, and splits of the slots (KB_split slot
// blocks each, whole turns of six stages), as many as bring one workgroup to every compute unit.  A call, unsplit -> split:
// N = 8000, n = 2000: 8 positions 30.5 -> 21.8 us, 128: 38.8 -> 32.2, 512: 94.3 -> 57.9; N = 2000, 512 positions 59.6 -> 24.4;
// N = 16000, 256 positions 76.8 -> 70.9.  Two workgroups to a unit were slower (36.1 and 88.1 us at 128 and 256 positions).
// Small vocabularies take the smallest workgroups at any batch, several rows of them: M comes out of the caches again
// (N = 4000, 512 positions, one row of the largest workgroups split seven ways 46.2 us, four rows 33.3).
// Up to 64 positions a workgroup has 64 rows: with 128, half of them padding, the vector memory pipe brings as many bytes of A as
// of M.  128 rows -> 64, two calls with q' kept: N = 50000, n = 20000, 8 positions 460 -> 396 us, N = 20000, n = 6000, 30 90.5 ->
// 74.4, N = 8000, n = 2000, 8 28.2 -> 24.5, N = 110000, n = 20000, 64 896 -> 827.
// With more workgroups than the chip holds, the ones that are left for a last round would have it to themselves.  Up to half of the
// compute units they are split as above, in a launch of their own: N = 40000, n = 15000, 200 positions (57 of 313 left) 440 -> 350
// us, 480 769 -> 577, N = 100000, n = 15000, 512 (14 of 782) 1646 -> 1415; with 213 of 469 left there is nothing to split, and 248
// of the smallest ones of 1016 still draw as many bytes from HBM as the full chip (887 us, split 905).
// Of the workgroups of four wavefronts the chip holds two on a unit: 65 to 128 positions, unsplit -> split, n = 8000, 8 of 520 groups left
// 270 -> 229 us, 128 of 640 293 -> 277, 4 of 1028 478 -> 461.  A half round more, one for every unit, takes three quarters as long as
// a full one.  What is left behind it is split where the rows are long (100 positions, n = 9000: 2 of 770 left 437 -> 417, 62 of 830
// 445 -> 417, 112 of 880 455 -> 446; n = 16000: 716 -> 640, 736 -> 681, 128 of 896 763 -> 725) or where it is little (n = 5000: 2 of 770
// left 263 -> 247, 32 of 800 266 -> 258; but n = 4000, 112 of 880 222 -> 225, and n = 8000 383 -> 391, 402 -> 446).
constexpr int kSmallGroups = 64;
constexpr int kHalfRoundSlots = 9000, kHalfRoundFewSlots = 7000;
struct Bf16Shape {
    int W, RB, B_pad, groups, KB, KB_split, splits;
    int whole, tail_split, tail_splits;   // groups of full rounds; slot blocks and number of the splits of the ones after them
};

// Cuts KB slot blocks into at most `want` splits of whole turns.
void split_turns(int KB, int want, int *KB_split, int *splits)
{
    const int turns = KB / 24;
    if (want > turns) want = turns;
    if (want < 1) want = 1;
    const int per = (turns + want - 1) / want;
    *KB_split = per * 24;
    *splits = (turns + per - 1) / per;
}

Bf16Shape bf16_shape(const KernelHandle &h, int B)
{
    Bf16Shape s;
    s.groups = ((h.N + kColBlock - 1) / kColBlock + kColBlocksPerWg - 1) / kColBlocksPerWg;
    if (B <= 64) { s.W = 2; s.RB = 1; }
    else if (B <= 128 || s.groups <= kSmallGroups) { s.W = 4; s.RB = 1; }
    else if (B <= 256) { s.W = 8; s.RB = 1; }
    else { s.W = 4; s.RB = 4; }   // one wavefront per SIMD with all 512 registers: half the LDS reads per MFMA
    const int rows = s.W * s.RB * 32;
    s.B_pad = (B + rows - 1) / rows * rows;
    s.KB = h.n_pad / kKStep;
    split_turns(s.KB, kComputeUnits / (s.groups * (s.B_pad / rows)), &s.KB_split, &s.splits);
    s.whole = s.groups;
    s.tail_split = s.KB;
    s.tail_splits = 1;
    // workgroups that a compute unit holds: LDS three of two wavefronts, the registers two of four, and one of the others
    const int resident = (s.RB > 1 || s.W == 8 ? 1 : s.W == 4 ? 2 : 3) * kComputeUnits;
    int tail = s.groups % resident;
    bool cut = tail * 2 <= kComputeUnits;
    if (resident == 2 * kComputeUnits && tail > kComputeUnits) {
        tail -= kComputeUnits;
        cut = tail * 2 <= kComputeUnits && (h.n >= kHalfRoundSlots || (tail * 8 <= kComputeUnits && h.n <= kHalfRoundFewSlots));
    }
    if (rows == s.B_pad && s.groups > resident && tail > 0 && cut) {
        split_turns(s.KB, resident / tail, &s.tail_split, &s.tail_splits);
        if (s.tail_splits > 1) s.whole = s.groups - tail;
    }
    return s;
}

struct ExactWs {
    SoftStat *qstat;   // [B]
    float *part;       // fp32 path: [splits, B, N_ld]  (after the A records of that path)
    uint16_t *A;       // bf16 path: [B_pad, n_pad]
    float *out_scale;  // bf16 path: [B]
};

// Split of the slot blocks of the fp32 path: as many workgroups as the chip holds at one per compute unit but no more, so that
// they all run side by side (a few left over would have a second round to themselves); splits of a whole number of ring turns.
// A workgroup counts whole where its last wavefronts lie beyond N.  Splits counted by wavefronts, which leave up to 64 workgroups over
// where the 128-id tiles are no multiple of four -> this, the product's calls: N = 13000, n = 5000, 64 positions (260 workgroups -> 234)
// 110 -> 77 us, N = 5200, n = 2000, 256 (264 -> 220) 65 -> 47, N = 18600, n = 5000, 64 (259 -> 222) 145 -> 91, N = 9849, n = 2954, 8
// (260 -> 220) 45 -> 31.  blocks = slot blocks per split.
int split_splits(const KernelHandle &h, int B, int *blocks)
{
    const int groups = ((h.N + kSplitWaves * kColSet - 1) / (kSplitWaves * kColSet)) * ((B + kRowGroup - 1) / kRowGroup);
    const int kb_total = (h.n + kSplitStep - 1) / kSplitStep;
    int want = kComputeUnits / groups;
    const int maxs = (kb_total + 2 * kSplitRing - 1) / (2 * kSplitRing);    // at least 96 slots per split
    if (want > maxs) want = maxs;
    if (want > 64) want = 64;
    if (want < 1) want = 1;
    const int per = ((kb_total + want - 1) / want + kSplitRing - 1) / kSplitRing * kSplitRing;
    const int splits = (kb_total + per - 1) / per;
    if (blocks) *blocks = per;
    return splits;
}

// Rows of partial products are padded to whole quads.
int64_t padded(int N) { return (N + 3) / 4 * 4; }

rdk_status_t launch_reduce(const float *part, int splits, const SoftStat *qstat, const float *out_scale, int N, int B, float *out,
                           int64_t ldo, hipStream_t st)
{
    RDK_TIMED_LAUNCH("exact_reduce_kernel", exact_reduce_kernel, dim3((N + 1023) / 1024, B < 32768 ? B : 32768), dim3(256), 0, st, part,
                     padded(N), (int64_t)B * padded(N), splits, qstat, out_scale, N, B, out, ldo);
    RDK_LAUNCH_CHECK("exact_reduce_kernel");
    return RDK_OK;
}

template <int QK>
rdk_status_t run_exact(const KernelHandle &h, RowInput q, int32_t B, float *out, int64_t ldo, void *ws, hipStream_t st)
{
    char *p = (char *)ws;
    ExactWs w;
    w.qstat = (SoftStat *)p; p += align_up((size_t)B * sizeof(SoftStat), 256);
    if (h.format == RDK_DENSE_F32) {
        int blocks;
        const int splits = split_splits(h, B, &blocks);
        const int KB = splits * blocks;
        const int row_groups = (B + kRowGroup - 1) / kRowGroup;
        const int64_t records = (int64_t)row_groups * 2 * KB;   // of three parts each
        uint16_t *Ap = (uint16_t *)p; p += align_up((size_t)records * 3 * kWave * 8 * sizeof(uint16_t), 256);
        w.part = (float *)p;
        const int64_t ldd = padded(h.N);
        {
            if (h.n <= (QK == RDK_PROB_F32 ? kPrepRowMaxProb : kPrepRowMax)) {
                RDK_TIMED_LAUNCH("prep_a_split_kernel", (prep_a_split_kernel<QK>), dim3(row_groups * kRowGroup), dim3(kPrepThreads), 0, st,
                                 q.ptr, q.ld, w.qstat, h.n, B, KB, Ap);
            } else {
                const rdk_status_t rc = QK == RDK_PROB_F32 ? RDK_OK : launch_row_stats<QK>(q, h.n, B, 1, w.qstat, st);
                if (rc != RDK_OK) return rc;
                const int64_t threads = records * kWave;
                RDK_TIMED_LAUNCH("prep_a_split_kernel", (prep_a_records_kernel<QK>),
                                 dim3((unsigned)((threads + kStatThreads - 1) / kStatThreads + (QK == RDK_PROB_F32 ? B : 0))), dim3(kStatThreads), 0, st, q.ptr, q.ld, w.qstat, h.n, B, KB, records, Ap);
            }
        }
        RDK_LAUNCH_CHECK("prep_a_split_kernel");
        const int tile_groups = (h.N + kColSet * kSplitWaves - 1) / (kColSet * kSplitWaves);
        const dim3 grid((tile_groups * row_groups * splits + 7) / 8 * 8);
        const bool stream = row_groups == 1 && (size_t)h.n * h.ldm * sizeof(float) > kLastLevelBytes;
        const auto kernel = stream ? exact_f32_split_kernel<true> : exact_f32_split_kernel<false>;
        if (splits == 1) {
            RDK_TIMED_LAUNCH("exact_f32_split_kernel", kernel, grid, dim3(kSplitWaves * kWave), 0, st, Ap, h.dense,
                             h.ldm, h.n, h.N, B, KB, blocks, row_groups, splits, w.qstat, out, ldo, (int64_t)0, true);
            RDK_LAUNCH_CHECK("exact_f32_split_kernel");
        } else {
            RDK_TIMED_LAUNCH("exact_f32_split_kernel", kernel, grid, dim3(kSplitWaves * kWave), 0, st, Ap, h.dense,
                             h.ldm, h.n, h.N, B, KB, blocks, row_groups, splits, w.qstat, w.part, ldd, (int64_t)B * ldd, false);
            RDK_LAUNCH_CHECK("exact_f32_split_kernel");
            return launch_reduce(w.part, splits, w.qstat, nullptr, h.N, B, out, ldo, st);
        }
        return RDK_OK;
    }
    // bf16
    const Bf16Shape c = bf16_shape(h, B);
    const int KB = c.KB, B_pad = c.B_pad;
    w.A = (uint16_t *)p; p += align_up((size_t)B_pad * h.n_pad * 2, 256);
    w.out_scale = (float *)p; p += align_up((size_t)B * sizeof(float), 256);
    w.part = (float *)p;
    {
        RDK_TIMED_LAUNCH("prep_a_bf16_kernel", (prep_a_bf16_kernel<QK>), dim3(B_pad), dim3(kPrepThreads), 0, st, q.ptr, q.ld, h.row_sum, h.n, KB, B, w.A, w.out_scale);
    }
    RDK_LAUNCH_CHECK("prep_a_bf16_kernel");
#define RDK_BF16_LAUNCH(W, RB, SPLIT)                                                                                              \
    RDK_TIMED_LAUNCH("exact_bf16_kernel", (exact_bf16_kernel<W, RB, SPLIT>), grid, dim3(W * 64), 0, st, w.A, h.packed, KB, per, group0, \
                     h.N, B, w.out_scale, dst, ldd, stride)
    const auto product = [&](int group0, int groups, int per, int splits) {
        const dim3 grid(groups, B_pad / (c.W * c.RB * 32), splits);
        const bool split = splits > 1;
        const int j0 = group0 * kColBlocksPerWg * kColBlock;
        float *dst = split ? w.part : out;
        const int64_t ldd = split ? padded(h.N - j0) : ldo, stride = split ? (int64_t)B * ldd : 0;
        if (c.W == 2) {
            if (split) RDK_BF16_LAUNCH(2, 1, true);
            else RDK_BF16_LAUNCH(2, 1, false);
        } else if (c.W == 4 && c.RB == 1) {
            if (split) RDK_BF16_LAUNCH(4, 1, true);
            else RDK_BF16_LAUNCH(4, 1, false);
        } else if (c.W == 8) {
            if (split) RDK_BF16_LAUNCH(8, 1, true);
            else RDK_BF16_LAUNCH(8, 1, false);
        } else {
            if (split) RDK_BF16_LAUNCH(4, 4, true);
            else RDK_BF16_LAUNCH(4, 4, false);
        }
        RDK_LAUNCH_CHECK("exact_bf16_kernel");
        return split ? launch_reduce(w.part, splits, nullptr, w.out_scale, h.N - j0, B, out + j0, ldo, st) : RDK_OK;
    };
#undef RDK_BF16_LAUNCH
    const rdk_status_t rc = product(0, c.whole, c.KB_split, c.splits);
    return rc == RDK_OK && c.whole < c.groups ? product(c.whole, c.groups - c.whole, c.tail_split, c.tail_splits) : rc;
}

}  // namespace

size_t packed_bf16_bytes(int32_t n, int32_t N, int32_t *n_pad, int32_t *N_pad)
{
    const int32_t np = (n + 24 * kKStep - 1) / (24 * kKStep) * (24 * kKStep);   // six whole stages of four MFMA steps
    const int32_t Np = (N + kColBlock - 1) / kColBlock * kColBlock;
    if (n_pad) *n_pad = np;
    if (N_pad) *N_pad = Np;
    return (size_t)np * Np * 2;
}

size_t exact_workspace_bytes(const KernelHandle &h, int32_t B)
{
    size_t bytes = align_up((size_t)B * sizeof(SoftStat), 256);
    if (h.format == RDK_DENSE_F32) {
        int blocks;
        const int splits = split_splits(h, B, &blocks);
        const size_t records = (size_t)((B + kRowGroup - 1) / kRowGroup) * 2 * splits * blocks;
        bytes += align_up(records * 3 * kWave * 8 * sizeof(uint16_t), 256);
        if (splits > 1) bytes += align_up((size_t)splits * B * padded(h.N) * sizeof(float), 256);
    } else if (h.format == RDK_DENSE_BF16) {
        const Bf16Shape c = bf16_shape(h, B);
        bytes += align_up((size_t)c.B_pad * h.n_pad * 2, 256) + align_up((size_t)B * sizeof(float), 256);
        // A workspace for a batch serves every smaller one, so what is asked for must not fall as B grows: the rows of partial
        // products, splits * B, are at most B times the splits that one row of workgroups can have, and at most those splits of
        // a full one (its rows, 64 to 512, grow with B).
        const size_t splits = std::min<size_t>(c.KB / 24, kComputeUnits / c.groups), full = (size_t)c.W * c.RB * 32 * (kComputeUnits / c.groups);
        const size_t rows = splits > 1 ? std::min(B * splits, full) : 0;
        size_t partials = rows * padded(h.N);
        for (int b : {std::min(B, 64), std::min(B, 128), std::min(B, 256), std::min(B, 512)}) {   // the largest batches of each shape that has a tail
            const Bf16Shape t = bf16_shape(h, b);
            if (t.whole < t.groups)
                partials = std::max(partials, (size_t)t.tail_splits * b * padded(h.N - t.whole * kColBlocksPerWg * kColBlock));
        }
        bytes += align_up(partials * sizeof(float), 256);
    }
    return bytes;
}

rdk_status_t launch_pack_bf16(const float *M, int64_t ldm, int32_t n, int32_t N, uint16_t *packed, float *row_sum,
                              hipStream_t st)
{
    int32_t n_pad, N_pad;
    packed_bf16_bytes(n, N, &n_pad, &N_pad);
    const int KB = n_pad / kKStep;
    hipLaunchKernelGGL(pack_bf16_kernel, dim3(N_pad / kColBlock, KB < 64 ? KB : 64), dim3(64), 0, st, M, ldm, n, N, KB, packed);
    RDK_LAUNCH_CHECK("pack_bf16_kernel");
    hipLaunchKernelGGL(rounded_row_sum_kernel, dim3(n), dim3(256), 0, st, M, ldm, N, row_sum);
    RDK_LAUNCH_CHECK("rounded_row_sum_kernel");
    return RDK_OK;
}

rdk_status_t launch_unpack_bf16(const KernelHandle &h, float *M, int64_t ldm, hipStream_t st)
{
    const int KB = h.n_pad / kKStep;
    hipLaunchKernelGGL(unpack_bf16_kernel, dim3(h.N_pad / kColBlock, KB < 64 ? KB : 64), dim3(64), 0, st, h.packed, h.n, h.N,
                       KB, M, ldm);
    RDK_LAUNCH_CHECK("unpack_bf16_kernel");
    return RDK_OK;
}

rdk_status_t launch_exact(const KernelHandle &h, RowInput q, int32_t B, float *out, int64_t ldo, void *ws, hipStream_t st)
{
    switch (q.kind) {
        case RDK_PROB_F32: return run_exact<RDK_PROB_F32>(h, q, B, out, ldo, ws, st);
        case RDK_LOGIT_F32: return run_exact<RDK_LOGIT_F32>(h, q, B, out, ldo, ws, st);
        case RDK_LOGIT_BF16: return run_exact<RDK_LOGIT_BF16>(h, q, B, out, ldo, ws, st);
    }
    return RDK_ERR_DTYPE;
}

}  // namespace rdk
