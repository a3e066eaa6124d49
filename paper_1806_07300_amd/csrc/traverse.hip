// Traversal kernels for gfx950 and the fp_predict entry points.
//
//  naive_kernel    the baseline: one lane per observation, trees one after the
//                  other, every node (leaves included) fetched from memory in
//                  breadth-first order, features read from memory.  This is the
//                  GPU form of the BF layout the paper measures against.
//
//  packed_kernel   Forest Packing (Sec. III) on CDNA4, one forest:
//  batched_kernel  the same walk for many forests in one persistent launch.
//
// Packed walk.  A work unit is one (observation, tree) walk.  A workgroup owns
// a tile of R observations -- the feature columns some split tests are staged
// in LDS -- and the trees of one tree group, whose bins keep their interleaved
// top levels (Sec. III-A, Bin) in LDS.  The tile's R x trees units form a pool.
// Every lane keeps K walks in flight (Bin+, Sec. III-B): per step it issues
// its K node loads, then its K compares, so K independent fetches per lane
// overlap, as the paper's prefetch plus out-of-order execution does on a CPU.
// When walks end the wavefront refills all its empty cursors at once: lane 0
// reserves as many units as there are empty cursors with one LDS atomic, and
// every empty cursor takes base + (empty cursors on lower lanes), a
// ballot/mbcnt prefix.  No lane idles behind a long walk while units remain
// (the longest-path skew noted in Sec. IV-D).  Leaves are class references
// (DF-), so a walk ends without fetching a leaf; nodes below the interleaved
// levels follow the Stat order.  Votes are LDS atomics per (observation,
// class), then stored, or added into global memory with integer atomics when
// several tree groups share the rows (order-independent: still exact).
//
// Split test everywhere: x <= threshold in fp32 (v_cmp_le_f32; NaN -> right).
// The CLUSTERED 48-byte form, whose thresholds are all exact in fp16, stages
// the tile as fp16 values rounded toward +infinity and compares in fp16
// (v_cmpx_nle_f16), which decides every test exactly as the fp32 compare: for
// t exact in fp16, x <= t exactly when the smallest fp16 value >= x is <= t.
// Blocks are walked in a form of their own, made when a forest is uploaded
// (WalkForm in fp_internal.h, walk_form_kernel).
// Built without fast-math and without denormal flushing.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <type_traits>

#include "fp_internal.h"

using fp::BinEntry;
using fp::JobDesc;
using fp::Node16;
using fp::WorkItem;

namespace {

constexpr int32_t kDone = INT32_MIN;
// Idle lanes of a wavefront that trigger a refill.  A block step is long and
// a refill adds two LDS round trips to it: later refills pay (40,000 rows x
// 1,024 trees: at 16 lanes 342 us, at 48 308; 10^6 rows x 32 trees 245 and
// 230); node steps are short (2,000 rows x 64 trees: 52 and 59 us).
constexpr int kDefaultRefillLanes = 16, kDefaultRefillLanesBlocks = 48, kDefaultRefillLanesDrift = 24;
constexpr double kDriftDepth = 21.5;  // levels of an average walk (see resolve_job)
// Rows of an automatic tile whose features stay in memory: the rows of a tile
// are read from L1, which holds few (30,000 image rows x 128 trees: 16-row
// tiles 340 us, 118-row ones 1420).
constexpr int kMemoryTileRows = 16;
// Levels below a bin's top region from which on PACKED nodes are fetched in
// pairs (run_tile): in launches of their own (100,000 rows in 64-row tiles: 128
// trees of depth 10 single 191 us, pairs 188, 768 trees of depth 9 823 and
// 997), in those too small to hide one walk's latency behind another's (few
// walks, or few threads a workgroup: 4,000 rows, depth 10, 256 threads: 36 and
// 43), and in launches that share the device, with their small tiles and two
// cursors (16 forests of depth 8 to 12 in one plan: from 3 levels on 701 us,
// from 5 on 761).
constexpr double kPairDepth = 7.0, kPairDepthIdle = 8.5, kPairDepthShared = 3.0;
constexpr int kStageBatch = 4;  // row loads a thread issues before scattering them (tile staging)

// ---------------------------------------------------------------------------
// naive kernel
// ---------------------------------------------------------------------------
struct NaiveArgs {
    const int64_t* tree_off;
    const Node16* nodes;
    const float* X;
    int64_t ld;
    int64_t n_rows;
    int32_t* votes;
    int32_t* cls;
    int32_t n_trees, C;
};

// Leaf statistics from observations (Sec. III-A: the access statistics Stat
// orders by may be inferred after training from a set of observations): one
// lane per observation walks every tree of a NAIVE-layout forest and adds one
// to the counter of the leaf it reaches (position in the layout).  Grid-stride
// over rows; integer atomics, so the counts are exact and order-independent.
__global__ __launch_bounds__(256) void leaf_count_kernel(const Node16* __restrict__ nodes,
                                                         const int64_t* __restrict__ tree_off, int32_t n_trees,
                                                         const float* __restrict__ X, int64_t n_rows, int64_t ld,
                                                         int32_t* __restrict__ counts) {
    for (int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; row < n_rows;
         row += (int64_t)gridDim.x * blockDim.x) {
        const float* x = X + row * ld;
        for (int32_t t = 0; t < n_trees; t++) {
            const Node16* tn = nodes + tree_off[t];
            int32_t n = 0;
            while (true) {  // a verified buffer's children come after their parent: the walk ends
                const Node16 nd = tn[n];
                if (nd.feat < 0) break;
                n = x[nd.feat] <= nd.thr ? nd.left : nd.right;
            }
            atomicAdd(&counts[tree_off[t] + n], 1);
        }
    }
}

template <bool LDS_VOTES>
__global__ __launch_bounds__(1024) void naive_kernel(NaiveArgs a) {
    extern __shared__ int32_t vl[];  // [C][blockDim] when LDS_VOTES
    const int64_t row = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    const bool live = row < a.n_rows;
    const int bd = blockDim.x, tid = threadIdx.x;
    int32_t* vg = a.votes + (live ? row : 0) * a.C;
    if (LDS_VOTES) {
        for (int c = 0; c < a.C; c++) vl[c * bd + tid] = 0;
    } else if (live) {
        for (int c = 0; c < a.C; c++) vg[c] = 0;
    }
    if (live) {
        const float* x = a.X + row * a.ld;
        for (int32_t t = 0; t < a.n_trees; t++) {
            const Node16* tn = a.nodes + a.tree_off[t];
            int32_t n = 0;
            while (true) {
                const Node16 nd = tn[n];
                if (nd.feat < 0) {
                    if (LDS_VOTES) vl[nd.left * bd + tid] += 1;
                    else vg[nd.left] += 1;
                    break;
                }
                n = (x[nd.feat] <= nd.thr) ? nd.left : nd.right;
            }
        }
        int32_t best = 0, bestv = INT_MIN;
        for (int c = 0; c < a.C; c++) {
            const int32_t v = LDS_VOTES ? vl[c * bd + tid] : vg[c];
            if (LDS_VOTES) vg[c] = v;
            if (v > bestv) { bestv = v; best = c; }
        }
        if (a.cls) a.cls[row] = best;
    }
}

// ---------------------------------------------------------------------------
// packed walk: device pieces shared by the single-forest and batched kernels
// ---------------------------------------------------------------------------
__device__ __forceinline__ int lane_id() { return __builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u)); }
__device__ __forceinline__ int bits_below(uint64_t m) {
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
}

// Unit u of a tile is (tree u / rows, row u % rows).  The division uses a
// 32-bit reciprocal m = floor((2^32 - 1) / rows): umulhi(u, m) is the
// quotient or one less for any u < 2^32, so one correction step is exact.
__device__ __forceinline__ uint32_t div_rows(uint32_t u, uint32_t rows, uint32_t m, uint32_t& rem) {
    uint32_t q = __umulhi(u, m);
    uint32_t r = u - q * rows;
    if (r >= rows) {
        q += 1;
        r -= rows;
    }
    rem = r;
    return q;
}

// Hands the idle cursors of a wavefront new units from the workgroup pool:
// per cursor slot one LDS atomic by lane 0 reserves as many units as there
// are idle lanes, and each idle lane takes base + (idle lanes below it).  A
// slot is refilled only once at least `min_idle` lanes have it idle, or when
// nothing in the wavefront is live, so most steps skip the refill's
// instructions.  take(k, row, ttab entry) sets cursor k up and returns its
// first reference, or kDone after voting when the tree's root is a leaf (the
// lane then stays idle and takes another unit).
template <int K, typename Take>
__device__ __forceinline__ void refill(int32_t (&ref)[K], int32_t* pool, int U, uint32_t rows, uint32_t rmagic,
                                       const int4* ttab, int min_idle, int lane, bool& drained, Take&& take) {
    uint64_t live = 0;
#pragma unroll
    for (int k = 0; k < K; k++) live |= __ballot(ref[k] >= 0);
#pragma unroll
    for (int k = 0; k < K; k++) {
        while (!drained) {
            const uint64_t m = __ballot(ref[k] < 0);
            const int cnt = (int)__popcll(m);
            if (cnt == 0 || (cnt < min_idle && live != 0)) break;
            int base = 0;
            if (lane == 0) base = atomicAdd(pool, cnt);
            base = __builtin_amdgcn_readfirstlane(base);
            if (base >= U) {
                drained = true;
                break;
            }
            if (ref[k] < 0) {
                const uint32_t u = (uint32_t)(base + bits_below(m));
                if (u < (uint32_t)U) {
                    uint32_t r;
                    const uint32_t t = div_rows(u, rows, rmagic, r);
                    ref[k] = take(k, (int)r, ttab[t]);
                }
            }
            if (base + cnt >= U) drained = true;
        }
    }
}

// fp16 bits (low half of each result) of the smallest fp16 values >= a, b,
// c, d (round toward +infinity; NaN stays NaN, beyond the fp16 range +inf
// or -65504): the wave's round mode for fp16 results (MODE bits 3:2) is set
// to +infinity for the four conversions and back to nearest-even, the
// kernel's mode, after them, inside one block so that no other instruction
// runs in between.
__device__ __forceinline__ void half_up4(float a, float b, float c, float d, uint32_t (&h)[4]) {
    asm volatile(
        "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 1\n\t"
        "s_nop 1\n\t"
        "v_cvt_f16_f32 %0, %4\n\t"
        "v_cvt_f16_f32 %1, %5\n\t"
        "v_cvt_f16_f32 %2, %6\n\t"
        "v_cvt_f16_f32 %3, %7\n\t"
        "s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 0"
        : "=&v"(h[0]), "=&v"(h[1]), "=&v"(h[2]), "=&v"(h[3])
        : "v"(a), "v"(b), "v"(c), "v"(d));
}
// The same for one value without touching the round mode (the column-wise
// staging path): the nearest-even conversion, moved up one step when it fell
// below x.  Stepping the bits up a positive value, or down a negative one,
// gives the next larger value, and -0 steps to the smallest subnormal.
__device__ __forceinline__ uint16_t half_up(float x) {
    const _Float16 h = (_Float16)x;
    uint32_t b = __builtin_bit_cast(uint16_t, h);
    if ((float)h < x) b = (b & 0x8000u) ? (b == 0x8000u ? 1u : b - 1u) : b + 1u;
    return (uint16_t)b;
}

// Stores one staged feature: fp32, or fp16 bits already rounded up.
template <bool X16>
__device__ __forceinline__ void put_feature(void* row, int c, float v, uint32_t h) {
    if constexpr (X16) static_cast<uint16_t*>(row)[c] = (uint16_t)h;
    else static_cast<float*>(row)[c] = v;
}

// Rows of the tile that starts at row0.
__device__ __forceinline__ int tile_rows(const JobDesc& j, int64_t row0) { return (int)min<int64_t>(j.R, j.n_rows - row0); }

// Whole-row staging: quad (four columns) qd of row r goes to thread
// (r Q + qd) mod blockDim.  The thread's first quad of a tile, issued ahead
// of the staging of its group so that the two wait for memory together;
// stage_tile takes it over.
template <int FMODE>
__device__ __forceinline__ float4 prefetch_quad(const JobDesc& j, int tile) {
    float4 v = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if (FMODE != 1 || !j.stage_rows || tile >= j.n_tiles) return v;
    const int Q = (j.F + 3) / 4, r = (int)threadIdx.x / Q, qd = (int)threadIdx.x - r * Q;
    const int64_t row0 = (int64_t)tile * j.R;
    if (r < tile_rows(j, row0)) v = reinterpret_cast<const float4*>(j.X + (row0 + r) * j.ld)[qd];
    return v;
}

// Copies the used feature columns of tile rows [row0, row0 + rows) into LDS
// (fp32 row-major, row stride Fcp; or, when X16, fp16 feature-major, feature
// stride Fcp, so that lanes reading one feature of consecutive rows share
// LDS words), clears
// the tile's vote counters and the unit pool, then synchronises.  kStageBatch
// independent 16-byte loads of a thread are in flight before their scatter.
// prefetched: the thread's first quad is `pre`.
template <bool X16 = false>
__device__ __forceinline__ void stage_tile(const JobDesc& j, float* xs, int32_t* vl, int32_t* pool, int64_t row0,
                                           int rows, bool feat_lds, float4 pre, bool prefetched) {
    const int tid = threadIdx.x, bd = blockDim.x;
    for (int i = tid; i < rows * j.C; i += bd) vl[i] = 0;
    if (tid == 0) *pool = 0;
    if (feat_lds && j.stage_rows) {
        // whole rows in 16-byte loads; each used column goes to its compacted
        // slot (imap, 4 entries per 8-byte LDS read; -1 = unused), or, when
        // every column is used, to its own place
        const int16_t* imap = reinterpret_cast<const int16_t*>(reinterpret_cast<const unsigned char*>(xs) - j.off_xs +
                                                               j.off_imap);
        auto scatter = [&](int r, int qd, float4 v) {
            int m0 = 4 * qd, m1 = m0 + 1, m2 = m0 + 2, m3 = m0 + 3;
            if (j.Fc < j.F) {
                const int2 m = *reinterpret_cast<const int2*>(imap + m0);
                m0 = (int16_t)(m.x & 0xFFFF);
                m1 = m.x >> 16;
                m2 = (int16_t)(m.y & 0xFFFF);
                m3 = m.y >> 16;
            } else if (m3 >= j.F) {  // the last quad of a row: columns past the features
                m1 = m1 < j.F ? m1 : -1;
                m2 = m2 < j.F ? m2 : -1;
                m3 = -1;
            }
            // fp32: row r, element m; fp16: element m * Fcp of row r
            void* dst = X16 ? static_cast<void*>(reinterpret_cast<uint16_t*>(xs) + r) : static_cast<void*>(xs + r * j.Fcp);
            const int es = X16 ? j.Fcp : 1;
            uint32_t h[4] = {0, 0, 0, 0};
            if constexpr (X16) half_up4(v.x, v.y, v.z, v.w, h);
            if (m0 >= 0) put_feature<X16>(dst, m0 * es, v.x, h[0]);
            if (m1 >= 0) put_feature<X16>(dst, m1 * es, v.y, h[1]);
            if (m2 >= 0) put_feature<X16>(dst, m2 * es, v.z, h[2]);
            if (m3 >= 0) put_feature<X16>(dst, m3 * es, v.w, h[3]);
        };
        const int Q = (j.F + 3) / 4;
        const int dq = bd / Q, dc = bd - dq * Q;
        int r = tid / Q, qd = tid - r * Q;
        auto step = [&]() {  // to the thread's next quad
            r += dq;
            qd += dc;
            if (qd >= Q) {
                qd -= Q;
                r += 1;
            }
        };
        if (prefetched) {
            if (r < rows) scatter(r, qd, pre);
            step();
        }
        const int64_t ld4 = j.ld / 4;
        const float4* x0 = reinterpret_cast<const float4*>(j.X + row0 * j.ld);
        while (r < rows) {
            float4 v[kStageBatch];
            int rr[kStageBatch], qq[kStageBatch];
#pragma unroll
            for (int u = 0; u < kStageBatch; u++) {
                rr[u] = r;
                qq[u] = qd;
                if (r < rows) v[u] = x0[r * ld4 + qd];
                step();
            }
#pragma unroll
            for (int u = 0; u < kStageBatch; u++) {
                if (rr[u] >= rows) break;
                scatter(rr[u], qq[u], v[u]);
            }
        }
    } else if (feat_lds) {
        // element i = r * Fc + c goes to thread i mod blockDim
        const int Fc = j.Fc;
        const int dq = bd / Fc, dc = bd - dq * Fc;
        int r = tid / Fc, c = tid - r * Fc;
        const float* xrow = j.X + (row0 + r) * j.ld;
        const int64_t dld = (int64_t)dq * j.ld;
#pragma unroll 4
        while (r < rows) {
            if constexpr (X16) reinterpret_cast<uint16_t*>(xs)[c * j.Fcp + r] = half_up(xrow[j.fmap[c]]);
            else xs[r * j.Fcp + c] = xrow[j.fmap[c]];
            r += dq;
            xrow += dld;
            c += dc;
            if (c >= Fc) {
                c -= Fc;
                r += 1;
                xrow += j.ld;
            }
        }
    }
    __syncthreads();
}

// After the walks of a tile: stores its vote counters (or adds them into the
// global votes when several tree groups share the rows), then the class of
// each row (lowest class on ties) when this workgroup saw every tree.  In a
// later pass (accumulate) each thread owns whole rows: it adds the tile's
// counters to the stored votes and, in the last pass (cls set), takes the
// class from the sums; no other workgroup touches these rows in the launch.
__device__ __forceinline__ void write_tile(const JobDesc& j, const int32_t* vl, int64_t row0, int rows) {
    const int tid = threadIdx.x, bd = blockDim.x;
    __syncthreads();
    if (j.accumulate) {
        for (int rr = tid; rr < rows; rr += bd) {
            int32_t* dst = j.votes + (row0 + rr) * j.C;
            int32_t best = 0, bestv = INT_MIN;
            for (int c = 0; c < j.C; c++) {
                const int32_t v = dst[c] + vl[rr * j.C + c];
                dst[c] = v;
                if (v > bestv) {
                    bestv = v;
                    best = c;
                }
            }
            if (j.cls) j.cls[row0 + rr] = best;
        }
        __syncthreads();
        return;
    }
    for (int i = tid; i < rows * j.C; i += bd) {
        int32_t* dst = j.votes + row0 * j.C + i;
        if (j.atomic_votes) {
            if (vl[i]) atomicAdd(dst, vl[i]);
        } else {
            *dst = vl[i];
        }
    }
    if (!j.atomic_votes && j.cls) {
        const int C = j.C;
        for (int rr = tid; rr < rows; rr += bd) {
            const int32_t* of = vl + rr * C;
            int32_t best = 0, bestv = of[0];
            int c = 1;
            // four reads in flight: one at a time, an LDS round trip per class is all that a tile of
            // many classes takes (one row x 1,000 classes: 47 us, now 31)
            for (; c + 4 <= C; c += 4) {
                const int32_t v[4] = {of[c], of[c + 1], of[c + 2], of[c + 3]};
#pragma unroll
                for (int i = 0; i < 4; i++) {
                    best = v[i] > bestv ? c + i : best;
                    bestv = max(v[i], bestv);
                }
            }
#pragma unroll 1
            for (; c < C; c++) {
                best = of[c] > bestv ? c : best;
                bestv = max(of[c], bestv);
            }
            j.cls[row0 + rr] = best;
        }
    }
    __syncthreads();
}

// A tile's observations as the walks see them: feature f of tile row r
// (staged in LDS, or read from memory through the feature map) and the LDS
// vote counters of row r.  Row offsets use 24-bit multiplies (full rate;
// rows < 4096 and columns, classes < 2^24).
struct TileRows {
    const JobDesc& j;
    const float* xs;
    int32_t* vl;
    const int32_t* fmap_l;
    int64_t row0;
    bool feat_lds;
    __device__ __forceinline__ float x(int r, uint32_t f) const {
        return feat_lds ? xs[__umul24((uint32_t)r, (uint32_t)j.Fcp) + f] : j.X[(row0 + r) * j.ld + fmap_l[f]];
    }
    __device__ __forceinline__ void vote(int r, int32_t cls) const {
        atomicAdd(&vl[__umul24((uint32_t)r, (uint32_t)j.C) + (uint32_t)cls], 1);
    }
};

// What a kernel walks: a node layout (PACKED nodes one by one or in pairs),
// blocks in their host form, or blocks in
// a walk form (with an fp16 tile: X); one kernel each, so that a launch
// fetches only its own code and the compiler knows the block's shape.
// kKindAnyNode, kKindAnyBlock: decided per job (batched launches).
enum Kind : int {
    kKindPacked, kKindCompact, kKindHost48, kKindHost64, kKind64, kKind48h, kKind48hX, kKind48b, kKind48f, kKind32h,
    kKind32hX, kKindPairs, kKindAnyNode, kKindAnyBlock
};
constexpr int32_t kind_form(int kind) {
    return kind == kKind64                           ? (int32_t)fp::kWalk64
           : kind == kKind48h || kind == kKind48hX   ? (int32_t)fp::kWalk48h
           : kind == kKind48b                        ? (int32_t)fp::kWalk48b
           : kind == kKind48f                        ? (int32_t)fp::kWalk48f
           : kind == kKind32h || kind == kKind32hX   ? (int32_t)fp::kWalk32h
                                                     : (int32_t)fp::kWalkNone;
}
__host__ __device__ __forceinline__ int job_kind(const JobDesc& j) {
    return j.layout == FP_LAYOUT_COMPACT       ? kKindCompact
           : j.layout < FP_LAYOUT_BLOCKED      ? (j.block_bytes == 2 * (int)sizeof(Node16) ? kKindPairs : kKindPacked)
           : j.form == fp::kWalk64             ? kKind64
           : j.form == fp::kWalk48h            ? (j.x16 ? kKind48hX : kKind48h)
           : j.form == fp::kWalk48b            ? kKind48b
           : j.form == fp::kWalk48f            ? kKind48f
           : j.form == fp::kWalk32h            ? (j.x16 ? kKind32hX : kKind32h)
           : j.block_bytes == 48               ? kKindHost48
                                               : kKindHost64;
}

// LDS and global pointers are typed with their address spaces so that the
// compiler keeps an LDS read and a global load apart rather than merging them
// into one flat load through a selected pointer.
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) const u32x4 lds_u32x4;
typedef __attribute__((address_space(1))) const u32x4 global_u32x4;

__device__ __forceinline__ uint4 as_uint4(u32x4 v) { return make_uint4(v.x, v.y, v.z, v.w); }

// LDS byte address of a pointer into the workgroup's shared memory, and back.
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(size_t)(__attribute__((address_space(3))) const void*)p;
}
template <typename T>
__device__ __forceinline__ __attribute__((address_space(3))) const T* lds_ptr(uint32_t a) {
    return (__attribute__((address_space(3))) const T*)(size_t)a;
}


// The base of a block in a walk form, in the piece that holds it (the last
// one, with the targets), and that piece with another base.
__device__ __forceinline__ uint32_t piece_base(int32_t form, const uint4& p) {
    return form == fp::kWalk32h                          ? (p.w >> 8) & 0xFFFFFu
           : form == fp::kWalk48h                        ? p.x
           : form == fp::kWalk48b                        ? p.y
                                                         : p.w;
}
__device__ __forceinline__ void set_piece_base(int32_t form, uint4& p, uint32_t base) {
    if (form == fp::kWalk32h) p.w = (p.w & ~0x0FFFFF00u) | base << 8;
    else if (form == fp::kWalk48h) p.x = base;
    else if (form == fp::kWalk48b) p.y = base;
    else p.w = base;
}
// Stage the bin tops, the tree table and (when features are read from memory)
// the feature map of tree group `group`; returns the group's tree count.
// The caller must have synchronised since the previous use of LDS.
template <int KIND>
__device__ __forceinline__ int stage_group(const JobDesc& j, int group, unsigned char* smem) {
    const int tid = threadIdx.x, bd = blockDim.x;
    const int b_lo = group * j.bins_per_group;
    const int b_hi = min(b_lo + j.bins_per_group, j.n_bins);
    if (b_lo >= b_hi) return 0;
    uint4* top = reinterpret_cast<uint4*>(smem);
    int4* ttab = reinterpret_cast<int4*>(smem + j.off_ttab);
    const int t_lo = b_lo * j.bin_size;
    const int nt = (int)min((int64_t)b_hi * j.bin_size, (int64_t)j.n_trees) - t_lo;
    constexpr bool any = KIND == kKindAnyNode || KIND == kKindAnyBlock;
    constexpr bool blk = KIND != kKindPacked && KIND != kKindPairs && KIND != kKindCompact && KIND != kKindAnyNode;
    const int32_t form = KIND == kKindAnyBlock ? j.form : kind_form(KIND);
    // PACKED: the bin's top nodes; block layouts: its first blocks (roots
    // first), as 16-byte pieces; cap pieces per bin
    const int bw = !blk ? 1 : any || form == fp::kWalkNone ? j.block_bytes / 16 : fp::walk_shape(form).bytes / 16;
    const int per = form == fp::kWalk32h ? 2 : 1;  // pieces a walk reference counts
    // Each table's loads are issued a round ahead: the first round's (tree
    // roots, their bins, the pieces' bins) go out together before any is used.
    const int pieces = (b_hi - b_lo) * j.cap;
    const uint32_t capm = 0xFFFFFFFFu / (uint32_t)max(j.cap, 1), binm = 0xFFFFFFFFu / (uint32_t)j.bin_size;
    uint32_t rem;
    auto bin_of_piece = [&](int i) { return j.bins[b_lo + (int)div_rows((uint32_t)i, (uint32_t)j.cap, capm, rem)]; };
    auto bin_of_tree = [&](int tl) { return j.bins[b_lo + (int)div_rows((uint32_t)tl, (uint32_t)j.bin_size, binm, rem)]; };
    BinEntry pe, te;
    int32_t root = 0;
    if (tid < pieces) pe = bin_of_piece(tid);
    if (tid < nt) {
        te = bin_of_tree(tid);
        root = j.roots[t_lo + tid];
    }
    for (int i = tid; i < pieces; i += bd) {
        uint32_t k;
        const int bl = (int)div_rows((uint32_t)i, (uint32_t)j.cap, capm, k);
        if (i != tid) pe = bin_of_piece(i);
        const int32_t have = min(blk ? pe.deep_len * bw : pe.top_len, j.cap);
        const int64_t first = blk ? pe.node_base / 2 : pe.node_base;
        if ((int)k >= have) continue;
        uint4 p = reinterpret_cast<const uint4*>(j.nodes)[first + k];
        if (form != fp::kWalkNone && (int)k % bw == bw - 1) {
            // a child group (up to eight blocks) that is copied too is named by its LDS address
            const int32_t child = ((int32_t)piece_base(form, p) - fp::kGlobalRef - (int32_t)(first / per)) * per;
            if (child + 8 * bw <= have)
                set_piece_base(form, p, (lds_addr(top) / 16u + (uint32_t)(bl * j.cap + child)) / (uint32_t)per);
        }
        top[i] = p;
    }
    for (int tl = tid; tl < nt; tl += bd) {
        if (tl != tid) {
            te = bin_of_tree(tl);
            root = j.roots[t_lo + tl];
        }
        const int bl = (int)div_rows((uint32_t)tl, (uint32_t)j.bin_size, binm, rem);
        const int32_t nb = (int32_t)te.node_base;
        if (form != fp::kWalkNone) {
            const int32_t at = root * bw;
            reinterpret_cast<int32_t*>(ttab)[tl] =
                root < 0                                  ? root
                : at + bw <= min(te.deep_len * bw, j.cap) ? ((int32_t)(lds_addr(top) / 16u) + bl * j.cap + at) / per
                                                          : fp::kGlobalRef + (int32_t)((te.node_base / 2 + at) / per);
            continue;
        }
        ttab[tl] = (any ? j.layout == FP_LAYOUT_COMPACT : KIND == kKindCompact)
                       ? make_int4(root, nb, te.top_len, 0)
                   : blk ? make_int4(root, nb, bl * j.cap, min(te.deep_len, j.cap / max(bw, 1)))
                         : make_int4(root, nb, bl * j.cap, min(te.top_len, j.cap));
    }
    if (!j.feat_lds) {
        int32_t* fmap_l = reinterpret_cast<int32_t*>(smem + j.off_fmap);
        for (int c = tid; c < j.Fc; c += bd) fmap_l[c] = j.fmap[c];
    }
    if (j.stage_rows && j.Fc < j.F) {
        int16_t* imap = reinterpret_cast<int16_t*>(smem + j.off_imap);
        const int n_imap = (j.F + 3) / 4 * 4;
        for (int c = tid; c < n_imap; c += bd) imap[c] = -1;
        __syncthreads();
        for (int i = tid; i < j.Fc; i += bd) imap[j.fmap[i]] = (int16_t)i;
        __syncthreads();  // the first tile's staging reads imap
    }
    return nt;
}

// FMODE: 0 features from memory, 1 features in LDS, 2 decided by j.feat_lds.
// PAIRS: a deep node is fetched with the one that follows it in Stat order,
// the likely next of its walk: a line fetched from beyond L1 costs 2.4 cycles
// of the CU (L2) to 11 (beyond), a further 16 bytes of it 0.7 (100,003 rows x
// 64 trees at their best tiles: single nodes 238 us, two 214, three 239, four
// 253; 2,000 rows: 18.0, 15.2, 14.6, 15.0).  Only where walks go on deep below
// staged top nodes and features are in LDS (resolve_job): 100,000 rows x 600
// trees of depth 6, 64-row tiles: single 523 us, pairs 814; features in
// memory, 128 trees of depth 10: 650 and 821.  Four cursors or more per lane
// have no registers for it.
template <int K, int FMODE, bool PAIRS>
__device__ __forceinline__ void run_tile(const JobDesc& j, int nt, int tile, unsigned char* smem) {
    constexpr int kRun = PAIRS ? 2 : 1;
    const bool feat_lds = FMODE == 2 ? (j.feat_lds != 0) : (FMODE == 1);
    const Node16* top = reinterpret_cast<const Node16*>(smem);
    const int4* ttab = reinterpret_cast<const int4*>(smem + j.off_ttab);
    const int32_t* fmap_l = reinterpret_cast<const int32_t*>(smem + j.off_fmap);
    float* xs = reinterpret_cast<float*>(smem + j.off_xs);
    int32_t* vl = reinterpret_cast<int32_t*>(smem + j.off_votes);
    int32_t* pool = reinterpret_cast<int32_t*>(smem + j.off_pool);
    const int lane = lane_id();

    const int64_t row0 = (int64_t)tile * j.R;
    const int rows_here = tile_rows(j, row0);

    const int U = rows_here * nt;
    const uint32_t rmagic = 0xFFFFFFFFu / (uint32_t)rows_here;
    TileRows tr{j, xs, vl, fmap_l, row0, feat_lds};
    const uint32_t f_max = (uint32_t)(j.Fc - 1);
    // per cursor: row in the tile, gb = bin base in the node array, lb = the
    // bin's first top node in LDS, cp = top nodes staged in LDS
    int32_t ref[K], rowk[K], gb[K], lb[K], cp[K];
#pragma unroll
    for (int k = 0; k < K; k++) { ref[k] = kDone; rowk[k] = 0; gb[k] = 0; lb[k] = 0; cp[k] = 0; }
    auto take = [&](int k, int r, int4 e) -> int32_t {
        rowk[k] = r; gb[k] = e.y; lb[k] = e.z; cp[k] = e.w;
        if (e.x < 0) {  // the root is a leaf
            tr.vote(r, -e.x - 1);
            return kDone;
        }
        return e.x;
    };
    bool drained = false;
    while (true) {
        if (!drained) refill<K>(ref, pool, U, (uint32_t)rows_here, rmagic, ttab, j.refill_min, lane, drained, take);
        bool live = false;
#pragma unroll
        for (int k = 0; k < K; k++) live |= ref[k] >= 0;
        if (__ballot(live) == 0) {
            if (drained) break;
            continue;
        }
        // a top node from LDS, or kRun consecutive nodes from memory (the last
        // node of the section repeated past its end)
        Node16 nd[K][kRun];
#pragma unroll
        for (int k = 0; k < K; k++)
            if (ref[k] >= 0 && ref[k] < cp[k]) nd[k][0] = top[lb[k] + ref[k]];
#pragma unroll
        for (int k = 0; k < K; k++)
            if (ref[k] >= 0 && ref[k] >= cp[k]) {
#pragma unroll
                for (int i = 0; i < kRun; i++) nd[k][i] = j.nodes[i == 0 ? gb[k] + ref[k] : min(gb[k] + ref[k] + i, j.n_nodes - 1)];
            }
#pragma unroll
        for (int k = 0; k < K; k++) {
            if (ref[k] >= 0) {
                int32_t nr = (tr.x(rowk[k], nd[k][0].feat) <= nd[k][0].thr) ? nd[k][0].left : nd[k][0].right;
                if (kRun > 1 && ref[k] >= cp[k]) {
                    // children come after their parent: one pass over the run follows the walk through it.
                    // A node that the walk does not reach may be a gap behind a bin, whose content the
                    // verifier does not look at: its feature is held inside the row
                    int32_t to[kRun];
#pragma unroll
                    for (int i = 1; i < kRun; i++)
                        to[i] = (tr.x(rowk[k], (int32_t)min((uint32_t)nd[k][i].feat, f_max)) <= nd[k][i].thr) ? nd[k][i].left
                                                                                                           : nd[k][i].right;
#pragma unroll
                    for (int i = 1; i < kRun; i++) nr = nr == ref[k] + i ? to[i] : nr;
                }
                if (nr < 0) {
                    tr.vote(rowk[k], -nr - 1);
                    nr = kDone;
                }
                ref[k] = nr;
            }
        }
    }
    write_tile(j, vl, row0, rows_here);
}

// COMPACT layout walk.  Top nodes (Node16) come from memory (L1/L2); a deep
// node is fetched with one 16-byte load that also brings its successor, the
// Stat hot child.  When the walk moves to that successor the lane uses the
// copy it already holds and issues no load at all.  Each cursor keeps the
// LDS byte addresses of its row's features and votes, set once per walk.
typedef uint32_t u32x4_a8 __attribute__((ext_vector_type(4), aligned(8)));

template <int K, int FMODE>
__device__ __forceinline__ void run_tile_compact(const JobDesc& j, int nt, int tile, unsigned char* smem) {
    const bool feat_lds = FMODE == 2 ? (j.feat_lds != 0) : (FMODE == 1);
    const int4* ttab = reinterpret_cast<const int4*>(smem + j.off_ttab);
    const int32_t* fmap_l = reinterpret_cast<const int32_t*>(smem + j.off_fmap);
    float* xs = reinterpret_cast<float*>(smem + j.off_xs);
    int32_t* vl = reinterpret_cast<int32_t*>(smem + j.off_votes);
    int32_t* pool = reinterpret_cast<int32_t*>(smem + j.off_pool);
    const uint2* words = reinterpret_cast<const uint2*>(j.nodes);
    const int lane = lane_id();
    const int fb = j.fbits, cb = j.cbits;
    const uint32_t fmask = (1u << fb) - 1u, cmask = (1u << cb) - 1u;

    const int64_t row0 = (int64_t)tile * j.R;
    const int rows_here = tile_rows(j, row0);

    const int U = rows_here * nt;
    const uint32_t rmagic = 0xFFFFFFFFu / (uint32_t)rows_here;
    TileRows tr{j, xs, vl, fmap_l, row0, feat_lds};
    // per cursor: row in the tile, nb = bin base (words), topl = top_len,
    // the successor copy (sref, sthr, sw)
    int32_t ref[K], rowk[K], nb[K], topl[K], sref[K];
    float sthr[K];
    uint32_t sw[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        ref[k] = kDone; rowk[k] = 0; nb[k] = 0; topl[k] = 0; sref[k] = -1; sthr[k] = 0.0f; sw[k] = 0;
    }
    auto take = [&](int k, int r, int4 e) -> int32_t {
        rowk[k] = r; nb[k] = e.y; topl[k] = e.z; sref[k] = -1;
        if (e.x < 0) {  // the root is a leaf
            tr.vote(r, -e.x - 1);
            return kDone;
        }
        return e.x;
    };
    bool drained = false;
    while (true) {
        if (!drained) refill<K>(ref, pool, U, (uint32_t)rows_here, rmagic, ttab, j.refill_min, lane, drained, take);
        bool live = false;
#pragma unroll
        for (int k = 0; k < K; k++) live |= ref[k] >= 0;
        if (__ballot(live) == 0) {
            if (drained) break;
            continue;
        }
        // loads: a top node (16 B), or a deep node with its successor (16 B), or nothing
        float thr[K];
        uint32_t a0[K], a1[K], a2[K];
        bool deep[K];
#pragma unroll
        for (int k = 0; k < K; k++) {
            deep[k] = false;
            if (ref[k] < 0) continue;
            if (ref[k] < topl[k]) {
                const int4 v = *reinterpret_cast<const int4*>(words + nb[k] + 2 * ref[k]);
                thr[k] = __int_as_float(v.x); a0[k] = (uint32_t)v.y; a1[k] = (uint32_t)v.z; a2[k] = (uint32_t)v.w;
            } else if (ref[k] == sref[k]) {
                deep[k] = true;
                thr[k] = sthr[k]; a0[k] = sw[k];
            } else {
                deep[k] = true;
                const u32x4_a8 v = *reinterpret_cast<const u32x4_a8*>(words + nb[k] + topl[k] + ref[k]);
                thr[k] = __uint_as_float(v.x); a0[k] = v.y;
                sthr[k] = __uint_as_float(v.z); sw[k] = v.w; sref[k] = ref[k] + 1;
            }
        }
#pragma unroll
        for (int k = 0; k < K; k++) {
            if (ref[k] < 0) continue;
            const uint32_t f = deep[k] ? (a0[k] & fmask) : a0[k];
            const bool go_left = tr.x(rowk[k], f) <= thr[k];
            int32_t nr;
            if (!deep[k]) {
                nr = go_left ? (int32_t)a1[k] : (int32_t)a2[k];
            } else {
                const uint32_t w = a0[k];
                const uint32_t pay = w >> (fb + 3);
                if ((w >> fb) & 1u) {
                    const bool adj_left = (w >> (fb + 1)) & 1u;
                    if (go_left == adj_left) nr = ref[k] + 1;
                    else if ((w >> (fb + 2)) & 1u) nr = -(int32_t)pay - 1;
                    else nr = ref[k] + (int32_t)pay;
                } else {
                    nr = -(int32_t)(go_left ? (pay & cmask) : (pay >> cb)) - 1;
                }
            }
            if (nr < 0) {
                tr.vote(rowk[k], -nr - 1);
                nr = kDone;
            }
            ref[k] = nr;
        }
    }
    write_tile(j, vl, row0, rows_here);
}

// A fetched block as the walk sees it: the word and threshold of each slot,
// the first child block, and how to read a child code.
struct BlockView {
    uint32_t w[7], t[7];
    uint32_t child_base, ranks;
};

// Fetches block `ref` of a bin in its host form: three (48-byte form) or four
// (64-byte form) 16-byte loads of one line, issued back to back; the bin's
// first `ns` blocks come from their LDS copy instead.
// bp = the bin's first block in memory, la = LDS byte address of its copy
// (blocks below ns).
template <bool B48>
__device__ __forceinline__ void fetch_block(const global_u32x4* bp, uint32_t la, int32_t ns, int32_t ref,
                                            uint4 (&q)[4]) {
    constexpr int bw = B48 ? 3 : 4;  // 16-byte pieces per block
    if (ref < ns) {
        const lds_u32x4* lp = lds_ptr<u32x4>(la + (B48 ? __umul24((uint32_t)ref, 48u) : (uint32_t)ref << 6));
        q[0] = as_uint4(lp[0]);
        q[1] = as_uint4(lp[1]);
        q[2] = as_uint4(lp[2]);
        if (!B48) q[3] = as_uint4(lp[3]);
    } else {
        const global_u32x4* gp = bp + bw * ref;
        q[0] = as_uint4(gp[0]);
        q[1] = as_uint4(gp[1]);
        q[2] = as_uint4(gp[2]);
        if (!B48) q[3] = as_uint4(gp[3]);
    }
}

// Unpacks a fetched block (Block48: 19-bit words at fixed offsets of the first
// 136 bits; Block64: (thr, word) pairs after the header).
template <bool B48>
__device__ __forceinline__ BlockView view_block(const uint4 (&q)[4]) {
    BlockView b;
    if (B48) {
        const uint32_t r[5] = {q[0].x, q[0].y, q[0].z, q[0].w, q[1].x};
        constexpr uint32_t M = (1u << fp::kBlock48WordBits) - 1u;
#pragma unroll
        for (int sl = 0; sl < 7; sl++) {
            const int o = fp::kBlock48WordBits * sl;
            b.w[sl] = __builtin_amdgcn_alignbit(r[o / 32 + 1 < 5 ? o / 32 + 1 : 4], r[o / 32], o % 32) & M;
        }
        b.t[0] = q[1].y; b.t[1] = q[1].z; b.t[2] = q[1].w;
        b.t[3] = q[2].x; b.t[4] = q[2].y; b.t[5] = q[2].z; b.t[6] = q[2].w;
        b.child_base = r[4] >> 8;
        b.ranks = 0;
    } else {
        b.child_base = q[0].x; b.ranks = q[0].y;
        b.t[0] = q[0].z; b.w[0] = q[0].w;
        b.t[1] = q[1].x; b.w[1] = q[1].y; b.t[2] = q[1].z; b.w[2] = q[1].w;
        b.t[3] = q[2].x; b.w[3] = q[2].y; b.t[4] = q[2].z; b.w[4] = q[2].w;
        b.t[5] = q[3].x; b.w[5] = q[3].y; b.t[6] = q[3].z; b.w[6] = q[3].w;
    }
    return b;
}

// BLOCKED layout walk.  Every reference is a block of the bin (or a class).
// A block is fetched whole and walked for up to three levels from registers:
// slot 0, then slot 1 or 2, then one of slots 3..6, ending in a class or an
// exit to a child block, which the next iteration fetches.  With the row's
// features in LDS all seven split tests are read in one LDS round trip and
// the path is resolved from a mask of sides by selects (no divergence inside
// a block).
// Only forests without a walk form (classes or features beyond its fields)
// come here: run_tile_walk below is the faster walk of the same blocks.
// B48: 48-byte blocks, else 64-byte ones.
template <int K, int FMODE, bool B48>
__device__ __forceinline__ void run_tile_blocked(const JobDesc& j, int nt, int tile, unsigned char* smem) {
    const bool feat_lds = FMODE == 2 ? (j.feat_lds != 0) : (FMODE == 1);
    const int4* ttab = reinterpret_cast<const int4*>(smem + j.off_ttab);
    const int32_t* fmap_l = reinterpret_cast<const int32_t*>(smem + j.off_fmap);
    float* xs = reinterpret_cast<float*>(smem + j.off_xs);
    int32_t* vl = reinterpret_cast<int32_t*>(smem + j.off_votes);
    int32_t* pool = reinterpret_cast<int32_t*>(smem + j.off_pool);
    const uint2* words = reinterpret_cast<const uint2*>(j.nodes);
    const int lane = lane_id();
    const int fb = j.fbits;
    const int cw = 1 + (B48 ? max(j.cbits, 3) : j.cbits);  // bits of one child code
    const uint32_t fmask = (1u << fb) - 1u, code_mask = (1u << cw) - 1u;
    const uint32_t sh_l = (uint32_t)fb, sh_r = (uint32_t)(fb + cw);  // where the left / right codes start

    const int64_t row0 = (int64_t)tile * j.R;
    const int rows_here = tile_rows(j, row0);

    const int U = rows_here * nt;
    const uint32_t rmagic = 0xFFFFFFFFu / (uint32_t)rows_here;
    // x <= thr for compacted feature f; xrow = LDS byte address of the row's
    // first feature in the tile (or its row in the tile when features stay
    // in memory)
    auto le = [&](int32_t xrow, uint32_t f, float thr) {
        const float x = feat_lds ? lds_ptr<float>((uint32_t)xrow)[f] : j.X[(row0 + xrow) * j.ld + fmap_l[f]];
        return x <= thr;
    };
    const uint32_t xs_addr = lds_addr(xs), blocks_addr = lds_addr(smem);
    // the block an exit leaves to: rank from the code (48-byte form) or the table
    auto exit_to = [&](const BlockView& b, uint32_t e, uint32_t code) -> int32_t {
        const uint32_t rank = B48 ? (code >> 1) : ((b.ranks >> (4 * e)) & 7u);
        return (int32_t)(b.child_base + rank);
    };
    // per cursor: xrow, vrow = the row's first vote counter, bp = the bin's
    // first block, la / ns = its LDS copy (byte address, blocks held)
    int32_t ref[K], xrow[K], vrow[K], ns[K];
    uint32_t la[K];
    const global_u32x4* bp[K];
#pragma unroll
    for (int k = 0; k < K; k++) {
        ref[k] = kDone; xrow[k] = 0; vrow[k] = 0; ns[k] = 0; la[k] = 0; bp[k] = nullptr;
    }
    auto take = [&](int k, int r, int4 e) -> int32_t {
        xrow[k] = feat_lds ? (int32_t)(xs_addr + 4u * __umul24((uint32_t)r, (uint32_t)j.Fcp)) : r;
        vrow[k] = (int32_t)__umul24((uint32_t)r, (uint32_t)j.C);
        bp[k] = (const global_u32x4*)(words + e.y);
        la[k] = blocks_addr + 16u * (uint32_t)e.z;
        ns[k] = e.w;
        if (e.x < 0) {  // the root is a leaf
            atomicAdd(&vl[vrow[k] - e.x - 1], 1);
            return kDone;
        }
        return e.x;
    };
    bool drained = false;
    while (true) {
        if (!drained) refill<K>(ref, pool, U, (uint32_t)rows_here, rmagic, ttab, j.refill_min, lane, drained, take);
        bool live = false;
#pragma unroll
        for (int k = 0; k < K; k++) live |= ref[k] >= 0;
        if (__ballot(live) == 0) {
            if (drained) break;
            continue;
        }
        uint4 q[K][4];
#pragma unroll
        for (int k = 0; k < K; k++)
            if (ref[k] >= 0) fetch_block<B48>(bp[k], la[k], ns[k], ref[k], q[k]);
#pragma unroll
        for (int k = 0; k < K; k++) {
            if (ref[k] < 0) continue;
            int32_t nr;
            if (const BlockView b = view_block<B48>(q[k]); feat_lds) {
                // all seven split tests (absent slots are zero words: feature
                // 0, harmless) packed into a mask of sides, bit s set = slot s
                // goes right; the path reads the mask, so the seven LDS reads
                // issue together, ahead of any branch
                uint32_t gm = 0;
#pragma unroll
                for (int sl = 0; sl < 7; sl++)
                    gm |= (lds_ptr<float>((uint32_t)xrow[k])[b.w[sl] & fmask] <= __uint_as_float(b.t[sl]) ? 0u : 1u) << sl;
                const uint32_t side0 = gm & 1u;
                const uint32_t c0 = (b.w[0] >> (side0 ? sh_r : sh_l)) & code_mask;
                const uint32_t side1 = (gm >> (1 + side0)) & 1u;
                const uint32_t w1 = side0 ? b.w[2] : b.w[1];
                const uint32_t c1 = (w1 >> (side1 ? sh_r : sh_l)) & code_mask;
                const uint32_t idx = 2 * side0 + side1;
                const uint32_t side2 = (gm >> (3 + idx)) & 1u;
                const uint32_t w2 = side0 ? (side1 ? b.w[6] : b.w[5]) : (side1 ? b.w[4] : b.w[3]);
                const uint32_t c2 = (w2 >> (side2 ? sh_r : sh_l)) & code_mask;
                int32_t r = exit_to(b, 2 * idx + side2, c2);
                r = (c2 & 1u) ? ~(int32_t)(c2 >> 1) : r;
                r = (c1 & 1u) ? ~(int32_t)(c1 >> 1) : r;
                nr = (c0 & 1u) ? ~(int32_t)(c0 >> 1) : r;
            } else {
                // features from memory: one level at a time
                uint32_t side = le(xrow[k], b.w[0] & fmask, __uint_as_float(b.t[0])) ? 0u : 1u;
                uint32_t c = (b.w[0] >> (side ? sh_r : sh_l)) & code_mask;
                if (c & 1u) {
                    nr = ~(int32_t)(c >> 1);
                } else {
                    const uint32_t s1 = side;
                    const uint32_t w1 = s1 ? b.w[2] : b.w[1];
                    side = le(xrow[k], w1 & fmask, __uint_as_float(s1 ? b.t[2] : b.t[1])) ? 0u : 1u;
                    c = (w1 >> (side ? sh_r : sh_l)) & code_mask;
                    if (c & 1u) {
                        nr = ~(int32_t)(c >> 1);
                    } else {
                        const uint32_t idx = 2 * s1 + side;
                        const uint32_t w2 = s1 ? (side ? b.w[6] : b.w[5]) : (side ? b.w[4] : b.w[3]);
                        const uint32_t t2 = s1 ? (side ? b.t[6] : b.t[5]) : (side ? b.t[4] : b.t[3]);
                        side = le(xrow[k], w2 & fmask, __uint_as_float(t2)) ? 0u : 1u;
                        c = (w2 >> (side ? sh_r : sh_l)) & code_mask;
                        nr = (c & 1u) ? ~(int32_t)(c >> 1) : exit_to(b, 2 * idx + side, c);
                    }
                }
            }
            if (nr < 0) {
                atomicAdd(&vl[vrow[k] - nr - 1], 1);
                nr = kDone;
            }
            ref[k] = nr;
        }
    }
    write_tile(j, vl, row0, rows_here);
}

// ---------------------------------------------------------------------------
// Walk form (fp_internal.h): conversion at upload, and the walk over it
// ---------------------------------------------------------------------------
// Blocks [lo, hi) of every bin, one thread each (blockIdx.y strides over
// bins): reads the host form and writes the walk form, block k at k times its
// smaller size from the bin's start.  The caller picks [lo, hi) so that what
// it writes was read by this workgroup before the barrier or by an earlier
// launch.
__global__ __launch_bounds__(256) void walk_form_kernel(const BinEntry* __restrict__ bins, int32_t n_bins, uint32_t* nodes,
                                                        int32_t layout, int32_t form, int32_t block_bytes, int32_t fbits,
                                                        int32_t cbits, int64_t lo, int64_t hi) {
    const int bd = block_bytes / 4;
    const fp::WalkShape ws = fp::walk_shape(form);
    const int64_t k = lo + (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    for (int32_t b = blockIdx.y; b < n_bins; b += gridDim.y) {
        const int64_t unit0 = bins[b].node_base / 2;  // the bin's first 16-byte unit
        const bool live = k < hi && k < bins[b].deep_len;
        uint32_t* const bin = nodes + unit0 * 4;
        uint32_t w[16];
        for (int i = 0; i < 16; i++) w[i] = live && i < bd ? bin[k * bd + i] : 0u;
        asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
        __syncthreads();  // every block of the workgroup has been read before any is written
        if (!live) continue;
        uint32_t thr0[7], feat0[7], kill[7], to[8], child;
        int n_exits = 0;
        for (int s = 0; s < 7; s++) kill[s] = 0;
        for (int e = 0; e < 8; e++) to[e] = ws.leaf;
        if (layout == FP_LAYOUT_CLUSTERED) {
            const bool c48 = block_bytes == 48;
            const int cv = c48 ? 4 : 7, rest = c48 ? 8 : 11;  // dwords of care/val bytes, of rest
            auto bits = [&](int pos, int width) -> uint32_t {  // rest bits; 48-byte form: bits from 128 in dword 3's high half
                const int i = pos / 32;
                const uint32_t l = w[rest + i];
                const uint32_t h = i + 1 < (c48 ? 4 : 5) ? w[rest + i + 1] : c48 ? w[3] >> 16 : 0u;
                return (uint32_t)((((uint64_t)h << 32) | l) >> (pos % 32)) & ((1u << width) - 1u);
            };
            uint32_t care[8], val[8];
            for (int e = 0; e < 8; e++) {
                care[e] = (w[cv + e / 4] >> (8 * (e % 4))) & 255u;
                val[e] = (w[cv + 2 + e / 4] >> (8 * (e % 4))) & 255u;
                n_exits += !(care[e] & 0x80u);
            }
            for (int s = 0; s < 7; s++) {
                if (c48) {
                    thr0[s] = (w[s / 2] >> (16 * (s % 2))) & 0xFFFFu;
                    feat0[s] = bits(s == 0 ? 48 : s <= 3 ? 64 + 9 * (s - 1) : 96 + 9 * (s - 4), fp::kCluster48FeatBits);
                } else {
                    thr0[s] = w[s];
                    feat0[s] = bits(48 + fp::kClusterFeatBits * s, fp::kClusterFeatBits);
                }
            }
            static_assert(fp::kC48FeatPos[0] == 48 && fp::kC48FeatPos[1] == 64 && fp::kC48FeatPos[3] == 82 &&
                              fp::kC48FeatPos[4] == 96 && fp::kC48FeatPos[6] == 114,
                          "feature positions of the 48-byte block");
            child = c48 ? bits(fp::kC48BasePos, fp::kC48BaseBits) : bits(132, 24);
            // two exits part at the one slot they both test with different
            // outcomes: the exit that goes left there lies left
            for (int e = 0; e < 8; e++) {
                if (care[e] & 0x80u) continue;  // unused
                int at = 0;
                for (int o = 0; o < 8; o++)
                    if (!(care[o] & 0x80u)) at += (val[e] & care[e] & care[o] & (val[e] ^ val[o])) != 0;  // o lies left of e
                const uint32_t t = bits(6 * e, 6), target = (t & 32u) ? (t & 7u) : ws.leaf | (t & 31u);
                for (int x = 0; x < 8; x++) to[x] = x == at ? target : to[x];
                for (int s = 0; s < 7; s++)
                    if ((care[e] >> s & 1u) && !(val[e] >> s & 1u)) kill[s] |= 1u << at;
            }
        } else {
            const bool b48 = block_bytes == 48;
            const int cw = 1 + (b48 ? max(cbits, 3) : cbits);
            const uint32_t cmask = (1u << cw) - 1u, fmask = (1u << fbits) - 1u;
            uint32_t code[14];
            for (int s = 0; s < 7; s++) {
                uint32_t word;
                if (b48) {
                    const int o = fp::kBlock48WordBits * s;
                    const uint64_t two = ((uint64_t)(o / 32 + 1 < 5 ? w[o / 32 + 1] : 0u) << 32) | w[o / 32];
                    word = (uint32_t)(two >> (o % 32)) & ((1u << fp::kBlock48WordBits) - 1u);
                    thr0[s] = w[5 + s];
                } else {
                    word = w[3 + 2 * s];
                    thr0[s] = w[2 + 2 * s];
                }
                feat0[s] = word & fmask;
                code[2 * s] = (word >> fbits) & cmask;
                code[2 * s + 1] = (word >> (fbits + cw)) & cmask;
            }
            child = b48 ? w[4] >> 8 : w[0];
            for (int e = 0; e < 8; e++) {
                // the first class on the path to bottom exit e, else its child block
                const uint32_t c0 = code[e / 4], c1 = code[2 * (1 + e / 4) + (e / 2) % 2], c2 = code[6 + e];
                const uint32_t c = (c0 & 1u) ? c0 : (c1 & 1u) ? c1 : c2;
                to[e] = (c & 1u) ? ws.leaf | (c >> 1) : b48 ? c2 >> 1 : (w[1] >> (4 * e)) & 7u;
            }
            kill[0] = 15; kill[1] = 3; kill[2] = 48; kill[3] = 1; kill[4] = 4; kill[5] = 16; kill[6] = 64;
            n_exits = 8;
        }
        // slots in order (the place of a slot is the last exit of its left
        // subtree), exits beyond the block's own repeating its last one
        uint32_t thr[7], feat[7], mask[7];
        for (int i = 0; i < 7; i++) {
            thr[i] = feat[i] = mask[i] = 0;
            for (int s = 0; s < 7; s++)
                if (kill[s] && 31 - __builtin_clz(kill[s]) == i) { thr[i] = thr0[s]; feat[i] = feat0[s]; mask[i] = kill[s]; }
        }
        if (form == fp::kWalk48b)  // in the tree's own order, its masks are constants
            for (int s = 0; s < 7; s++) { thr[s] = thr0[s]; feat[s] = feat0[s]; }
        for (int e = 1; e < 8; e++) to[e] = e < n_exits ? to[e] : to[e - 1];
        uint64_t targets = 0;
        for (int e = 0; e < 8; e++) targets |= (uint64_t)to[e] << (ws.tbits * e);
        uint32_t below = 0;  // the stored mask bits: slot i's i bits below bit i, from bit i (i - 1) / 2
        for (int i = 1; i < 7; i++) below |= (mask[i] & ((1u << i) - 1u)) << (i * (i - 1) / 2);
        const uint32_t base = (uint32_t)(fp::kGlobalRef + unit0 / (ws.unit / 16) + (int64_t)child * (ws.bytes / ws.unit));
        const uint32_t t_lo = (uint32_t)targets, t_hi = (uint32_t)(targets >> 32);
        const uint32_t m_lo = mask[0] | mask[1] << 8 | mask[2] << 16 | mask[3] << 24, m_hi = mask[4] | mask[5] << 8 | mask[6] << 16;
        const uint32_t f10a = feat[0] | feat[1] << 10 | feat[2] << 20, f10b = feat[3] | feat[4] << 10 | feat[5] << 20;
        uint32_t* d = bin + k * (ws.bytes / 4);
        if (form == fp::kWalk64) {
            for (int s = 0; s < 7; s++) d[s] = thr[s];
            d[7] = m_lo;
            d[8] = m_hi;
            for (int s = 0; s < 3; s++) d[9 + s] = feat[2 * s] | feat[2 * s + 1] << 16;
            d[12] = feat[6];
            d[13] = t_lo;
            d[14] = t_hi;
            d[15] = base;
        } else if (form == fp::kWalk48h) {
            for (int s = 0; s < 3; s++) d[s] = thr[2 * s] | thr[2 * s + 1] << 16;
            d[3] = thr[6] | feat[6] << 16;
            for (int s = 0; s < 3; s++) d[4 + s] = feat[2 * s] | feat[2 * s + 1] << 16;
            d[7] = m_lo;
            d[8] = base;
            d[9] = t_lo;
            d[10] = t_hi;
            d[11] = m_hi;
        } else if (form == fp::kWalk32h) {
            // mask 6 is a run that ends in bit 6: its start
            const uint32_t start6 = mask[6] ? (uint32_t)__builtin_ctz(mask[6]) : 6u;
            for (int s = 0; s < 3; s++) d[s] = thr[2 * s] | thr[2 * s + 1] << 16;
            d[3] = thr[6] | (below & 0x7FFFu) << 16;
            d[4] = feat[0] | feat[1] << 9 | feat[2] << 18 | (feat[6] & 31u) << 27;
            d[5] = feat[3] | feat[4] << 9 | feat[5] << 18 | (feat[6] >> 5) << 27;
            d[6] = t_lo;
            d[7] = t_hi | base << 8 | start6 << 28;
        } else {
            for (int s = 0; s < 7; s++) d[s] = thr[s];
            d[7] = f10a;
            d[8] = f10b;
            if (form == fp::kWalk48f) {
                d[9] = feat[6] | below << 10;
                d[10] = t_lo;
                d[11] = base;
            } else {
                d[9] = base;
                d[10] = t_lo;
                d[11] = t_hi | feat[6] << 16;
            }
        }
    }
}

// a + half HI of w times m (16 bits each): one instruction.
template <int HI>
__device__ __forceinline__ uint32_t mad_half(uint32_t w, uint32_t m, uint32_t a) {
    uint32_t r;
    if constexpr (HI) asm("v_mad_u32_u16 %0, %1, %2, %3 op_sel:[1,0,0,0]" : "=v"(r) : "v"(w), "s"(m), "v"(a));
    else asm("v_mad_u32_u16 %0, %1, %2, %3" : "=v"(r) : "v"(w), "s"(m), "v"(a));
    return r;
}

// Exits killed by a block's seven tests: per slot one compare that leaves
// only the lanes going right (!(x <= t): NaN goes right) active, and one OR
// of the slot's kill byte under that mask.  exec is the caller's on exit.
#define FP_KILL(CMP, M) CMP "\n\t" M "\n\ts_mov_b64 exec, %[sv]\n\t"
#define FP_OR_BYTE(W, B) "v_or_b32_sdwa %[k], %[k], %[" W "] dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:DWORD src1_sel:BYTE_" B
__device__ __forceinline__ uint32_t killed_f32(const float (&x)[7], const float (&t)[7], uint32_t lo, uint32_t hi) {
    uint32_t k = 0;
    uint64_t sv;
    asm volatile("s_mov_b64 %[sv], exec\n\t"
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x0], %[t0]", FP_OR_BYTE("lo", "0"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x1], %[t1]", FP_OR_BYTE("lo", "1"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x2], %[t2]", FP_OR_BYTE("lo", "2"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x3], %[t3]", FP_OR_BYTE("lo", "3"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x4], %[t4]", FP_OR_BYTE("hi", "0"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x5], %[t5]", FP_OR_BYTE("hi", "1"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x6], %[t6]", FP_OR_BYTE("hi", "2"))
                 : [k] "+v"(k), [sv] "=&s"(sv)
                 : [x0] "v"(x[0]), [x1] "v"(x[1]), [x2] "v"(x[2]), [x3] "v"(x[3]), [x4] "v"(x[4]), [x5] "v"(x[5]),
                   [x6] "v"(x[6]), [t0] "v"(t[0]), [t1] "v"(t[1]), [t2] "v"(t[2]), [t3] "v"(t[3]), [t4] "v"(t[4]),
                   [t5] "v"(t[5]), [t6] "v"(t[6]), [lo] "v"(lo), [hi] "v"(hi)
                 : "vcc");
    return k;
}
// fp16 features (low halves of x) against the fp16 thresholds t01 .. t6 (two to a word, t6 low).
__device__ __forceinline__ uint32_t killed_f16(const uint32_t (&x)[7], uint32_t t01, uint32_t t23, uint32_t t45,
                                               uint32_t t6, uint32_t lo, uint32_t hi) {
    uint32_t k = 0;
    uint64_t sv;
#define FP_NLE_HI(X, T) "v_cmpx_nle_f16_sdwa vcc, %[" X "], %[" T "] src0_sel:DWORD src1_sel:WORD_1"
    asm volatile("s_mov_b64 %[sv], exec\n\t"
                 FP_KILL("v_cmpx_nle_f16_e32 vcc, %[x0], %[t01]", FP_OR_BYTE("lo", "0"))
                 FP_KILL(FP_NLE_HI("x1", "t01"), FP_OR_BYTE("lo", "1"))
                 FP_KILL("v_cmpx_nle_f16_e32 vcc, %[x2], %[t23]", FP_OR_BYTE("lo", "2"))
                 FP_KILL(FP_NLE_HI("x3", "t23"), FP_OR_BYTE("lo", "3"))
                 FP_KILL("v_cmpx_nle_f16_e32 vcc, %[x4], %[t45]", FP_OR_BYTE("hi", "0"))
                 FP_KILL(FP_NLE_HI("x5", "t45"), FP_OR_BYTE("hi", "1"))
                 FP_KILL("v_cmpx_nle_f16_e32 vcc, %[x6], %[t6]", FP_OR_BYTE("hi", "2"))
                 : [k] "+v"(k), [sv] "=&s"(sv)
                 : [x0] "v"(x[0]), [x1] "v"(x[1]), [x2] "v"(x[2]), [x3] "v"(x[3]), [x4] "v"(x[4]), [x5] "v"(x[5]),
                   [x6] "v"(x[6]), [t01] "v"(t01), [t23] "v"(t23), [t45] "v"(t45), [t6] "v"(t6), [lo] "v"(lo),
                   [hi] "v"(hi)
                 : "vcc");
    return k;
}
// Masks in registers.  m[i]: slot i's bits below bit i; bit i itself is a constant.
#define FP_OR_MASK(I, C) "v_or3_b32 %[k], %[k], %[m" I "], " C
__device__ __forceinline__ uint32_t killed_f32(const float (&x)[7], const float (&t)[7], const uint32_t (&m)[7]) {
    uint32_t k = 0;
    uint64_t sv;
    asm volatile("s_mov_b64 %[sv], exec\n\t"
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x0], %[t0]", "v_or_b32_e32 %[k], 1, %[k]")
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x1], %[t1]", FP_OR_MASK("1", "2"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x2], %[t2]", FP_OR_MASK("2", "4"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x3], %[t3]", FP_OR_MASK("3", "8"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x4], %[t4]", FP_OR_MASK("4", "16"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x5], %[t5]", FP_OR_MASK("5", "32"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x6], %[t6]", FP_OR_MASK("6", "64"))
                 : [k] "+v"(k), [sv] "=&s"(sv)
                 : [x0] "v"(x[0]), [x1] "v"(x[1]), [x2] "v"(x[2]), [x3] "v"(x[3]), [x4] "v"(x[4]), [x5] "v"(x[5]),
                   [x6] "v"(x[6]), [t0] "v"(t[0]), [t1] "v"(t[1]), [t2] "v"(t[2]), [t3] "v"(t[3]), [t4] "v"(t[4]),
                   [t5] "v"(t[5]), [t6] "v"(t[6]), [m1] "v"(m[1]), [m2] "v"(m[2]), [m3] "v"(m[3]), [m4] "v"(m[4]),
                   [m5] "v"(m[5]), [m6] "v"(m[6])
                 : "vcc");
    return k;
}
__device__ __forceinline__ uint32_t killed_f16(const uint32_t (&x)[7], uint32_t t01, uint32_t t23, uint32_t t45, uint32_t t6,
                                               const uint32_t (&m)[7]) {
    uint32_t k = 0;
    uint64_t sv;
    asm volatile("s_mov_b64 %[sv], exec\n\t"
                 FP_KILL("v_cmpx_nle_f16_e32 vcc, %[x0], %[t01]", "v_or_b32_e32 %[k], 1, %[k]")
                 FP_KILL(FP_NLE_HI("x1", "t01"), FP_OR_MASK("1", "2"))
                 FP_KILL("v_cmpx_nle_f16_e32 vcc, %[x2], %[t23]", FP_OR_MASK("2", "4"))
                 FP_KILL(FP_NLE_HI("x3", "t23"), FP_OR_MASK("3", "8"))
                 FP_KILL("v_cmpx_nle_f16_e32 vcc, %[x4], %[t45]", FP_OR_MASK("4", "16"))
                 FP_KILL(FP_NLE_HI("x5", "t45"), FP_OR_MASK("5", "32"))
                 FP_KILL("v_cmpx_nle_f16_e32 vcc, %[x6], %[t6]", FP_OR_MASK("6", "64"))
                 : [k] "+v"(k), [sv] "=&s"(sv)
                 : [x0] "v"(x[0]), [x1] "v"(x[1]), [x2] "v"(x[2]), [x3] "v"(x[3]), [x4] "v"(x[4]), [x5] "v"(x[5]),
                   [x6] "v"(x[6]), [t01] "v"(t01), [t23] "v"(t23), [t45] "v"(t45), [t6] "v"(t6), [m1] "v"(m[1]),
                   [m2] "v"(m[2]), [m3] "v"(m[3]), [m4] "v"(m[4]), [m5] "v"(m[5]), [m6] "v"(m[6])
                 : "vcc");
    return k;
}
#undef FP_OR_MASK
#undef FP_NLE_HI
// A complete three-level subtree: the kill masks are constants.
__device__ __forceinline__ uint32_t killed_full(const float (&x)[7], const float (&t)[7]) {
    uint32_t k = 0;
    uint64_t sv;
#define FP_OR_CONST(C) "v_or_b32_e32 %[k], " C ", %[k]"
    asm volatile("s_mov_b64 %[sv], exec\n\t"
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x0], %[t0]", FP_OR_CONST("15"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x1], %[t1]", FP_OR_CONST("3"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x2], %[t2]", FP_OR_CONST("48"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x3], %[t3]", FP_OR_CONST("1"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x4], %[t4]", FP_OR_CONST("4"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x5], %[t5]", FP_OR_CONST("16"))
                 FP_KILL("v_cmpx_nle_f32_e32 vcc, %[x6], %[t6]", FP_OR_CONST("64"))
                 : [k] "+v"(k), [sv] "=&s"(sv)
                 : [x0] "v"(x[0]), [x1] "v"(x[1]), [x2] "v"(x[2]), [x3] "v"(x[3]), [x4] "v"(x[4]), [x5] "v"(x[5]),
                   [x6] "v"(x[6]), [t0] "v"(t[0]), [t1] "v"(t[1]), [t2] "v"(t[2]), [t3] "v"(t[3]), [t4] "v"(t[4]),
                   [t5] "v"(t[5]), [t6] "v"(t[6])
                 : "vcc");
#undef FP_OR_CONST
    return k;
}
#undef FP_OR_BYTE
#undef FP_KILL

// Low / high fp16 half of a word widened to fp32 (exact).
__device__ __forceinline__ float half_lo(uint32_t v) {
    return (float)__builtin_bit_cast(_Float16, (unsigned short)(v & 0xFFFFu));
}
__device__ __forceinline__ float half_hi(uint32_t v) {
    return (float)__builtin_bit_cast(_Float16, (unsigned short)(v >> 16));
}

// One step through a complete three-level subtree (BLOCKED) with features in
// memory: only the features of the walk's own path are read, and none below a
// class (all exits there hold it).  A feature read is a lane's own line, the
// step's whole cost: reading all seven took 30,000 image rows x 128 trees
// from 643 to 1418 us.
template <int FORM>
__device__ __forceinline__ int32_t path_step(const JobDesc& j, const uint4 (&q)[4], int64_t row, const int32_t* fmap_l,
                                             bool& leaf) {
    static_assert(FORM == fp::kWalk48b || FORM == fp::kWalk64, "the forms of BLOCKED blocks");
    constexpr fp::WalkShape ws = fp::walk_shape(FORM);
    const float* x = j.X + row * j.ld;
    // in the order of the tree: slot s has its children at 2s + 1, 2s + 2
    uint32_t f[7], t[7];
    if constexpr (FORM == fp::kWalk48b) {
#pragma unroll
        for (int s = 0; s < 3; s++) {
            f[s] = (q[1].w >> (10 * s)) & 1023u;
            f[3 + s] = (q[2].x >> (10 * s)) & 1023u;
        }
        f[6] = q[2].w >> 16;
        t[0] = q[0].x; t[1] = q[0].y; t[2] = q[0].z; t[3] = q[0].w; t[4] = q[1].x; t[5] = q[1].y; t[6] = q[1].z;
    } else {  // stored left to right
        f[3] = q[2].y & 0xFFFFu; f[1] = q[2].y >> 16; f[4] = q[2].z & 0xFFFFu; f[0] = q[2].z >> 16;
        f[5] = q[2].w & 0xFFFFu; f[2] = q[2].w >> 16; f[6] = q[3].x & 0xFFFFu;
        t[3] = q[0].x; t[1] = q[0].y; t[4] = q[0].z; t[0] = q[0].w; t[5] = q[1].x; t[2] = q[1].y; t[6] = q[1].z;
    }
    const uint64_t all = FORM == fp::kWalk48b ? (uint64_t)q[2].w << 32 | q[2].z : (uint64_t)q[3].z << 32 | q[3].y;
    constexpr uint32_t tm = (1u << ws.tbits) - 1u;
    // targets of the four and of the two exits that are left
    constexpr uint32_t two = 1u | 1u << ws.tbits, m4 = ws.tbits == 8 ? ~0u : (1u << (4 * ws.tbits)) - 1u;
    const bool g0 = !(x[fmap_l[f[0]]] <= __uint_as_float(t[0]));
    uint32_t to = (uint32_t)(all >> (g0 ? 4 * ws.tbits : 0)) & m4;
    uint32_t c = to & tm;
    if (!(c & ws.leaf) || to != c * two * (1u | 1u << 2 * ws.tbits)) {
        const bool g1 = !(x[fmap_l[g0 ? f[2] : f[1]]] <= __uint_as_float(g0 ? t[2] : t[1]));
        to = (to >> (g1 ? 2 * ws.tbits : 0)) & ((1u << 2 * ws.tbits) - 1u);
        c = to & tm;
        if (!(c & ws.leaf) || to != c * two) {
            const uint32_t f2 = g0 ? (g1 ? f[6] : f[5]) : (g1 ? f[4] : f[3]), t2 = g0 ? (g1 ? t[6] : t[5]) : (g1 ? t[4] : t[3]);
            if (!(x[fmap_l[f2]] <= __uint_as_float(t2))) c = to >> ws.tbits;
        }
    }
    leaf = (c & ws.leaf) != 0;
    return leaf ? (int32_t)c : (int32_t)((FORM == fp::kWalk48b ? q[2].y : q[3].w) + __umul24(c, (uint32_t)(ws.bytes / ws.unit)));
}

// One step: decodes the block in q and returns the next reference, or the
// target of a leaf with `leaf` set.
template <int FMODE, int FORM, bool X16>
__device__ __forceinline__ int32_t walk_step(const JobDesc& j, const uint4 (&q)[4], uint32_t xrow, uint32_t es, int64_t row0,
                                             const int32_t* fmap_l, bool& leaf) {
    constexpr fp::WalkShape ws = fp::walk_shape(FORM);
    constexpr bool F16 = FORM == fp::kWalk48h || FORM == fp::kWalk32h;
    constexpr bool BELOW = FORM == fp::kWalk48f || FORM == fp::kWalk32h;  // masks stored as the bits below each slot's
    if constexpr (FMODE == 0 && (FORM == fp::kWalk48b || FORM == fp::kWalk64))
        if (FORM == fp::kWalk48b || j.layout == FP_LAYOUT_BLOCKED)
            return path_step<FORM>(j, q, row0 + (int64_t)xrow, fmap_l, leaf);
    // LDS address (or number) of slot s's feature
    uint32_t at[7];
    const uint32_t m = FMODE == 1 ? es : 1u, a0 = FMODE == 1 ? xrow : 0u;
    if constexpr (FORM == fp::kWalk48b || FORM == fp::kWalk48f || FORM == fp::kWalk32h) {
        constexpr int fb = FORM == fp::kWalk32h ? 9 : 10;
        const uint32_t fw[2] = {FORM == fp::kWalk32h ? q[1].x : q[1].w, FORM == fp::kWalk32h ? q[1].y : q[2].x};
#pragma unroll
        for (int s = 0; s < 6; s++) at[s] = a0 + __umul24((fw[s / 3] >> (fb * (s % 3))) & ((1u << fb) - 1u), m);
        if constexpr (FORM == fp::kWalk48b) at[6] = mad_half<1>(q[2].w, m, a0);
        else if constexpr (FORM == fp::kWalk48f) at[6] = a0 + __umul24(q[2].y & 1023u, m);
        else at[6] = a0 + __umul24(__builtin_amdgcn_alignbit(q[1].y >> 27, q[1].x, 27), m);
    } else {
        const uint32_t fw[3] = {FORM == fp::kWalk64 ? q[2].y : q[1].x, FORM == fp::kWalk64 ? q[2].z : q[1].y,
                                FORM == fp::kWalk64 ? q[2].w : q[1].z};
#pragma unroll
        for (int s = 0; s < 3; s++) {
            at[2 * s] = mad_half<0>(fw[s], m, a0);
            at[2 * s + 1] = mad_half<1>(fw[s], m, a0);
        }
        at[6] = FORM == fp::kWalk48h ? mad_half<1>(q[0].w, m, a0) : mad_half<0>(q[3].x, m, a0);
    }
    uint32_t mask[7] = {0, 0, 0, 0, 0, 0, 0};
    if constexpr (BELOW) {
        const uint32_t w = FORM == fp::kWalk48f ? q[2].y : q[0].w;
        constexpr int o = FORM == fp::kWalk48f ? 10 : 16;
#pragma unroll
        for (int i = 1; i < 7; i++) mask[i] = (w >> (o + i * (i - 1) / 2)) & ((1u << i) - 1u);
        if constexpr (FORM == fp::kWalk32h) mask[6] = (0x7Fu << (q[1].w >> 28)) & 0x7Fu;
    }
    uint32_t killed;
    if constexpr (X16) {
        uint32_t x[7];
#pragma unroll
        for (int s = 0; s < 7; s++) x[s] = *lds_ptr<uint16_t>(at[s]);
        if constexpr (BELOW) killed = killed_f16(x, q[0].x, q[0].y, q[0].z, q[0].w, mask);
        else killed = killed_f16(x, q[0].x, q[0].y, q[0].z, q[0].w, q[1].w, q[2].w);
    } else {
        float x[7], t[7];
#pragma unroll
        for (int s = 0; s < 7; s++)
            x[s] = FMODE == 1 ? *lds_ptr<float>(at[s]) : j.X[(row0 + (int64_t)xrow) * j.ld + fmap_l[at[s]]];
        if constexpr (F16) {
            t[0] = half_lo(q[0].x); t[1] = half_hi(q[0].x); t[2] = half_lo(q[0].y); t[3] = half_hi(q[0].y);
            t[4] = half_lo(q[0].z); t[5] = half_hi(q[0].z); t[6] = half_lo(q[0].w);
        } else {
            t[0] = __uint_as_float(q[0].x); t[1] = __uint_as_float(q[0].y); t[2] = __uint_as_float(q[0].z);
            t[3] = __uint_as_float(q[0].w); t[4] = __uint_as_float(q[1].x); t[5] = __uint_as_float(q[1].y);
            t[6] = __uint_as_float(q[1].z);
        }
        if constexpr (FORM == fp::kWalk48b) killed = killed_full(x, t);
        else if constexpr (BELOW) killed = killed_f32(x, t, mask);
        else killed = killed_f32(x, t, q[1].w, FORM == fp::kWalk64 ? q[2].x : q[2].w);
    }
    const uint32_t e = (uint32_t)__builtin_ctz(~killed);  // the lowest exit alive, 0..7
    uint32_t t, base;
    if constexpr (FORM == fp::kWalk64) {
        t = __builtin_amdgcn_perm(q[3].z, q[3].y, e | 0x0C0C0C00u);
        base = q[3].w;
    } else if constexpr (FORM == fp::kWalk48h) {
        t = __builtin_amdgcn_perm(q[2].z, q[2].y, e | 0x0C0C0C00u);
        base = q[2].x;
    } else if constexpr (FORM == fp::kWalk48f) {
        t = (q[2].z >> (4u * e)) & 15u;
        base = q[2].w;
    } else if constexpr (FORM == fp::kWalk48b) {
        t = (uint32_t)((((uint64_t)q[2].w << 32) | q[2].z) >> (6u * e)) & 63u;
        base = q[2].y;
    } else {
        t = (uint32_t)((((uint64_t)q[1].w << 32) | q[1].z) >> (5u * e)) & 31u;
        base = (q[1].w >> 8) & 0xFFFFFu;
    }
    leaf = (t & ws.leaf) != 0;
    return leaf ? (int32_t)t : (int32_t)(base + __umul24(t, (uint32_t)(ws.bytes / ws.unit)));
}

// The walk over blocks in their walk form: one walk per lane, a block a step
// (two per lane were no faster on the large tabular forest, 7.00 against
// 7.03 ms, and slower on the image one, 2.27 against 1.67 ms).
// X16: the tile holds fp16 features (forms with fp16 thresholds).  A walk's state is its
// reference (LDS or memory, see fp_internal.h), the LDS address of its row's
// features (or its row, when features stay in memory) and of its votes.
// Bound by 16-byte pieces a lane loads (0.74 cycles of the CU's vector memory
// path each) together with LDS (seven feature reads a step, 8 cycles a
// wavefront at random banks) and instruction issue; the working set hardly
// matters (210-260 G blocks/s from 2 MB to 300 MB of forest).  Against host
// blocks with care/value exit patterns (80 VALU instructions a step, four or
// three pieces): 1M image rows x 128 trees 2.03 -> 1.64 ms, 2M tabular rows x
// 160 trees 8.30 -> 7.04 ms, 4,096 rows x 1,024 trees 231 -> 191 us.
template <int FMODE, int FORM, bool X16>
__device__ __forceinline__ void run_tile_walk(const JobDesc& j, int nt, int tile, unsigned char* smem) {
    static_assert(!X16 || (FMODE == 1 && (FORM == fp::kWalk48h || FORM == fp::kWalk32h)),
                  "fp16 tiles live in LDS and need fp16 thresholds");
    constexpr fp::WalkShape ws = fp::walk_shape(FORM);
    constexpr int bw = ws.bytes / 16;
    const int32_t* ttab = reinterpret_cast<const int32_t*>(smem + j.off_ttab);
    const int32_t* fmap_l = reinterpret_cast<const int32_t*>(smem + j.off_fmap);
    float* xs = reinterpret_cast<float*>(smem + j.off_xs);
    int32_t* vl = reinterpret_cast<int32_t*>(smem + j.off_votes);
    int32_t* pool = reinterpret_cast<int32_t*>(smem + j.off_pool);
    const int lane = lane_id();

    const int64_t row0 = (int64_t)tile * j.R;
    const int rows_here = tile_rows(j, row0);

    const int U = rows_here * nt;
    const uint32_t rmagic = 0xFFFFFFFFu / (uint32_t)rows_here;
    const uint32_t es = X16 ? 2u * (uint32_t)j.Fcp : 4u;  // bytes from one feature of a row to the next
    const uint32_t rs = X16 ? 2u : 4u * (uint32_t)j.Fcp;  // and from one row to the next
    const uint32_t xs_addr = lds_addr(xs), pool_addr = lds_addr(pool);
    const uint32_t votes_addr = lds_addr(vl) - 4u * ws.leaf;  // a target with its leaf bit indexes from here
    const global_u32x4* gbase = (const global_u32x4*)j.nodes - fp::kGlobalRef * (ws.unit / 16);
    int32_t ref = kDone;
    uint32_t xrow = 0, vrow = 0;
    bool drained = false;
    while (true) {
        uint64_t idle = __ballot(ref < 0);
        int cnt = (int)__popcll(idle);
        while (cnt >= j.refill_min && !drained) {
            int base = 0;
            if (lane == 0)
                asm volatile("ds_add_rtn_u32 %0, %1, %2\n\ts_waitcnt lgkmcnt(0)" : "=&v"(base) : "v"(pool_addr), "v"(cnt) : "memory");
            base = __builtin_amdgcn_readfirstlane(base);
            drained = base + cnt >= U;
            if (ref < 0) {
                const uint32_t u = (uint32_t)(base + bits_below(idle));
                if (u < (uint32_t)U) {
                    uint32_t r;
                    const uint32_t t = div_rows(u, (uint32_t)rows_here, rmagic, r);
                    ref = ttab[t];
                    xrow = FMODE == 1 ? xs_addr + __umul24(r, rs) : r;
                    vrow = votes_addr + 4u * __umul24(r, (uint32_t)j.C);
                    if (ref < 0) {  // the root is a leaf
                        atomicAdd(&vl[__umul24(r, (uint32_t)j.C) - ref - 1], 1);
                        ref = kDone;
                    }
                }
            }
            idle = __ballot(ref < 0);
            cnt = (int)__popcll(idle);
        }
        if (cnt == 64) break;  // a wavefront with nothing live has drained the pool
        // LDS blocks first: the loads from memory into the same registers
        // then wait for LDS only, not LDS reads for memory (7.5 against
        // 8.0 ms on the large tabular forest)
        uint4 q[4];
        if ((uint32_t)ref < (uint32_t)fp::kGlobalRef) {
            const lds_u32x4* lp = lds_ptr<u32x4>((uint32_t)ref * (uint32_t)ws.unit);
#pragma unroll
            for (int i = 0; i < bw; i++) q[i] = as_uint4(lp[i]);
        }
        if (ref >= fp::kGlobalRef) {
            const global_u32x4* gp = gbase + (size_t)(uint32_t)ref * (ws.unit / 16);
#pragma unroll
            for (int i = 0; i < bw; i++) q[i] = as_uint4(gp[i]);
        }
        if (ref >= 0) {
            bool leaf;
            ref = walk_step<FMODE, FORM, X16>(j, q, xrow, es, row0, fmap_l, leaf);
            if (leaf) {
                __hip_atomic_fetch_add(const_cast<__attribute__((address_space(3))) int32_t*>(
                                           lds_ptr<int32_t>(vrow + 4u * (uint32_t)ref)),
                                       1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
                ref = kDone;
            }
        }
    }
    write_tile(j, vl, row0, rows_here);
}

// Stages one tile of a job of kind KIND; prefetched: the thread's first quad is `pre`.
template <int FMODE, int KIND>
__device__ __forceinline__ void stage_kind(const JobDesc& j, int tile, unsigned char* smem, float4 pre, bool prefetched) {
    const int64_t row0 = (int64_t)tile * j.R;
    stage_tile<KIND == kKind48hX || KIND == kKind32hX>(
        j, reinterpret_cast<float*>(smem + j.off_xs), reinterpret_cast<int32_t*>(smem + j.off_votes),
        reinterpret_cast<int32_t*>(smem + j.off_pool), row0, tile_rows(j, row0), FMODE == 1, pre, prefetched);
}

// Walks one staged tile of a job of kind KIND, K cursors per lane (block
// layouts: one), and writes its votes.
template <int K, int FMODE, int KIND>
__device__ __forceinline__ void walk_tile(const JobDesc& j, int nt, int tile, unsigned char* smem) {
    if constexpr (KIND == kKindPacked || KIND == kKindPairs) run_tile<K, FMODE, KIND == kKindPairs>(j, nt, tile, smem);
    else if constexpr (KIND == kKindCompact) run_tile_compact<K, FMODE>(j, nt, tile, smem);
    else if constexpr (KIND == kKindHost48 || KIND == kKindHost64) run_tile_blocked<1, FMODE, KIND == kKindHost48>(j, nt, tile, smem);
    else run_tile_walk<FMODE, kind_form(KIND), KIND == kKind48hX || KIND == kKind32hX>(j, nt, tile, smem);
}

// One forest: persistent workgroups, group = blockIdx % G (consecutive
// workgroups land on different XCDs, so G = 8 gives each XCD its own trees).
// Waves per SIMD the kernel must allow: two 1024-thread workgroups per CU
// (8 waves per SIMD, at most 64 VGPRs) while the cursors fit in that budget.
// A 1024-thread workgroup needs 4 waves per SIMD, so no variant gets more
// than 128 VGPRs.
template <int K, int KIND>
struct MinWaves {
    static constexpr int value = KIND == kKindPacked    ? (K <= 4 ? 8 : 4)
                                 : KIND == kKindCompact ? (K <= 2 ? 8 : K == 4 ? 6 : 4)
                                                        : 8;
    static_assert(KIND != kKindPairs || K <= 2, "four cursors or more have no registers for pairs");
};

template <int K, int FMODE, int KIND>
__global__ __launch_bounds__(1024, (MinWaves<K, KIND>::value)) void packed_kernel(JobDesc j) {
    extern __shared__ __align__(32) unsigned char smem[];
    const int group = j.group_base + (int)(blockIdx.x % j.G);
    const int blocks_per_group = gridDim.x / j.G;
    int tile = blockIdx.x / j.G;
    // Single nodes with four cursors have no registers for the first quad (five
    // spilled: 1M tabular rows x 16 trees, 256-row tiles 1.69 ms with it, 1.51
    // without; 1M image rows x 128 trees, 32-row tiles 14.2 and 10.9)
    constexpr bool kPrefetch = K < 4 || KIND != kKindPacked;
    float4 pre = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    if constexpr (kPrefetch) pre = prefetch_quad<FMODE>(j, tile);
    const int nt = stage_group<KIND>(j, group, smem);
    if (nt == 0) return;  // uniform per block
    bool first = kPrefetch;
    for (; tile < j.n_tiles; tile += blocks_per_group) {
        stage_kind<FMODE, KIND>(j, tile, smem, pre, first);
        first = false;
        walk_tile<K, FMODE, KIND>(j, nt, tile, smem);
    }
}

// Many forests: persistent workgroups pull work items from a global counter
// (items are ordered largest first) and restage LDS when the (job, group)
// changes.  Every workgroup exits once the counter passes n_items.
// One tile, staged and walked.
template <int K, int FM, int KIND>
__device__ __forceinline__ void item_tile(const JobDesc& j, int nt, int tile, unsigned char* smem) {
    stage_kind<FM, KIND>(j, tile, smem, make_float4(0.0f, 0.0f, 0.0f, 0.0f), false);
    walk_tile<K, FM, KIND>(j, nt, tile, smem);
}

// Tiles [tile_begin, tile_end) of one work item, features in LDS (FM 1) or
// read from memory (FM 0).  Block layouts walk one block per lane.
// BLOCKS: the job is in a block layout, else in a node layout: one kernel
// each, so that neither sets the other's register budget (a mixed list of
// jobs in one kernel spilled its walks: 64 forests 42 ms against 15).
template <int K, int FM, bool BLOCKS>
__device__ __forceinline__ void item_tiles(const JobDesc& j, const WorkItem& w, int nt, unsigned char* smem) {
    const int kind = job_kind(j);
    for (int tile = w.tile_begin; tile < w.tile_end; tile++) {
        if constexpr (!BLOCKS) {
            if (kind == kKindCompact) {
                item_tile<K, FM, kKindCompact>(j, nt, tile, smem);
                continue;
            }
            if constexpr (FM == 1 && K <= 2) {
                if (kind == kKindPairs) {
                    item_tile<K, 1, kKindPairs>(j, nt, tile, smem);
                    continue;
                }
            }
            item_tile<K, FM, kKindPacked>(j, nt, tile, smem);
        } else {
            switch (kind) {
                case kKindHost48: item_tile<1, FM, kKindHost48>(j, nt, tile, smem); break;
                case kKindHost64: item_tile<1, FM, kKindHost64>(j, nt, tile, smem); break;
                case kKind64: item_tile<1, FM, kKind64>(j, nt, tile, smem); break;
                case kKind48h: item_tile<1, FM, kKind48h>(j, nt, tile, smem); break;
                case kKind48b: item_tile<1, FM, kKind48b>(j, nt, tile, smem); break;
                case kKind48f: item_tile<1, FM, kKind48f>(j, nt, tile, smem); break;
                case kKind32h: item_tile<1, FM, kKind32h>(j, nt, tile, smem); break;
                case kKind48hX:
                    if constexpr (FM == 1) item_tile<1, 1, kKind48hX>(j, nt, tile, smem);
                    break;
                case kKind32hX:
                    if constexpr (FM == 1) item_tile<1, 1, kKind32hX>(j, nt, tile, smem);
                    break;
            }
        }
    }
}

// The item number is broadcast through a slot at the end of the dynamic LDS
// (item_slot bytes in), not a static __shared__ variable: static LDS would
// add to every job's budget and leave two workgroups no longer fitting a CU.
// The counter wraps to 0 after n_items + gridDim.x draws, which is what a
// launch makes (each workgroup draws one number past the list), so no kernel
// has to clear it first.  Launches of one list that overlap share the draws:
// each number past the list still ends one workgroup, so together they make
// whole rounds of the counter, walk every item once per launch and leave 0.
template <int K, bool BLOCKS>
__device__ __forceinline__ void batched_walk(const JobDesc* jobs, const WorkItem* items, int32_t n_items, int32_t* counter,
                                             int32_t item_slot, unsigned char* smem) {
    int32_t* s_item = reinterpret_cast<int32_t*>(smem + item_slot);
    int staged_job = -1, staged_group = -1, nt = 0;
    while (true) {
        if (threadIdx.x == 0)
            *s_item = (int32_t)atomicInc(reinterpret_cast<unsigned*>(counter), (unsigned)n_items + gridDim.x - 1);
        __syncthreads();
        // the item is the workgroup's: readfirstlane makes that visible to the
        // compiler, so the item and its job descriptor are loaded into scalar
        // registers instead of occupying vector registers in every lane
        const int it = __builtin_amdgcn_readfirstlane(*s_item);
        __syncthreads();
        if (it >= n_items) break;
        const WorkItem w = items[it];
        const JobDesc& j = jobs[w.job];
        if (w.job != staged_job || w.group != staged_group) {
            nt = stage_group<BLOCKS ? kKindAnyBlock : kKindAnyNode>(j, w.group, smem);
            staged_job = w.job;
            staged_group = w.group;
        }
        if (nt == 0) continue;
        // the feature source is fixed per job: walk with it compiled in
        if (j.feat_lds) item_tiles<K, 1, BLOCKS>(j, w, nt, smem);
        else item_tiles<K, 0, BLOCKS>(j, w, nt, smem);
    }
}

// A list of jobs of one layout class.
template <int K, bool BLOCKS>
__global__ __launch_bounds__(1024, (BLOCKS || K <= 2 ? 8 : 4)) void batched_kernel(const JobDesc* __restrict__ jobs,
                                                                                   const WorkItem* __restrict__ items,
                                                                                   int32_t n_items, int32_t* counter,
                                                                                   int32_t item_slot) {
    extern __shared__ __align__(32) unsigned char smem[];
    batched_walk<K, BLOCKS>(jobs, items, n_items, counter, item_slot, smem);
}

// Both lists, one after the other in each workgroup: workgroups that find the
// blocks' list drawn go on to the nodes', where a kernel each would wait for
// the other's last item (3 jobs of up to 600 trees and 1,500 columns: 117 us
// as two kernels, 77 as one; 16 jobs of up to 60,000 rows: 364 and 325).  The
// walks are in sequence, not in one loop, so that neither class sets the
// other's registers.
template <int K>
__global__ __launch_bounds__(1024, (K <= 2 ? 8 : 4)) void batched_mixed_kernel(const JobDesc* __restrict__ jobs,
                                                                               const WorkItem* __restrict__ items,
                                                                               int32_t n_block_items, int32_t n_items,
                                                                               int32_t* counters, int32_t item_slot) {
    extern __shared__ __align__(32) unsigned char smem[];
    batched_walk<1, true>(jobs, items, n_block_items, counters, item_slot, smem);
    batched_walk<K, false>(jobs, items + n_block_items, n_items - n_block_items, counters + 1, item_slot, smem);
}

__global__ void fill_i32_kernel(int32_t* p, int64_t n, int32_t v) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        p[i] = v;
}

__global__ void argmax_kernel(const int32_t* votes, int32_t* cls, int64_t n, int32_t C) {
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t* v = votes + i * C;
        int32_t best = 0, bestv = v[0];
        for (int c = 1; c < C; c++)
            if (v[c] > bestv) { bestv = v[c]; best = c; }
        cls[i] = best;
    }
}

// blockIdx.y = job: zero the votes of jobs that accumulate with atomics (run
// only when the launch has any, as is the epilogue).
__global__ void batched_prologue_kernel(const JobDesc* jobs) {
    const JobDesc& j = jobs[blockIdx.y];
    if (!j.atomic_votes) return;
    const int64_t n = j.n_rows * j.C;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
        j.votes[i] = 0;
}

__global__ void batched_epilogue_kernel(const JobDesc* jobs) {
    const JobDesc& j = jobs[blockIdx.y];
    if (!j.atomic_votes || !j.cls) return;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < j.n_rows; i += (int64_t)gridDim.x * blockDim.x) {
        const int32_t* v = j.votes + i * j.C;
        int32_t best = 0, bestv = v[0];
        for (int c = 1; c < j.C; c++)
            if (v[c] > bestv) { bestv = v[c]; best = c; }
        j.cls[i] = best;
    }
}

int check_launch(const char* what) {
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return fp_set_error(FP_EHIP, "%s launch: %s", what, hipGetErrorString(e));
    return FP_OK;
}

template <int K, int KIND>
const void* packed_fn(int fmode) {
    return fmode == 0 ? reinterpret_cast<const void*>(&packed_kernel<K, 0, KIND>)
                      : reinterpret_cast<const void*>(&packed_kernel<K, 1, KIND>);
}

// A block walk keeps one block in flight per lane whatever `cursors` says.
const void* pick_packed(int K, int fmode, int kind) {
    if (K != 1 && K != 2 && K != 4 && K != 8) return nullptr;
    switch (kind) {
        case kKindHost48: return packed_fn<1, kKindHost48>(fmode);
        case kKindHost64: return packed_fn<1, kKindHost64>(fmode);
        case kKind64: return packed_fn<1, kKind64>(fmode);
        case kKind48h: return packed_fn<1, kKind48h>(fmode);
        case kKind48b: return packed_fn<1, kKind48b>(fmode);
        case kKind48f: return packed_fn<1, kKind48f>(fmode);
        case kKind32h: return packed_fn<1, kKind32h>(fmode);
        case kKind48hX: return reinterpret_cast<const void*>(&packed_kernel<1, 1, kKind48hX>);
        case kKind32hX: return reinterpret_cast<const void*>(&packed_kernel<1, 1, kKind32hX>);
        case kKindPairs:
            if (K == 1) return reinterpret_cast<const void*>(&packed_kernel<1, 1, kKindPairs>);
            if (K == 2) return reinterpret_cast<const void*>(&packed_kernel<2, 1, kKindPairs>);
    }
#define FP_PICK(KK) \
    if (K == KK) return kind == kKindCompact ? packed_fn<KK, kKindCompact>(fmode) : packed_fn<KK, kKindPacked>(fmode);
    FP_PICK(1)
    FP_PICK(2)
    FP_PICK(4)
    FP_PICK(8)
#undef FP_PICK
    return nullptr;
}

// The batched kernel of block layouts (which walk one block per lane whatever
// K is) or of node layouts.
const void* pick_batched(int K, bool blocks) {
    if (K != 1 && K != 2 && K != 4 && K != 8) return nullptr;
    if (blocks) return reinterpret_cast<const void*>(&batched_kernel<1, true>);
    switch (K) {
        case 1: return reinterpret_cast<const void*>(&batched_kernel<1, false>);
        case 2: return reinterpret_cast<const void*>(&batched_kernel<2, false>);
        case 4: return reinterpret_cast<const void*>(&batched_kernel<4, false>);
        default: return reinterpret_cast<const void*>(&batched_kernel<8, false>);
    }
}
// The kernel of both, or null where the node walk's registers would halve the
// wavefronts of the block walk (eight cursors).
const void* pick_mixed(int K) {
    return K == 1   ? reinterpret_cast<const void*>(&batched_mixed_kernel<1>)
           : K == 2 ? reinterpret_cast<const void*>(&batched_mixed_kernel<2>)
           : K == 4 ? reinterpret_cast<const void*>(&batched_mixed_kernel<4>)
                    : nullptr;
}

std::mutex g_props_mu;
fp::DeviceProps g_props[64];
bool g_props_ok[64];

size_t round16(size_t v) { return (v + 15) / 16 * 16; }

}  // namespace

namespace fp {

int current_device(int* dev) {
    hipError_t e = hipGetDevice(dev);
    if (e != hipSuccess) return fp_set_error(FP_EHIP, "hipGetDevice: %s", hipGetErrorString(e));
    return FP_OK;
}

int device_props(int dev, DeviceProps* out) {
    if (dev < 0 || dev >= 64) return fp_set_error(FP_ENODEV, "device id %d out of range", dev);
    std::lock_guard<std::mutex> lk(g_props_mu);
    if (!g_props_ok[dev]) {
        hipDeviceProp_t pr;
        hipError_t e = hipGetDeviceProperties(&pr, dev);
        if (e != hipSuccess) return fp_set_error(FP_EHIP, "hipGetDeviceProperties: %s", hipGetErrorString(e));
        g_props[dev].cus = pr.multiProcessorCount;
        g_props[dev].lds_per_block = pr.sharedMemPerBlock;
        g_props[dev].lds_per_cu = pr.maxSharedMemoryPerMultiProcessor;
        g_props_ok[dev] = true;
    }
    *out = g_props[dev];
    return FP_OK;
}

size_t default_lds_block(const DeviceProps& dp) {
    const size_t blk = dp.lds_per_block ? dp.lds_per_block : 65536;
    const size_t cu = dp.lds_per_cu ? dp.lds_per_cu : blk;
    return std::min(blk, cu / 2);
}

size_t job_lds_layout(JobDesc* j) {
    size_t o = (size_t)j->cap * j->bins_per_group * sizeof(Node16);
    j->off_ttab = (int32_t)o;  o += round16((size_t)j->trees_per_group * (j->form != kWalkNone ? 4 : 16));
    j->off_fmap = (int32_t)o;  o += j->feat_lds ? 0 : round16((size_t)j->Fc * 4);
    j->off_imap = (int32_t)o;  o += j->stage_rows ? round16((size_t)(j->F + 3) / 4 * 4 * 2) : 0;
    j->off_xs = (int32_t)o;    o += j->feat_lds ? round16(j->x16 ? (size_t)j->Fc * j->Fcp * 2 : (size_t)j->R * j->Fcp * 4) : 0;
    j->off_votes = (int32_t)o; o += round16((size_t)j->R * j->C * 4);
    j->off_pool = (int32_t)o;  o += 16;
    j->lds_bytes = (int32_t)o;
    return o;
}

const BinEntry* bins_host(const fp_packed* p) {
    return reinterpret_cast<const BinEntry*>(p->bytes.data() + p->hdr.table_offset);
}

int resolve_job(const fp_packed* p, const fp_tune* t, const float* X, int64_t n_rows, int64_t ld, int32_t* votes,
                int32_t* cls, size_t lds_block, int cus, JobDesc* j) {
    const Header& h = p->hdr;
    if (h.layout != FP_LAYOUT_PACKED && h.layout != FP_LAYOUT_COMPACT && h.layout != FP_LAYOUT_BLOCKED &&
        h.layout != FP_LAYOUT_CLUSTERED)
        return fp_set_error(FP_EINVAL, "forest is not in a packed layout");
    if (!p->dev) return fp_set_error(FP_ENODEV, "packed forest is not uploaded");
    if (h.n_nodes >= INT32_MAX)
        return fp_set_error(FP_E2BIG, "packed forest has %lld nodes (limit 2^31-1)", (long long)h.n_nodes);
    const bool blocks = h.layout >= FP_LAYOUT_BLOCKED;
    const bool auto_R = t->rows_per_block <= 0;
    if (t->rows_per_block > 4096) return fp_set_error(FP_EINVAL, "rows_per_block %d exceeds 4096", t->rows_per_block);
    // tree_groups 0: one, except for launches of their own (cus > 0) of at
    // least 2^18 walks, which pay for zeroing the votes and the classes' own
    // launch, on forests larger than an XCD's L2 (4 MB; 600 trees of 0.4 MB,
    // 4,000 rows: one group 20.5 us, four 26.3; COMPACT 8 MB: 100,000 rows x
    // 256 trees of 4.3 MB: one group 510 us, eight 548):
    //  - block layouts of 512 trees or more: a group per 128 trees, so that a
    //    workgroup's LDS holds several blocks of each of its trees instead of
    //    one or none (4,096 rows x 1,024 trees: one group 60 us at its best
    //    tile, eight 47; 40,000 rows: 382 and 337);
    //  - node layouts: 8, 4 or 2 groups, which workgroup numbers spread over
    //    the 8 XCDs, so that each L2 sees only its groups' nodes (100,003 rows
    //    x 64 trees, 20 MB: one group 285 us at its best tile, four 214); as
    //    many as hold a like number of bins each (9 bins: two groups 690 us,
    //    five 767).
    // Every row is staged, and its votes added, once per group: not where
    // that outweighs the walks (30,000 rows x 2,000 columns x 640 trees: one
    // group 403 us, five 600; 10,000 image rows x 128 trees: 62 and, with
    // eight, 76); nor where a group's explicit tile has fewer walks than the
    // workgroup threads (100,000 rows x 64 trees, 16-row tiles: one 311 us,
    // four 398).  Explicit tiles that leave CUs idle take groups for those
    // (4,000 rows x 600 trees, 64-row tiles: one 55 us, four 24), and, within
    // a tighter bound on staging, for wavefronts that smaller workgroups leave
    // idle (128 trees, 16-row tiles in 256 threads, 64 columns: 40 classes,
    // one 50 us, two 33; 100 classes 27 and 38).
    int G = std::max(1, t->tree_groups);
    const int threads = t->block_threads > 0 ? t->block_threads : 1024;
    if (t->tree_groups <= 0 && cus > 0 && t->tree_passes <= 1 && n_rows * h.n_trees >= (1 << 18)) {
        auto staged = [&](int64_t g, int64_t most) { return (h.n_features + h.n_classes) * g <= most * h.n_trees; };
        if (h.total_bytes > (int64_t(h.layout == FP_LAYOUT_COMPACT ? 8 : 4) << 20)) {
            auto bins_of = [&](int g) { return (h.n_bins + g - 1) / g; };
            if (blocks) G = std::max(1, h.n_trees >= 512 ? std::min(8, h.n_trees / 128) : 1);
            else for (G = 8; G > 1 && (bins_of(bins_of(G)) != G || 5 * h.n_bins < 4 * G * bins_of(G));) G /= 2;
            if (!staged(G, 3)) G = 1;
            while (!auto_R && G > 1 && (int64_t)t->rows_per_block * h.n_trees < (int64_t)threads * G) G /= 2;
        }
        if (!auto_R) {
            const int64_t tiles = (n_rows + t->rows_per_block - 1) / t->rows_per_block;
            int64_t idle = std::min<int64_t>(8, (int64_t)cus * (1024 / threads) / tiles);
            while (idle > 1 && !staged(idle, 2)) idle /= 2;
            G = (int)std::max({(int64_t)G, std::min<int64_t>(8, cus / tiles), idle});
        }
    }
    if (G > h.n_bins) G = h.n_bins;
    int P = t->tree_passes > 0 ? t->tree_passes : 1;
    if ((int64_t)P * G > h.n_bins) P = std::max(1, h.n_bins / G);
    const int bpg = (h.n_bins + P * G - 1) / (P * G);
    // passes that would hold no bin are dropped: the last pass writes the classes
    P = ((h.n_bins + bpg - 1) / bpg + G - 1) / G;
    if (P == 1) G = (h.n_bins + bpg - 1) / bpg;  // nor do groups without a bin take workgroups
    const int tpg = (int)std::min<int64_t>((int64_t)bpg * h.bin_size, h.n_trees);
    // rows_per_block 0, alone on the device.  Fewer, larger tiles leave CUs
    // idle (300 image rows x 128 trees: 16-row tiles 15.9 us, 2-row ones
    // 10.8); smaller ones stage the trees' tops and wait for their last walks
    // more often (4,096 rows x 1,024 trees: 8-row tiles 71 us, 16-row ones 60;
    // 10^6 rows x 32 trees: 16-row tiles 558 us, 128-row ones 270, 512-row
    // ones 241).
    //  - blocks: a tile per CU (with tree groups two), at most 16,384 walks
    //    and 512 rows;
    //  - nodes: two tiles per CU (4,000 rows x 272 trees, COMPACT: one 43 us,
    //    two 35), or one where two would not have a walk for each of their
    //    threads; at most 256 rows, COMPACT 64 (its top nodes come from
    //    memory: 100,000 rows x 600 trees: 256-row tiles 618 us, 64-row ones
    //    525);
    //  - features in memory: at most kMemoryTileRows.
    // With 512 threads or fewer twice the tiles (not with four cursors or
    // more, which hold half the wavefronts; COMPACT, 256 threads: 16 rows).
    // A plan's jobs share the device: 16 to 64 rows, 64 tiles of 1,024 threads
    // or more (16 forests of up to 512 trees and 60,000 rows: 16-row tiles 488
    // us, 32-row ones 393, 64-row ones 333; 8 forests, 10,000 rows: 78, 58 and
    // 58; 6 forests, 4,000 rows, 256 threads: 16-row tiles 48 us, 62-row ones
    // 71).  Node layouts there, and serving, take 16.
    const int64_t most = t->feature_lds < 0                ? kMemoryTileRows
                         : cus <= 0                        ? 64
                         : blocks                          ? std::min<int64_t>(512, std::max<int64_t>(32, 16384 / tpg))
                         : h.layout == FP_LAYOUT_COMPACT   ? (threads <= 256 ? 16 : 64)
                                                           : 256;
    const int64_t slots = (int64_t)cus * (threads <= 512 && t->cursors < 4 ? 2 : 1);
    auto rows_for = [&](int64_t per_cu) { return (n_rows * G + per_cu * slots - 1) / (per_cu * slots); };
    int64_t want = 16;
    if (cus > 0 && G > 1) want = std::max<int64_t>(16, rows_for(2));
    else if (cus > 0 && blocks) want = rows_for(1);
    else if (cus > 0) want = std::max(rows_for(2), std::min<int64_t>((n_rows + cus - 1) / cus, (threads + tpg - 1) / tpg));
    else if (cus == 0 && blocks) want = std::min<int64_t>(64, std::max<int64_t>(16, n_rows * threads / 65536));
    int R = auto_R ? (int)std::min(most, want) : t->rows_per_block;
    if ((int64_t)R * tpg >= (1 << 30)) return fp_set_error(FP_E2BIG, "rows_per_block x trees per group too large");
    const uint8_t* base = static_cast<const uint8_t*>(p->dev);
    memset(j, 0, sizeof *j);
    j->bins = reinterpret_cast<const BinEntry*>(base + h.table_offset);
    j->roots = reinterpret_cast<const int32_t*>(base + h.roots_offset);
    j->fmap = reinterpret_cast<const int32_t*>(base + h.fmap_offset);
    j->nodes = reinterpret_cast<const Node16*>(base + h.nodes_offset);
    j->X = X;
    j->ld = ld;
    j->n_rows = n_rows;
    j->votes = votes;
    j->cls = cls;
    j->Fc = h.n_used_features;
    j->Fcp = h.n_used_features | 1;
    j->C = h.n_classes;
    j->n_bins = h.n_bins;
    j->n_trees = h.n_trees;
    j->n_nodes = (int32_t)h.n_nodes;
    j->bin_size = h.bin_size;
    j->R = R;
    j->G = G;
    j->passes = P;
    j->bins_per_group = bpg;
    j->trees_per_group = tpg;
    j->n_tiles = (int32_t)((n_rows + R - 1) / R);
    j->atomic_votes = G > 1;
    j->layout = h.layout;
    j->fbits = h.compact_fbits;
    j->cbits = h.compact_cbits;
    j->form = walk_form(h);
    j->block_bytes = j->form != kWalkNone ? walk_shape(j->form).bytes : h.block_bytes;
    if (t->refill_lanes < 0 || t->refill_lanes > 64) return fp_set_error(FP_EINVAL, "refill_lanes %d outside [0, 64]", t->refill_lanes);
    // Explicit tiles of few rows, long walks and a forest of which L2 holds a
    // small part: late refills let wavefronts drift apart over the trees, and
    // workgroups no longer share what they fetch (2M rows x 448 trees of 24
    // levels, 1.06 GB, 128-row tiles: 66.0 ms at 48 lanes, 50.8 at 24; 704
    // trees, 192 rows: 102.6 and 74.2; 64 trees, 177 MB, 192 rows: 5.18 and
    // 4.44).  For larger tiles 48 is the better one (448 trees, 256 rows, which
    // full rounds make 253: 45.4 and 46.6; 512 rows: 35.3 and 38.7), and for
    // walks of 19 levels (384 trees x 160 features, 96 rows: 5.8 and 6.3).
    const bool drifts = blocks && cus > 0 && !auto_R && R < 224 && h.expected_depth > kDriftDepth &&
                        (h.total_bytes - h.nodes_offset) / P > (int64_t(128) << 20);
    j->refill_min = t->refill_lanes > 0 ? t->refill_lanes
                    : drifts            ? kDefaultRefillLanesDrift
                    : blocks            ? kDefaultRefillLanesBlocks
                                        : kDefaultRefillLanes;
    // feature_lds: 1 force LDS staging, 2 force it in fp32, -1 read features
    // from memory, 0 automatic
    if (t->feature_lds < -1 || t->feature_lds > 2) return fp_set_error(FP_EINVAL, "feature_lds %d outside [-1, 2]", t->feature_lds);
    // fp16 tile: exact where every threshold is exact in fp16 (the CLUSTERED
    // 48-byte form)
    const bool x16_ok = t->feature_lds != 2 && h.layout == FP_LAYOUT_CLUSTERED && h.block_bytes == 48;
    j->F = h.n_features;
    j->cap = 0;
    // LDS need of a tile of r rows, with or without the row tile in LDS
    auto size_for = [&](int r, bool feat) {
        j->R = r;
        j->n_tiles = (int32_t)((n_rows + r - 1) / r);
        j->feat_lds = feat;
        j->x16 = feat && x16_ok;
        // fp16 tile: feature-major, the feature stride an odd number of
        // 4-byte words (rows rounded up to 2 mod 4) so that strided writes
        // and reads spread over the banks; fp32 tile: row-major, odd stride
        j->Fcp = j->x16 ? r + (6 - r % 4) % 4 : h.n_used_features | 1;
        // whole-row staging: rows start on 16 bytes and the column map fits 8 KB
        j->stage_rows = feat && ld % 4 == 0 && reinterpret_cast<uintptr_t>(X) % 16 == 0 && h.n_features <= 4096;
        return job_lds_layout(j);
    };
    // An automatic tile of a node layout in workgroups of 512 threads or fewer
    // shares a CU with three others: half of the LDS that 1,024 threads take
    if (auto_R && !blocks && cus > 0 && threads <= 512 && t->cursors < 4 && t->lds_bytes == 0 &&
        t->feature_lds >= 0 && size_for(1, true) <= lds_block / 2)
        lds_block /= 2;
    // fit by shrinking an automatic tile first (features in LDS matter most),
    // then by reading features from memory.  An automatic tile leaves LDS for
    // a block per tree, up to an eighth of the budget, or for half of the
    // bins' top nodes (these only beyond 8 rows: 30,000 rows x 2,000 columns x
    // 640 trees, PACKED: 4 rows and tops 681 us, 8 rows 585)
    const size_t tops = !auto_R                         ? 0
                        : blocks                        ? std::min(lds_block / 8, (size_t)tpg * (size_t)j->block_bytes)
                        : h.layout == FP_LAYOUT_COMPACT ? 0
                        : cus > 0 ? std::min(lds_block / 2, (size_t)bpg * (size_t)h.max_top_len * sizeof(Node16)) : 0;
    auto fit = [&](bool feat) {
        const size_t need = size_for(R, feat);
        if (!auto_R || need + (feat ? tops : 0) <= lds_block) return need;
        auto largest = [&](int most_r, size_t leave) {  // the largest tile that fits (1 if none does)
            int lo = 1, hi = most_r + 1;
            while (hi - lo > 1) {
                const int r = (lo + hi) / 2;
                if (size_for(r, feat) + leave <= lds_block) lo = r;
                else hi = r;
            }
            return lo;
        };
        const int r = largest(R, feat ? tops : 0);
        return size_for(blocks || r >= 8 ? r : largest(std::min(R, 8), 0), feat);
    };
    size_t need = fit(t->feature_lds >= 0);
    if (need > lds_block) {
        if (t->feature_lds >= 1)
            return fp_set_error(FP_E2BIG, "observation tile of %d rows x %d columns does not fit in %zu bytes of LDS",
                                R, j->Fc, lds_block);
        if (auto_R) R = (int)std::min<int64_t>(R, kMemoryTileRows);
        need = fit(false);
        if (need > lds_block)
            return fp_set_error(FP_E2BIG, "per-workgroup tables of %zu bytes exceed %zu bytes of LDS", need, lds_block);
    } else if (auto_R && !blocks && cus > 0 && tpg <= 1024 && j->R * tpg > 1024 && j->R * tpg < 8 * 1024 / 7) {
        // a walk per thread rather than a second round of few (30,000 rows x
        // 2,000 columns x 128 trees: 9-row tiles 143 us, 8-row ones 120)
        need = size_for(1024 / tpg, j->feat_lds != 0);
    }
    // LDS left over holds the hottest nodes: PACKED bin tops, or the first
    // blocks of each BLOCKED bin (its trees' root blocks come first), counted
    // in 16-byte pieces per bin
    size_t top_nodes = (lds_block - need) / sizeof(Node16);
    if (t->lds_top_nodes < 0 || h.layout == FP_LAYOUT_COMPACT) top_nodes = 0;  // COMPACT: tops from memory
    else if (t->lds_top_nodes > 0) top_nodes = std::min(top_nodes, (size_t)t->lds_top_nodes);
    if (h.layout >= FP_LAYOUT_BLOCKED) {
        const size_t bw = (size_t)j->block_bytes / 16;
        int64_t max_blocks = 0;
        for (int32_t b = 0; b < h.n_bins; b++) max_blocks = std::max<int64_t>(max_blocks, bins_host(p)[b].deep_len);
        j->cap = (int32_t)(std::min<size_t>(top_nodes / bpg / bw, (size_t)max_blocks) * bw);
    } else {
        j->cap = (int32_t)std::min<size_t>(top_nodes / bpg, (size_t)h.max_top_len);
        // PACKED nodes come in pairs where walks are long below the top region
        // and features are in LDS; in a launch of its own only where nothing
        // but those deep nodes is read from memory (top nodes of a bin's trees
        // are interleaved: the next one is another tree's)
        const double deep = h.expected_depth - (h.interleave_depth + 1);
        const bool busy = n_rows * h.n_trees >= (1 << 18) && threads >= 512;
        const bool pairs = h.layout == FP_LAYOUT_PACKED && j->feat_lds && (cus <= 0 || j->cap >= h.max_top_len) &&
                           deep >= (cus <= 0 ? kPairDepthShared : busy ? kPairDepth : kPairDepthIdle);
        j->block_bytes = pairs ? 2 * (int32_t)sizeof(Node16) : (int32_t)sizeof(Node16);
    }
    job_lds_layout(j);
    return FP_OK;
}

int packed_occupancy(int K, const JobDesc& j, int threads, int* blocks_per_cu) {
    const void* fn = pick_packed(K, j.feat_lds ? 1 : 0, job_kind(j));
    if (!fn) return fp_set_error(FP_EINVAL, "cursors must be 1, 2, 4 or 8");
    int occ = 0;
    hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, threads, (size_t)j.lds_bytes);
    *blocks_per_cu = (e == hipSuccess && occ > 0) ? occ : 1;
    return FP_OK;
}

size_t batched_job_budget(size_t lds_block) { return lds_block > kItemSlotBytes ? lds_block - kItemSlotBytes : 0; }

int batched_shape(const JobDesc* jobs, int32_t n_jobs, int K, int threads, int cus, BatchedShape* sh) {
    *sh = BatchedShape{};
    sh->K = K;
    sh->threads = threads;
    sh->n_jobs = n_jobs;
    bool any[2] = {false, false};
    for (int32_t i = 0; i < n_jobs; i++) {
        const int c = batched_class(jobs[i]);
        any[c] = true;
        sh->lds[c] = std::max(sh->lds[c], (size_t)jobs[i].lds_bytes);
        sh->atomics |= jobs[i].atomic_votes != 0;
        sh->atomic_classes |= jobs[i].atomic_votes != 0 && jobs[i].cls != nullptr;
    }
    if (any[0] && any[1] && pick_mixed(K)) {
        sh->mixed = true;
        sh->lds[0] = sh->lds[1] = std::max(sh->lds[0], sh->lds[1]);
    }
    for (int c = 0; c < 2; c++) {
        const void* fn = sh->mixed ? pick_mixed(K) : pick_batched(K, c == 0);
        if (!fn) return fp_set_error(FP_EINVAL, "cursors must be 1, 2, 4 or 8");
        if (!any[c]) continue;
        int occ = 0;
        hipError_t e = hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, fn, threads, round16(sh->lds[c]) + kItemSlotBytes);
        sh->resident[c] = (int64_t)cus * ((e == hipSuccess && occ > 0) ? occ : 1);
    }
    return FP_OK;
}

int launch_leaf_counts(const Node16* nodes, const int64_t* tree_off, int32_t n_trees, const float* X, int64_t n_rows,
                       int64_t ld, int32_t* counts, hipStream_t s) {
    if (n_rows <= 0 || n_trees <= 0) return FP_OK;
    const int64_t blocks = std::min<int64_t>((n_rows + 255) / 256, 65536);
    hipLaunchKernelGGL(leaf_count_kernel, dim3((unsigned)blocks), dim3(256), 0, s, nodes, tree_off, n_trees, X, n_rows,
                       ld, counts);
    return check_launch("leaf_count_kernel");
}

int device_upload(void* dev, const void* src, size_t n, void* stream_v, int* dev_id) {
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    hipError_t e = hipGetDevice(dev_id);
    if (e != hipSuccess) return fp_set_error(FP_EHIP, "hipGetDevice: %s", hipGetErrorString(e));
    e = hipMemcpyAsync(dev, src, n, hipMemcpyHostToDevice, stream);
    if (e != hipSuccess) return fp_set_error(FP_EHIP, "hipMemcpyAsync: %s", hipGetErrorString(e));
    Header h;
    memcpy(&h, src, sizeof h);
    if (const int32_t form = walk_form(h); form != kWalkNone && h.n_bins > 0) {
        uint8_t* base = static_cast<uint8_t*>(dev);
        const BinEntry* bins = reinterpret_cast<const BinEntry*>(static_cast<const uint8_t*>(src) + h.table_offset);
        int64_t blocks = 0;  // of the largest bin
        for (int32_t b = 0; b < h.n_bins; b++) blocks = std::max<int64_t>(blocks, bins[b].deep_len);
        const int64_t from = h.block_bytes, to = walk_shape(form).bytes;
        const unsigned rows = (unsigned)std::min(h.n_bins, 65535);
        for (int64_t lo = 0, hi; lo < blocks; lo = hi) {
            // the blocks of one launch are written over blocks that earlier
            // launches have read, [lo to / from, lo) when they shrink; the
            // first 256 of a bin are one workgroup's
            hi = from == to ? blocks : std::max<int64_t>(256, std::min(blocks, lo * from / to));
            hipLaunchKernelGGL(walk_form_kernel, dim3((unsigned)((hi - lo + 255) / 256), rows), dim3(256), 0, stream,
                               reinterpret_cast<const BinEntry*>(base + h.table_offset), h.n_bins,
                               reinterpret_cast<uint32_t*>(base + h.nodes_offset), h.layout, form, h.block_bytes,
                               h.compact_fbits, h.compact_cbits, lo, hi);
        }
        if (const int rc = check_launch("walk_form_kernel")) {
            (void)hipStreamSynchronize(stream);
            return rc;
        }
    }
    e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return fp_set_error(FP_EHIP, "hipStreamSynchronize: %s", hipGetErrorString(e));
    return FP_OK;
}

int device_leaf_counts(const uint8_t* bytes, size_t nbytes, const Header& h, int32_t n_trees, const float* X,
                       int64_t n_rows, int64_t ld, int32_t* counts, void* stream_v) {
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    DevBuf buf, cnt;
    int rc = buf.ensure(nbytes);
    if (!rc) rc = cnt.ensure(sizeof(int32_t) * (size_t)h.n_nodes);
    if (rc) return rc;
    // once work is queued, every exit waits for the stream before the
    // buffers above (and the host arrays the copies use) go away
    struct Drain {
        hipStream_t s;
        ~Drain() { (void)hipStreamSynchronize(s); }
    } drain{stream};
    hipError_t e = hipMemcpyAsync(buf.p, bytes, nbytes, hipMemcpyHostToDevice, stream);
    if (e == hipSuccess) e = hipMemsetAsync(cnt.p, 0, sizeof(int32_t) * (size_t)h.n_nodes, stream);
    if (e != hipSuccess) return fp_set_error(FP_EHIP, "upload: %s", hipGetErrorString(e));
    const uint8_t* base = static_cast<const uint8_t*>(buf.p);
    rc = launch_leaf_counts(reinterpret_cast<const Node16*>(base + h.nodes_offset),
                            reinterpret_cast<const int64_t*>(base + h.table_offset), n_trees, X, n_rows, ld,
                            static_cast<int32_t*>(cnt.p), stream);
    if (rc) return rc;
    e = hipMemcpyAsync(counts, cnt.p, sizeof(int32_t) * (size_t)h.n_nodes, hipMemcpyDeviceToHost, stream);
    if (e == hipSuccess) e = hipStreamSynchronize(stream);
    if (e != hipSuccess) return fp_set_error(FP_EHIP, "counts: %s", hipGetErrorString(e));
    return FP_OK;
}

int launch_fill(int32_t* p, int64_t n, int32_t v, hipStream_t s) {
    if (n <= 0) return FP_OK;
    hipLaunchKernelGGL(fill_i32_kernel, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)), dim3(256), 0, s, p, n, v);
    return check_launch("fill_i32_kernel");
}

int launch_argmax(const int32_t* votes, int32_t* cls, int64_t n, int32_t C, hipStream_t s) {
    if (n <= 0) return FP_OK;
    hipLaunchKernelGGL(argmax_kernel, dim3((unsigned)std::min<int64_t>((n + 255) / 256, 4096)), dim3(256), 0, s, votes,
                       cls, n, C);
    return check_launch("argmax_kernel");
}

int launch_packed(const JobDesc& j, int K, int threads, int blocks, hipStream_t s) {
    const void* fn = pick_packed(K, j.feat_lds ? 1 : 0, job_kind(j));
    if (!fn) return fp_set_error(FP_EINVAL, "cursors must be 1, 2, 4 or 8");
    JobDesc a = j;
    void* args[] = {&a};
    hipError_t e = hipLaunchKernel(fn, dim3(blocks), dim3(threads), args, (size_t)j.lds_bytes, s);
    if (e != hipSuccess) return fp_set_error(FP_EHIP, "packed_kernel launch: %s", hipGetErrorString(e));
    return FP_OK;
}

int launch_batched(const BatchedShape& sh, const JobDesc* jobs, const WorkItem* items, int32_t n_block_items, int32_t n_items,
                   int32_t* counters, hipStream_t s) {
    if (sh.atomics) {
        hipLaunchKernelGGL(batched_prologue_kernel, dim3(64, sh.n_jobs), dim3(256), 0, s, jobs);
        if (const int rc = check_launch("batched_prologue_kernel")) return rc;
    }
    const bool mixed = sh.mixed && n_block_items > 0 && n_items > n_block_items;
    if (mixed) {
        int32_t item_slot = (int32_t)round16(sh.lds[0]);
        void* args[] = {&jobs, &items, &n_block_items, &n_items, &counters, &item_slot};
        hipError_t e = hipLaunchKernel(pick_mixed(sh.K), dim3((unsigned)std::min<int64_t>(sh.resident[0], n_items)), dim3(sh.threads),
                                       args, (size_t)item_slot + kItemSlotBytes, s);
        if (e != hipSuccess) return fp_set_error(FP_EHIP, "batched_mixed_kernel launch: %s", hipGetErrorString(e));
    }
    for (int c = 0; c < 2 && !mixed; c++) {
        const WorkItem* list = items + (c == 0 ? 0 : n_block_items);
        int32_t n = c == 0 ? n_block_items : n_items - n_block_items;
        if (n == 0) continue;
        const void* fn = pick_batched(sh.K, c == 0);
        if (!fn) return fp_set_error(FP_EINVAL, "cursors must be 1, 2, 4 or 8");
        int32_t item_slot = (int32_t)round16(sh.lds[c]);
        int32_t* counter = counters + c;
        void* args[] = {&jobs, &list, &n, &counter, &item_slot};
        const int blocks = (int)std::max<int64_t>(1, std::min<int64_t>(sh.resident[c], n));
        hipError_t e = hipLaunchKernel(fn, dim3(blocks), dim3(sh.threads), args, (size_t)item_slot + kItemSlotBytes, s);
        if (e != hipSuccess) return fp_set_error(FP_EHIP, "batched_kernel launch: %s", hipGetErrorString(e));
    }
    if (sh.atomic_classes) {
        hipLaunchKernelGGL(batched_epilogue_kernel, dim3(64, sh.n_jobs), dim3(256), 0, s, jobs);
        return check_launch("batched_epilogue_kernel");
    }
    return FP_OK;
}

}  // namespace fp

// ---------------------------------------------------------------------------
// single-forest entry points
// ---------------------------------------------------------------------------
namespace {
// A launch of one forest in a packed layout: everything that the tune leaves
// open decided.
struct Launch {
    JobDesc j;
    int K, threads, blocks;
};

int resolve_launch(const fp_packed* p, const fp_tune* tune, const float* X, int64_t n_rows, int64_t ld, int32_t* votes,
                   int32_t* cls, const fp::DeviceProps& dp, Launch* L) {
    const fp::Header& h = p->hdr;
    // 16 waves a workgroup share its tile and the trees' tops (20,001 rows x
    // 784 features x 256 trees in blocks, 16-row tiles: 256 threads 142 us,
    // 1024 threads 102; COMPACT, 30,000 rows x 353 columns x 128 trees: 512
    // threads 168 us, 1024 threads 145).  In node layouts 8 for explicit tiles
    // and, with four cursors or more, which hold half the wavefronts, 8 (4
    // for many rows of a COMPACT forest that do not fill LDS); 8 for many rows
    // whose features come from memory: the L1 holds few of their lines
    const bool nodes = h.layout < FP_LAYOUT_BLOCKED, many = n_rows >= 16 * (int64_t)dp.cus;
    int threads = tune && tune->block_threads > 0                              ? tune->block_threads
                  : tune && nodes && tune->cursors >= 4
                      ? (h.layout == FP_LAYOUT_COMPACT && many && h.n_used_features <= 512 ? 256 : 512)
                  : tune && ((nodes && tune->rows_per_block > 0) || (many && tune->feature_lds < 0)) ? 512
                                                                               : 1024;
    if (threads % 64 || threads < 64 || threads > 1024)
        return fp_set_error(FP_EINVAL, "block_threads %d must be a multiple of 64 in [64, 1024]", threads);
    // one walk per lane: more cost registers and gain nothing (100,003 rows x
    // 64 trees: one 214 us, two 227)
    const int K = tune && tune->cursors > 0 ? tune->cursors : 1;
    if (K != 1 && K != 2 && K != 4 && K != 8) return fp_set_error(FP_EINVAL, "cursors must be 1, 2, 4 or 8");
    const size_t lds_max = dp.lds_per_block ? dp.lds_per_block : 65536;
    if (tune && tune->lds_bytes < 0) return fp_set_error(FP_EINVAL, "lds_bytes %d < 0", tune->lds_bytes);
    const size_t lds_block = tune && tune->lds_bytes > 0      ? std::min((size_t)tune->lds_bytes, lds_max)
                             : tune && tune->lds_top_nodes > 0 ? lds_max
                                                               : fp::default_lds_block(dp);
    fp_tune at = tune ? *tune : fp_tune{};
    at.block_threads = threads;
    JobDesc& j = L->j;
    int rc = fp::resolve_job(p, &at, X, n_rows, ld, votes, cls, lds_block, dp.cus, &j);
    if (rc) return rc;
    // 8 wavefronts also for an automatic tile that has far fewer walks than
    // 1,024 (nodes), or of few rows in half of the usual LDS, which leaves
    // room for two more workgroups a CU
    if (!(tune && tune->block_threads > 0) && threads == 1024 && at.rows_per_block <= 0 &&
        (nodes ? j.R * j.trees_per_group < 768 : j.R < 16 && 2 * lds_block <= fp::default_lds_block(dp))) {
        threads = at.block_threads = 512;
        rc = fp::resolve_job(p, &at, X, n_rows, ld, votes, cls, lds_block, dp.cus, &j);
        if (rc) return rc;
    }
    int occ = 1;
    rc = fp::packed_occupancy(K, j, threads, &occ);
    if (rc) return rc;
    const int64_t resident = std::max<int64_t>(1, (int64_t)dp.cus * occ / j.G);  // workgroups of a group
    if ((!nodes || at.rows_per_block <= 0) && j.n_tiles > resident) {
        // full rounds of tiles: rows spread evenly, so that the last round
        // does not leave most workgroups idle (2M rows in 768-row tiles, 10.2
        // rounds of 256: 7.04 ms, 11 full ones 6.38).  An automatic tile may
        // grow for a round less if it still fits (20,001 rows x 784 features:
        // 3 rounds of 14 rows 113 us, 2 of 20 100)
        const bool grow = !tune || tune->rows_per_block <= 0;
        const int64_t rounds = (j.n_tiles + resident - 1) / resident;
        for (int64_t r = grow && rounds <= 4 ? rounds - 1 : rounds; r <= rounds; r++) {
            fp_tune even = at;
            even.rows_per_block = (int32_t)std::min<int64_t>(4096, (n_rows + r * resident - 1) / (r * resident));
            if (even.rows_per_block == j.R || even.rows_per_block > j.R + j.R / 4) continue;
            fp::JobDesc e;
            int occ_e = 0;
            if (fp::resolve_job(p, &even, X, n_rows, ld, votes, cls, lds_block, dp.cus, &e) == FP_OK &&
                fp::packed_occupancy(K, e, threads, &occ_e) == FP_OK && e.feat_lds == j.feat_lds && e.G == j.G &&
                occ_e == occ) {
                j = e;
                break;
            }
            fp_clear_error();
        }
    }
    const int64_t per_group = std::min<int64_t>(j.n_tiles, resident);
    L->K = K;
    L->threads = threads;
    L->blocks = (int)std::max<int64_t>(1, per_group) * j.G;
    return FP_OK;
}
}  // namespace

static int predict_impl(const fp_packed* p, const fp_tune* tune, const float* X, int64_t n_rows, int64_t ld,
                        int32_t* votes, int32_t* cls, void* stream_v) {
    fp_clear_error();
    if (!p) return fp_set_error(FP_EINVAL, "packed forest is NULL");
    const fp::Header& h = p->hdr;
    if (n_rows < 0 || n_rows > INT32_MAX) return fp_set_error(FP_EINVAL, "n_rows %lld outside [0, 2^31)", (long long)n_rows);
    if (ld < h.n_features) return fp_set_error(FP_EINVAL, "ld %lld < n_features %d", (long long)ld, h.n_features);
    if (n_rows == 0) return FP_OK;
    if (!X || !votes) return fp_set_error(FP_EINVAL, "X or votes is NULL");
    if (!p->dev) return fp_set_error(FP_ENODEV, "packed forest is not uploaded");
    int dev = -1;
    int rc = fp::current_device(&dev);
    if (rc) return rc;
    if (dev != p->dev_id) return fp_set_error(FP_ENODEV, "forest uploaded to device %d, current device is %d", p->dev_id, dev);
    fp::DeviceProps dp;
    rc = fp::device_props(dev, &dp);
    if (rc) return rc;
    hipStream_t stream = static_cast<hipStream_t>(stream_v);
    if (h.layout == FP_LAYOUT_NAIVE) {
        const int threads = tune && tune->block_threads > 0 ? tune->block_threads : 256;
        if (threads % 64 || threads < 64 || threads > 1024)
            return fp_set_error(FP_EINVAL, "block_threads %d must be a multiple of 64 in [64, 1024]", threads);
        const uint8_t* base = static_cast<const uint8_t*>(p->dev);
        NaiveArgs a{reinterpret_cast<const int64_t*>(base + h.table_offset),
                    reinterpret_cast<const Node16*>(base + h.nodes_offset), X, ld, n_rows, votes, cls, h.n_trees,
                    h.n_classes};
        const size_t lds = (size_t)h.n_classes * threads * 4;
        const bool use_lds = lds <= 32768;
        const int blocks = (int)((n_rows + threads - 1) / threads);
        if (use_lds)
            hipLaunchKernelGGL(naive_kernel<true>, dim3(blocks), dim3(threads), lds, stream, a);
        else
            hipLaunchKernelGGL(naive_kernel<false>, dim3(blocks), dim3(threads), 0, stream, a);
        return check_launch("naive_kernel");
    }

    Launch L;
    rc = resolve_launch(p, tune, X, n_rows, ld, votes, cls, dp, &L);
    if (rc) return rc;
    const fp::JobDesc& j = L.j;
    if (j.atomic_votes) {
        rc = fp::launch_fill(votes, n_rows * h.n_classes, 0, stream);
        if (rc) return rc;
    }
    // one launch per pass; with one group per pass the first stores the votes
    // and later ones add to them (the last also writes the classes), with
    // several concurrent groups every pass adds with atomics
    for (int pass = 0; pass < j.passes; pass++) {
        fp::JobDesc jp = j;
        jp.group_base = pass * j.G;
        jp.accumulate = !j.atomic_votes && pass > 0;
        jp.cls = (!j.atomic_votes && pass == j.passes - 1) ? cls : nullptr;
        rc = fp::launch_packed(jp, L.K, L.threads, L.blocks, stream);
        if (rc) return rc;
    }
    if (j.atomic_votes && cls) return fp::launch_argmax(votes, cls, n_rows, h.n_classes, stream);
    return FP_OK;
}

namespace fp {
int default_launch(const fp_packed* p, const float* X, int64_t n_rows, int64_t ld, int32_t threads, int32_t cursors,
                   int32_t* votes, fp_tune* out) {
    int dev = -1;
    int rc = current_device(&dev);
    if (rc) return rc;
    DeviceProps dp;
    rc = device_props(dev, &dp);
    if (rc) return rc;
    fp_tune t{};
    t.block_threads = threads;
    t.cursors = cursors;
    Launch L;
    rc = resolve_launch(p, &t, X, n_rows, ld, votes, nullptr, dp, &L);
    if (rc) return rc;
    *out = fp_tune{};
    out->rows_per_block = L.j.R;
    out->cursors = L.K;
    out->tree_groups = L.j.G;
    out->block_threads = L.threads;
    out->refill_lanes = L.j.refill_min;
    if (p->hdr.layout < FP_LAYOUT_BLOCKED && L.threads <= 512) out->lds_bytes = L.j.lds_bytes;  // its share of a CU
    return FP_OK;
}
}  // namespace fp

// The launch parameters: the tune recorded for p's batch-size bucket
// (fp_tune_launch, this process or the FP_TUNE_CACHE file), else p's own.
extern "C" int fp_predict(const fp_packed* p, const float* X_dev, int64_t n_rows, int64_t ld, int32_t* votes_dev,
                          int32_t* class_dev, void* stream) {
    if (!p) return fp_set_error(FP_EINVAL, "packed forest is NULL");
    fp_tune t;
    if (p->hdr.layout != FP_LAYOUT_NAIVE && n_rows > 0 && fp::launch_tune_get(p, n_rows, 0, 0, &t))
        return predict_impl(p, &t, X_dev, n_rows, ld, votes_dev, class_dev, stream);
    return predict_impl(p, &p->tune, X_dev, n_rows, ld, votes_dev, class_dev, stream);
}

extern "C" int fp_predict_tune_get(const fp_packed* p, int64_t n_rows, fp_tune* out, int32_t* source) {
    fp_clear_error();
    if (!p || !out) return fp_set_error(FP_EINVAL, "NULL argument");
    int32_t src = p->has_tune ? 1 : 0;
    *out = p->tune;
    fp_tune t;
    if (p->hdr.layout != FP_LAYOUT_NAIVE && n_rows > 0 && fp::launch_tune_get(p, n_rows, 0, 0, &t)) {
        *out = t;
        src = 2;
    }
    if (source) *source = src;
    return FP_OK;
}

extern "C" int fp_predict_tuned(const fp_packed* p, const fp_tune* tune, const float* X_dev, int64_t n_rows,
                                int64_t ld, int32_t* votes_dev, int32_t* class_dev, void* stream) {
    if (!p) return fp_set_error(FP_EINVAL, "packed forest is NULL");
    return predict_impl(p, tune ? tune : &p->tune, X_dev, n_rows, ld, votes_dev, class_dev, stream);
}
