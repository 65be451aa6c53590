// The two scans of a syndrome by segments (raa.hip, p1 and p2), as the part of one
// workgroup of kSegThreads threads: shared by the syndrome launches, the gather
// launch that holds the second one (prepare.hip) and the decode/verify of long
// blocks (client.hip).
#pragma once
#include "field.h"
#include "mvk_internal.h"
#include "syn_block.h"

namespace mvk {
namespace synseg {

using syn::wave_incl_scan_dpp;

constexpr int kSegThreads = 256;
constexpr int kSegPer = 4;
constexpr uint32_t kSegLen = kSegThreads * kSegPer;
static_assert(kSegLen == kSynSegLen, "segment length of the scratch layout");
// Bound on the polls of one look-back read (each followed by a short sleep):
// every awaited segment belongs to a workgroup that is already running, so the
// bound is only a guard that makes every wave exit.
constexpr uint32_t kLookSpinLimit = 1u << 22;

__device__ __forceinline__ unsigned long long* look_state(uint32_t* scratch, uint32_t count, uint32_t N, uint32_t c) {
    const uint32_t nseg = (N + kSegLen - 1) / kSegLen;
    return reinterpret_cast<unsigned long long*>(scratch + (size_t)count * 2 * N) + (size_t)c * (nseg + 1);
}

__device__ __forceinline__ uint64_t block_sum_u64_256(uint64_t v, uint64_t* red) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) {
        const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)v, s);
        const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(v >> 32), s);
        v += ((uint64_t)hi << 32) | lo;
    }
    if (lane == 0) red[wave] = v;
    __syncthreads();
    const uint64_t t = red[0] + red[1] + red[2] + red[3];
    __syncthreads();
    return t;
}

// A workgroup takes NS stripes of kSegLen positions, a segment of NS kSegLen:
// thread t holds positions kSegLen v + kSegPer t + e of its segment as [v][e],
// so that every access of four words is coalesced.  A segment costs its
// workgroup a chain of dependent memory accesses (ticket, loads, publication,
// look-back) of about 7 us whatever its length; with many vectors four stripes
// pay it for a quarter of the workgroups (seg_shape).
//
// kSegPer consecutive words from position j on (those from `end` on read
// position `end` - 1; j may lie past it).
__device__ __forceinline__ void load_seg(const uint32_t* p, uint32_t j, uint32_t end, uint32_t (&x)[kSegPer]) {
    typedef uint32_t u32x4_w __attribute__((ext_vector_type(4), aligned(4)));
    static_assert(kSegPer == 4, "one load of four words");
    if (j + kSegPer <= end) {
        const u32x4_w v = *reinterpret_cast<const u32x4_w*>(p + j);
        x[0] = v.x, x[1] = v.y, x[2] = v.z, x[3] = v.w;
    } else {
#pragma unroll
        for (int e = 0; e < kSegPer; ++e) x[e] = p[j + e < end ? j + e : end - 1];
    }
}

// Inclusive suffix scan of a segment, plus `carry`.
template <int NS>
__device__ __forceinline__ void seg_suffix_scan(uint32_t (&x)[NS][kSegPer], uint32_t carry, uint32_t (*wsum)[4]) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    uint32_t incl[NS];
#pragma unroll
    for (int v = 0; v < NS; ++v) {
#pragma unroll
        for (int e = kSegPer - 2; e >= 0; --e) x[v][e] = fadd(x[v][e], x[v][e + 1]);
        incl[v] = wave_incl_scan_dpp(x[v][0]);  // prefix over lanes of thread totals
        if (lane == 63) wsum[v][wave] = incl[v];
    }
    __syncthreads();
#pragma unroll
    for (int v = NS - 1; v >= 0; --v) {
        const uint32_t w0 = wsum[v][0], w1 = wsum[v][1], w2 = wsum[v][2], w3 = wsum[v][3];
        const uint32_t total = fadd(fadd(w0, w1), fadd(w2, w3));
        uint32_t before = 0;  // totals of earlier waves
        if (wave > 0) before = w0;
        if (wave > 1) before = fadd(before, w1);
        if (wave > 2) before = fadd(before, w2);
        // sum over later threads = total - (prefix through this thread)
        const uint32_t off = fadd(fsub(total, fadd(before, incl[v])), carry);
#pragma unroll
        for (int e = 0; e < kSegPer; ++e) x[v][e] = fadd(x[v][e], off);
        carry = fadd(carry, total);
    }
}

// Vectors of one sequence of launches (grid.y).
constexpr uint32_t kMaxVectors = 65535u;
// A set of `count` vectors over one code, with its work region.
struct SegSet {
    const uint32_t *pi1, *pi2, *v1, *v2;
    const uint32_t *vin, *idx, *val, *X;
    uint32_t* out;
    uint32_t* work;
    uint32_t k, r, t, count;
};
// Several syndromes share each of the launches (long blocks, and short ones that
// join them): set i is count vectors over its own code, with its own work region
// (count x 2N words and the look-back state).  grid.y runs over the vectors of all sets, grid.x
// over the segments (p1, p2) or the fold chunks (p3) of the longest; the
// workgroups past a shorter set's end return at once (before p2's ticket).
struct SegArgs {
    uint32_t S;
    uint32_t by_xcd;             // vectors [0, by_xcd) are placed by XCD (seg_place)
    uint32_t vend[kMaxSynSets];  // vectors of sets < i + 1
    SegSet set[kMaxSynSets];
};

// Which vector and segment a workgroup of the (segments, vectors) grid takes.
// Workgroups go to the 8 XCDs in turn by their linear index, and each XCD has
// its own L2.  The scatters write 4-byte words all over a vector's work array:
// with a vector's segments on every XCD each L2 held a few words of every line,
// and the lines went to memory in pieces.  Vectors below by_xcd (a multiple of
// 8) are taken eight at a time, one per XCD, so that one L2 collects whole
// lines; the vectors left over keep the plain order, which spreads each over
// the chip.
constexpr uint32_t kXcds = 8;
__device__ __forceinline__ void seg_place(const SegArgs& a, uint32_t bx, uint32_t by, uint32_t gx, uint32_t* vy,
                                          uint32_t* seg) {
    if (by >= a.by_xcd) {
        *vy = by;
        *seg = bx;
        return;
    }
    const uint32_t within = bx + gx * (by % kXcds);  // of eight vectors' workgroups
    *vy = by - by % kXcds + within % kXcds;
    *seg = within / kXcds;
}

// The set of global vector vy (grid.y) and the vector's index within it.
__device__ __forceinline__ const SegSet& seg_set(const SegArgs& a, uint32_t vy, uint32_t* c) {
    uint32_t i = 0;
    while (vy >= a.vend[i]) ++i;
    *c = vy - (i ? a.vend[i - 1] : 0u);
    return a.set[i];
}

// The grid of the passes over a set of sets: gx workgroups (segments) for each of
// `rows` vectors (some of them empty places), `stripes` per workgroup.
struct SegShape {
    uint32_t gx, rows, stripes, maxk;
};
// The arguments for S sparse sets with their work regions in scratch (false:
// too little of it, or too many vectors); the shape (sets a.by_xcd); the first
// pass, the fold.  The second pass is seg_second_scatter.
bool seg_args(const SynSet* sets, uint32_t S, uint32_t* scratch, size_t scratch_bytes, SegArgs* out);
SegShape seg_shape(SegArgs& a);
hipError_t launch_seg_first(const SegArgs& a, const SegShape& h, hipStream_t s);
hipError_t launch_seg_last(const SegArgs& a, const SegShape& h, hipStream_t s);

// Segments of a block of N positions.
template <int NS>
__host__ __device__ inline uint32_t seg_count(uint32_t N) {
    return (N + NS * kSegLen - 1) / (NS * kSegLen);
}

template <int NS>
struct SegLds {
    __align__(16) uint32_t seg[NS * kSegLen];
    uint64_t red[4];
    uint32_t wsum[NS][4];
    uint32_t sh_seg, sh_carry;
};

// p1 of segment sg of vector c.
template <bool SPARSE, int NS>
__device__ __forceinline__ void seg_first(const SegSet& S, uint32_t c, uint32_t sg, SegLds<NS>& lds) {
    constexpr uint32_t L = NS * kSegLen;
    const uint32_t N = S.k * S.r;
    const uint32_t j0 = sg * L, j1 = j0 + L < N ? j0 + L : N;
    const uint32_t tid = threadIdx.x, jt = j0 + tid * kSegPer;
    const uint32_t t = S.t;
    const uint32_t* __restrict__ idx = S.idx;
    const uint32_t* __restrict__ val = S.val;
    uint32_t* bbuf = S.work + (size_t)c * 2 * N;
    if (tid == 0) {
        // p2's look-back state: this segment's status word, and (segment 0) the ticket
        unsigned long long* st = look_state(S.work, S.count, N, c);
        st[1 + sg] = 0ull;
        if (sg == 0) st[0] = 0ull;
    }
    // code entries of this thread's positions (in flight during the carry)
    uint32_t p2[NS][kSegPer], w2[NS][kSegPer], x[NS][kSegPer];
#pragma unroll
    for (int v = 0; v < NS; ++v) {
        load_seg(S.pi2, jt + v * kSegLen, j1, p2[v]);
        load_seg(S.v2, jt + v * kSegLen, j1, w2[v]);
    }
    uint64_t part = 0;
    if (SPARSE) {
#pragma unroll
        for (int v = 0; v < NS; ++v)
#pragma unroll
            for (int e = 0; e < kSegPer; ++e) lds.seg[v * kSegLen + tid * kSegPer + e] = 0u;
        __syncthreads();
        for (uint32_t q = tid; q < t; q += kSegThreads) {
            const uint32_t j = idx[(size_t)c * t + q], u = val[(size_t)c * t + q];
            if (j >= j1 && j < N) part += u;
            if (j >= j0 && j < j1) lds.seg[j - j0] = u;
        }
    } else {
        const uint32_t* src = S.vin + (size_t)c * N;
#pragma unroll
        for (int v = 0; v < NS; ++v) {
            load_seg(src, jt + v * kSegLen, j1, x[v]);
#pragma unroll
            for (int e = 0; e < kSegPer; ++e)
                if (jt + v * kSegLen + e >= j1) x[v][e] = 0u;
        }
        for (uint32_t j = j1 + tid; j < N; j += kSegThreads) part += src[j];
    }
    const uint32_t carry = fred64(block_sum_u64_256(part, lds.red));  // (its barrier: the terms are in LDS)
    if (SPARSE) {
#pragma unroll
        for (int v = 0; v < NS; ++v)
#pragma unroll
            for (int e = 0; e < kSegPer; ++e) x[v][e] = lds.seg[v * kSegLen + tid * kSegPer + e];
    }
    seg_suffix_scan<NS>(x, carry, lds.wsum);  // A
#pragma unroll
    for (int v = 0; v < NS; ++v)
#pragma unroll
        for (int e = 0; e < kSegPer; ++e)
            if (jt + v * kSegLen + e < j1)
                bbuf[p2[v][e] < N ? p2[v][e] : N - 1] = fmul(w2[v][e], x[v][e]);  // V2, then Pi2 scatter
}

// p2 of the segment that this workgroup is given (returned), in two parts.  The
// first loads its positions, with p1 and w1 the entries of Pi1 and V1, and
// publishes its sum; the second (seg_second_scan) turns x into the second suffix
// sum (meaningless from N on).  Loads that depend on p1 go between them: the
// look-back then hides them.
template <int NS>
__device__ __forceinline__ uint32_t seg_second_load(const SegSet& S, uint32_t c, SegLds<NS>& lds,
                                               uint32_t (&x)[NS][kSegPer], uint32_t (&p1)[NS][kSegPer],
                                               uint32_t (&w1)[NS][kSegPer]) {
    constexpr uint32_t L = NS * kSegLen;
    const uint32_t N = S.k * S.r, nseg = seg_count<NS>(N);
    const uint32_t tid = threadIdx.x;
    unsigned long long* st = look_state(S.work, S.count, N, c);
    if (tid == 0) {
        const uint32_t ticket = atomicAdd(reinterpret_cast<uint32_t*>(st), 1u);  // < nseg: one per workgroup
        lds.sh_seg = ticket < nseg ? nseg - 1 - ticket : 0u;
    }
    __syncthreads();
    const uint32_t sg = lds.sh_seg;
    const uint32_t j0 = sg * L, j1 = j0 + L < N ? j0 + L : N, jt = j0 + tid * kSegPer;
    const uint32_t* bbuf = S.work + (size_t)c * 2 * N;
    uint64_t part = 0;
#pragma unroll
    for (int v = 0; v < NS; ++v) {
        load_seg(bbuf, jt + v * kSegLen, j1, x[v]);
        load_seg(S.pi1, jt + v * kSegLen, j1, p1[v]);
        load_seg(S.v1, jt + v * kSegLen, j1, w1[v]);
    }
#pragma unroll
    for (int v = 0; v < NS; ++v)
#pragma unroll
        for (int e = 0; e < kSegPer; ++e) {
            if (jt + v * kSegLen + e >= j1) x[v][e] = 0u;
            part += x[v][e];
        }
    // publish this segment's sum
    const uint32_t own = fred64(block_sum_u64_256(part, lds.red));
    if (tid == 0) __hip_atomic_store(&st[1 + sg], (1ull << 32) | own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    return sg;
}

template <int NS>
__device__ __forceinline__ void seg_second_scan(const SegSet& S, uint32_t c, uint32_t sg, SegLds<NS>& lds,
                                                uint32_t (&x)[NS][kSegPer]) {
    const uint32_t N = S.k * S.r, nseg = seg_count<NS>(N);
    const uint32_t tid = threadIdx.x, lane = tid & 63;
    unsigned long long* st = look_state(S.work, S.count, N, c);
    // carry = sum of the later segments' sums, read 64 segments at a time
    if (tid < 64) {
        uint64_t acc = 0;
        for (uint32_t base = sg + 1; base < nseg; base += 64) {
            const uint32_t q = base + lane;
            if (q < nseg) {
                unsigned long long v = __hip_atomic_load(&st[1 + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                for (uint32_t spin = 0; !(v >> 32) && spin < kLookSpinLimit; ++spin) {
                    __builtin_amdgcn_s_sleep(1);
                    v = __hip_atomic_load(&st[1 + q], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
                acc += (uint32_t)v;
            }
        }
#pragma unroll
        for (int sh = 32; sh >= 1; sh >>= 1) {
            const uint32_t lo = (uint32_t)__shfl_xor((int)(uint32_t)acc, sh);
            const uint32_t hi = (uint32_t)__shfl_xor((int)(uint32_t)(acc >> 32), sh);
            acc += ((uint64_t)hi << 32) | lo;
        }
        if (tid == 0) lds.sh_carry = fred64(acc);
    }
    __syncthreads();
    seg_suffix_scan<NS>(x, lds.sh_carry, lds.wsum);  // A
}

// p2 of workgroup (bx, by) of a grid gx wide.
template <int NS>
__device__ __forceinline__ void seg_second_scatter(const SegArgs& a, uint32_t bx, uint32_t by, uint32_t gx,
                                                   SegLds<NS>& lds) {
    uint32_t c, vy, place;
    seg_place(a, bx, by, gx, &vy, &place);
    if (vy >= a.vend[a.S - 1]) return;
    const SegSet& S = seg_set(a, vy, &c);
    const uint32_t N = S.k * S.r;
    if (place >= seg_count<NS>(N)) return;  // (uniform: no ticket taken)
    uint32_t x[NS][kSegPer], p1[NS][kSegPer], w1[NS][kSegPer];
    const uint32_t sg = seg_second_load<NS>(S, c, lds, x, p1, w1);
    seg_second_scan<NS>(S, c, sg, lds, x);
    const uint32_t j0 = sg * NS * kSegLen + threadIdx.x * kSegPer;
    uint32_t* dbuf = S.work + (size_t)c * 2 * N + N;
#pragma unroll
    for (int v = 0; v < NS; ++v)
#pragma unroll
        for (int e = 0; e < kSegPer; ++e)
            if (j0 + v * kSegLen + e < N)
                dbuf[p1[v][e] < N ? p1[v][e] : N - 1] = fmul(w1[v][e], x[v][e]);  // V1, then Pi1 scatter
}

}  // namespace synseg
}  // namespace mvk
