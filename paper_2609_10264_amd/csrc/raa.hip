// RAA code maps (App. B) on gfx950.
//
//   encoding  G^T w = A^T V2 Pi2^T A^T V1 Pi1^T R^T w   (repeat, gather by pi1,
//             scale, prefix sum, gather by pi2, scale, prefix sum)
//   syndrome  G v   = R Pi1 V1 A Pi2 V2 A v             (suffix sum, scale,
//             scatter by pi2, suffix sum, scale, scatter by pi1, fold r)
//
// Kernel shapes:
//  * enc_pass1/2: many vectors at once (Preprocess encodes every row and every
//    column of W).  One lane owns one vector within a segment of positions, so
//    each prefix sum is a running sum per lane plus a scan over segments, and
//    every access to the batch (vector index innermost) is a coalesced row.
//    The code arrays are indexed by the position only, which is uniform across
//    the workgroup, so they come through scalar loads.
//  * enc_seg: the same for many vectors of an int8 matrix (from 2048 vectors and
//    192 MB of intermediate sums on), the value of both prefix sums before every
//    segment from one server product in place of the passes that add up segments.
//  * syn_wg: few vectors (Encrypt: one per query column; Verify: one per
//    repetition) of length up to 16384.  One 1024-thread workgroup owns one
//    vector; both work arrays stay in LDS.
//  * syn_p1/p2/p3: longer vectors (and shorter ones that go with them), cut into
//    segments over three launches.
#include "field.h"
#include "mvk_internal.h"
#include "syn_block.h"
#include "syn_seg.h"

#include <type_traits>

namespace mvk {

namespace {

__device__ __forceinline__ uint32_t load_elem(const uint32_t* p, size_t i) { return p[i]; }
__device__ __forceinline__ uint32_t load_elem(const int8_t* p, size_t i) { return femb(p[i]); }

template <int RR>
__device__ __forceinline__ uint32_t div_r(uint32_t x, uint32_t r) {
    if constexpr (RR > 0)
        return x / RR;
    else
        return x / r;
}

// Batched encoding.  The N positions are cut into segments of L positions
// (L from enc_seg_len), and a one-wave workgroup takes one segment for 64*V
// vectors (V consecutive vectors per lane; vectors innermost in every array,
// so each position is one coalesced row).  Each prefix sum is a reduce, a
// scan over the segment sums, then a second pass that starts every segment
// from its offset (so no output is written twice):
//   sum 1     tot[s][v] = sum over segment s of v1[j] * w_v[pi1[j] / r]
//   scan      off[s][v] = sum of tot[s'][v] for s' < s
//   write 1   t3[j][v] = off[seg(j)][v] + running sum within the segment
//   sum 2, scan, write 2: the same with v2[j] * t3[pi2[j]][v] into out[j][v]
// Every output is the field sum of the same terms as one running sum over all N
// positions; field addition is exact, so the grouping does not change it.
constexpr int kEncLanes = 64;

// Segment length: the longest of 256, 128, 64 that still gives at least 2048
// workgroups (eight waves per compute unit) at four vectors per lane.
uint32_t enc_seg_len(size_t N, size_t nvec) {
    const size_t vg = (nvec + 4 * kEncLanes - 1) / (4 * kEncLanes);
    for (uint32_t L : {256u, 128u})
        if (((N + L - 1) / L) * vg >= 2048) return L;
    return 64u;
}

template <int V>
struct Lanes {
    uint32_t x[V];
};

// V elements (vectors vb .. vb+V-1, stride vs) of one position
template <int V>
__device__ __forceinline__ Lanes<V> load_lanes(const uint32_t* p, size_t vs) {
    Lanes<V> r;
    if constexpr (V == 4) {
        const uint4 q = *(const uint4*)p;
        r.x[0] = q.x, r.x[1] = q.y, r.x[2] = q.z, r.x[3] = q.w;
    } else {
#pragma unroll
        for (int q = 0; q < V; ++q) r.x[q] = p[q * vs];
    }
    return r;
}
template <int V>
__device__ __forceinline__ Lanes<V> load_lanes(const int8_t* p, size_t vs) {
    Lanes<V> r;
    if constexpr (V == 4) {
        const uint32_t w = *(const uint32_t*)p;
#pragma unroll
        for (int q = 0; q < 4; ++q) r.x[q] = femb((int8_t)(w >> (8 * q)));
    } else {
#pragma unroll
        for (int q = 0; q < V; ++q) r.x[q] = femb(p[q * vs]);
    }
    return r;
}
template <int V>
__device__ __forceinline__ void store_lanes(uint32_t* p, size_t vs, const Lanes<V>& v) {
    if constexpr (V == 4) {
        *(uint4*)p = make_uint4(v.x[0], v.x[1], v.x[2], v.x[3]);
    } else {
#pragma unroll
        for (int q = 0; q < V; ++q) p[q * vs] = v.x[q];
    }
}

// First prefix sum (over v1 .* Pi1^T R^T w).  WRITE = false: segment sums
// into tot; WRITE = true: t3 from the offsets in off.
template <typename T, int RR, int V, bool WRITE>
__global__ __launch_bounds__(kEncLanes) void enc_pass1(uint32_t N, uint32_t r, uint32_t L,
                                                       const uint32_t* __restrict__ pi1,
                                                       const uint32_t* __restrict__ v1, const T* __restrict__ in,
                                                       size_t ld_in, size_t vs_in, uint32_t nvec,
                                                       const uint32_t* __restrict__ off, uint32_t* __restrict__ t3,
                                                       uint32_t* __restrict__ tot) {
    const uint32_t seg = blockIdx.x, vb = (blockIdx.y * kEncLanes + threadIdx.x) * V;
    if (vb >= nvec) return;
    const T* src = in + (size_t)vb * vs_in;
    const uint32_t j0 = seg * L, j1 = j0 + L < N ? j0 + L : N;
    Lanes<V> acc;
    if (WRITE)
        acc = load_lanes<V>(off + (size_t)seg * nvec + vb, 1);
    else
#pragma unroll
        for (int q = 0; q < V; ++q) acc.x[q] = 0;
#pragma unroll 8
    for (uint32_t j = j0; j < j1; ++j) {
        uint32_t pj = pi1[j];
        if (pj >= N) pj = N - 1;
        const Lanes<V> x = load_lanes<V>(src + (size_t)div_r<RR>(pj, r) * ld_in, vs_in);
        const uint32_t c = v1[j];
#pragma unroll
        for (int q = 0; q < V; ++q) acc.x[q] = fadd(acc.x[q], fmul(c, x.x[q]));
        if (WRITE) store_lanes<V>(t3 + (size_t)j * nvec + vb, 1, acc);
    }
    if (!WRITE) store_lanes<V>(tot + (size_t)seg * nvec + vb, 1, acc);
}

// Second prefix sum (over v2 .* Pi2^T t3), the same two forms, into out.
template <int V, bool WRITE>
__global__ __launch_bounds__(kEncLanes) void enc_pass2(uint32_t N, uint32_t L, const uint32_t* __restrict__ pi2,
                                                       const uint32_t* __restrict__ v2,
                                                       const uint32_t* __restrict__ t3, uint32_t nvec,
                                                       const uint32_t* __restrict__ off, uint32_t* __restrict__ out,
                                                       size_t ld_out, size_t vs_out, uint32_t* __restrict__ tot) {
    const uint32_t seg = blockIdx.x, vb = (blockIdx.y * kEncLanes + threadIdx.x) * V;
    if (vb >= nvec) return;
    uint32_t* dst = out + (size_t)vb * vs_out;
    const uint32_t j0 = seg * L, j1 = j0 + L < N ? j0 + L : N;
    Lanes<V> acc;
    if (WRITE)
        acc = load_lanes<V>(off + (size_t)seg * nvec + vb, 1);
    else
#pragma unroll
        for (int q = 0; q < V; ++q) acc.x[q] = 0;
#pragma unroll 8
    for (uint32_t j = j0; j < j1; ++j) {
        uint32_t pj = pi2[j];
        if (pj >= N) pj = N - 1;
        const Lanes<V> a = load_lanes<V>(t3 + (size_t)pj * nvec + vb, 1);
        const uint32_t c = v2[j];
#pragma unroll
        for (int q = 0; q < V; ++q) acc.x[q] = fadd(acc.x[q], fmul(c, a.x[q]));
        if (WRITE) store_lanes<V>(dst + (size_t)j * ld_out, vs_out, acc);
    }
    if (!WRITE) store_lanes<V>(tot + (size_t)seg * nvec + vb, 1, acc);
}

// off[s][v] = sum_{s' < s} tot[s'][v] for every vector v (one thread each)
__global__ __launch_bounds__(256) void enc_scan(uint32_t nseg, uint32_t nvec, const uint32_t* __restrict__ tot,
                                                uint32_t* __restrict__ off) {
    const uint32_t v = blockIdx.x * 256 + threadIdx.x;
    if (v >= nvec) return;
    uint32_t run = 0;
#pragma unroll 8
    for (uint32_t sg = 0; sg < nseg; ++sg) {
        const uint32_t t = tot[(size_t)sg * nvec + v];
        off[(size_t)sg * nvec + v] = run;
        run = fadd(run, t);
    }
}

template <typename T, int RR, int V>
hipError_t launch_enc_v(const mvk_code& c, const T* in, size_t ld_in, size_t vs_in, uint32_t nvec, uint32_t* t3,
                        uint32_t* tot, uint32_t* off, uint32_t* out, size_t ld_out, size_t vs_out, hipStream_t s) {
    const uint32_t N = c.k * c.r, L = enc_seg_len(N, nvec), nseg = ceil_div(N, L);
    const dim3 grid(nseg, ceil_div(nvec, kEncLanes * V)), block(kEncLanes), sgrid(ceil_div(nvec, 256u));
    hipLaunchKernelGGL((enc_pass1<T, RR, V, false>), grid, block, 0, s, N, c.r, L, c.pi1, c.v1, in, ld_in, vs_in,
                       nvec, nullptr, nullptr, tot);
    hipLaunchKernelGGL(enc_scan, sgrid, dim3(256), 0, s, nseg, nvec, tot, off);
    hipLaunchKernelGGL((enc_pass1<T, RR, V, true>), grid, block, 0, s, N, c.r, L, c.pi1, c.v1, in, ld_in, vs_in,
                       nvec, off, t3, nullptr);
    hipLaunchKernelGGL((enc_pass2<V, false>), grid, block, 0, s, N, L, c.pi2, c.v2, t3, nvec, nullptr, nullptr,
                       ld_out, vs_out, tot);
    hipLaunchKernelGGL(enc_scan, sgrid, dim3(256), 0, s, nseg, nvec, tot, off);
    hipLaunchKernelGGL((enc_pass2<V, true>), grid, block, 0, s, N, L, c.pi2, c.v2, t3, nvec, off, out, ld_out,
                       vs_out, nullptr);
    return hipGetLastError();
}

template <typename T, int RR>
hipError_t launch_enc_r(const mvk_code& c, const T* in, size_t ld_in, size_t vs_in, uint32_t nvec, uint32_t* t3,
                        uint32_t* tot, uint32_t* off, uint32_t* out, size_t ld_out, size_t vs_out, hipStream_t s) {
    // four vectors per lane when every lane's four elements are adjacent and aligned
    const size_t al = 4 * sizeof(T);
    const bool v4 = nvec % 4 == 0 && vs_in == 1 && ld_in % 4 == 0 && (uintptr_t)in % al == 0 && vs_out == 1 &&
                    ld_out % 4 == 0 && (uintptr_t)out % 16 == 0 && (uintptr_t)t3 % 16 == 0 &&
                    (uintptr_t)tot % 16 == 0 && (uintptr_t)off % 16 == 0;
    if (v4) return launch_enc_v<T, RR, 4>(c, in, ld_in, vs_in, nvec, t3, tot, off, out, ld_out, vs_out, s);
    return launch_enc_v<T, RR, 1>(c, in, ld_in, vs_in, nvec, t3, tot, off, out, ld_out, vs_out, s);
}

template <typename T>
hipError_t launch_encT(const mvk_code& c, const T* in, size_t ld_in, size_t vs_in, uint32_t nvec, uint32_t* t3,
                       uint32_t* seg_scratch, uint32_t* out, size_t ld_out, size_t vs_out, hipStream_t s) {
    if (nvec == 0) return hipSuccess;
    if (nvec > kMaxEncVectors) return hipErrorInvalidValue;
    const uint32_t N = c.k * c.r;
    uint32_t* tot = seg_scratch;
    uint32_t* off = seg_scratch + (size_t)ceil_div(N, enc_seg_len(N, nvec)) * nvec;
    switch (c.r) {
        case 1: return launch_enc_r<T, 1>(c, in, ld_in, vs_in, nvec, t3, tot, off, out, ld_out, vs_out, s);
        case 2: return launch_enc_r<T, 2>(c, in, ld_in, vs_in, nvec, t3, tot, off, out, ld_out, vs_out, s);
        case 3: return launch_enc_r<T, 3>(c, in, ld_in, vs_in, nvec, t3, tot, off, out, ld_out, vs_out, s);
        case 4: return launch_enc_r<T, 4>(c, in, ld_in, vs_in, nvec, t3, tot, off, out, ld_out, vs_out, s);
        case 8: return launch_enc_r<T, 8>(c, in, ld_in, vs_in, nvec, t3, tot, off, out, ld_out, vs_out, s);
        default: return launch_enc_r<T, 0>(c, in, ld_in, vs_in, nvec, t3, tot, off, out, ld_out, vs_out, s);
    }
}

// ---------------------------------------------------------------------------
// Batched encoding of the rows of an int8 matrix M (nvec x k; Preprocess: W for
// P^T, W^T for Q) with the segment offsets taken from one server product.
//
// The value of either prefix sum just before a segment is a fixed linear map of
// the vector: with the segments starting at s L,
//   t3[s L - 1]  = D_s . w,  D_s[i]  = sum of v1[j] over j < s L, pi1[j] / r = i
//   out[s L - 1] = E_s . w,  E_s     = G e_(sL-1)  (the syndrome of a unit vector)
// so the offsets of every segment of every vector are the product of M with the
// 2 (nseg - 1) "queries" D_s, E_s (the matrix-core server product, exact), and
// neither prefix sum needs a pass that only adds up segments: t3 is written and
// read once, and the output written once.  (The three-pass form above read W and
// t3 twice: 1310 us for an 11008 x 4096 keygen at r = 3.)
// ---------------------------------------------------------------------------
constexpr uint32_t kSegWaves = 8;   // waves per workgroup
constexpr uint32_t kSegRows = 8;    // positions per wave and step
constexpr uint32_t kSegStep = kSegWaves * kSegRows;
constexpr uint32_t kSegVec = 256;   // vectors per workgroup (four per lane)

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
// (loads and stores of four words at any word, of one word at any byte)
typedef uint32_t u32x4_w __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32_b __attribute__((aligned(1)));

// The code arrays in the form the passes read, padded to whole steps (and one
// step more, which the passes load ahead) with coefficient 0: row1 = pi1 / r and
// row2 = pi2 (in range), c1, c1off, c2 as fmadd_c takes them.  Besides, pos =
// pi1^-1 and the unit vectors e_(sL-1), s = 1 .. nq, of the offsets.
__global__ __launch_bounds__(256) void enc_prep(uint32_t N, uint32_t npad, uint32_t r, uint32_t L, uint32_t nq,
                                                const uint32_t* __restrict__ pi1, const uint32_t* __restrict__ pi2,
                                                const uint32_t* __restrict__ v1, const uint32_t* __restrict__ v2,
                                                uint32_t* __restrict__ pos, uint32_t* __restrict__ row1,
                                                uint32_t* __restrict__ row2, uint32_t* __restrict__ c1,
                                                uint32_t* __restrict__ c1off, uint32_t* __restrict__ c2,
                                                uint32_t* __restrict__ idx, uint32_t* __restrict__ val) {
    const uint32_t j = blockIdx.x * 256 + threadIdx.x;
    if (j < nq) {
        idx[j] = (j + 1) * L - 1;
        val[j] = 1u;
    }
    if (j >= npad) return;
    const bool in = j < N;
    const uint32_t a = in ? pi1[j] : 0u, b = in ? pi2[j] : 0u;
    const uint32_t p1 = a < N ? a : N - 1;
    if (in) pos[p1] = j;
    row1[j] = p1 / r;
    row2[j] = b < N ? b : N - 1;
    c1[j] = in ? fcoef(v1[j]) : 0u;
    c1off[j] = in ? fcoef_off(v1[j]) : 0u;
    c2[j] = in ? fcoef(v2[j]) : 0u;
}

// D_s for s = s0+1 .. (grid.y ranges of kDqPer): D[s-1][i], row i per thread.
constexpr uint32_t kDqPer = 8;
__global__ __launch_bounds__(256) void enc_dq(uint32_t k, uint32_t r, uint32_t N, uint32_t L, uint32_t nq,
                                              const uint32_t* __restrict__ pos, const uint32_t* __restrict__ v1,
                                              uint32_t* __restrict__ D) {
    const uint32_t i = blockIdx.x * 256 + threadIdx.x, s0 = blockIdx.y * kDqPer;
    if (i >= k) return;
    uint64_t acc[kDqPer] = {};
    for (uint32_t q = 0; q < r; ++q) {
        uint32_t j = pos[(size_t)i * r + q];
        if (j >= N) j = N - 1;
        const uint32_t v = v1[j], sj = j / L;  // position j counts from segment sj + 1 on
#pragma unroll
        for (uint32_t e = 0; e < kDqPer; ++e) acc[e] += s0 + e >= sj ? v : 0u;
    }
#pragma unroll
    for (uint32_t e = 0; e < kDqPer; ++e)
        if (s0 + e < nq) D[(size_t)(s0 + e) * k + i] = fred64(acc[e]);
}

// One prefix sum of one segment of L positions for the 256 vectors of a tile
// (four per lane): FIRST: t3 from the int8 rows (in + row * nvec), else the
// output from t3.  t3 is held tile by tile (N rows of 256 words each).  Each
// step the waves take kSegRows consecutive positions each, sum them in
// registers, and add the totals of the waves before them (through LDS) and the
// segment's running offset.  The code entries (scalar loads of a whole step)
// are fetched two steps ahead and the rows one step ahead, unconditionally.
//
// Bound by HBM: the first sum writes 4 bytes an element and the second reads
// and writes 4.  At 11008 x 4096, r = 3 (541 MB of t3 and of output): 119 and
// 215 us, 4.6 and 5.0 TB/s, where a copy of 512 MB runs at 5.4 TB/s; the whole
// keygen 803 us.  t3 and the output are streamed with the non-temporal hint (950
// us without it); t3 kept for chunks of 36 to 256 MB of vectors, to stay in the
// memory-side cache between its write and its read, measured 890 to 1180 us:
// each launch then has too few workgroups.  The BabyBear build's second sum keeps
// 15 registers in scratch (128 is what four waves per SIMD leave) and is bound by
// HBM all the same: 4.3 GB in 774 us, 5.5 TB/s (8192 x 8192, r = 8).
struct SegIdx {
    uint32_t row[kSegRows];
};
template <bool FIRST>
__global__ __launch_bounds__(kSegWaves * 64, 4) void enc_seg(
    uint32_t N, uint32_t L, uint32_t nseg, uint32_t ntile, const uint32_t* __restrict__ rows,
    const uint32_t* __restrict__ coef, const uint32_t* __restrict__ coef_off, const int8_t* __restrict__ in,
    uint32_t nvec, const uint32_t* __restrict__ off, uint32_t* __restrict__ t3,
    uint32_t* __restrict__ out) {
    __shared__ u32x4 tot[2][kSegWaves][64];
    // (neighbouring workgroups take the tiles of one segment: adjacent output)
    const uint32_t seg = blockIdx.x / ntile, tile = blockIdx.x - seg * ntile;
    const int lane = threadIdx.x & 63;
    const uint32_t wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    // Lanes past the last vector take the last four, and positions past N
    // (coefficient 0: their sum is that of position N - 1) are stored to row
    // N - 1: both write what their neighbours write there, so every store is
    // unconditional and the waits can count them.
    const uint32_t vl = (uint32_t)lane * 4;
    const uint32_t vb = tile * kSegVec + vl + 4 <= nvec ? tile * kSegVec + vl : nvec - 4;
    t3 += (size_t)tile * N * kSegVec + vl;

    typedef typename std::conditional<FIRST, uint32_t, u32x4>::type Row;
    auto load_idx = [&](SegIdx& d, uint32_t j) { d = *reinterpret_cast<const SegIdx*>(rows + j); };
    auto load_rows = [&](Row(&x)[kSegRows], const SegIdx& d) {
#pragma unroll
        for (uint32_t e = 0; e < kSegRows; ++e) {
            if constexpr (FIRST)
                x[e] = *reinterpret_cast<const u32_b*>(in + (size_t)d.row[e] * nvec + vb);
            else
                x[e] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(t3 + (size_t)d.row[e] * kSegVec));
        }
    };
    uint32_t jw = seg * L + wave * kSegRows;  // this wave's positions of the current step
    SegIdx d;
    Row cur[kSegRows], nxt[kSegRows];
    load_idx(d, jw);
    load_rows(cur, d);
    load_idx(d, jw + kSegStep);
    u32x4 carry = {0u, 0u, 0u, 0u};
    if (seg) carry = *reinterpret_cast<const u32x4_w*>(off + (size_t)(seg - 1) * nvec + vb);
    auto step = [&](Row(&x)[kSegRows], Row(&y)[kSegRows], int buf) {
        load_rows(y, d);
        load_idx(d, jw + 2 * kSegStep);
        __builtin_amdgcn_sched_barrier(0);  // (the loads stay ahead of the arithmetic)
        const SegIdx c = *reinterpret_cast<const SegIdx*>(coef + jw);
        u32x4 a[kSegRows];
        u32x4 run = {0u, 0u, 0u, 0u};
        if constexpr (FIRST) {
            const SegIdx co = *reinterpret_cast<const SegIdx*>(coef_off + jw);
#pragma unroll
            for (uint32_t e = 0; e < kSegRows; ++e) {
                const uint32_t u = x[e] ^ 0x80808080u;
#pragma unroll
                for (int q = 0; q < 4; ++q) run[q] = fmadd_c8(run[q], c.row[e], co.row[e], (u >> (8 * q)) & 0xffu);
                a[e] = run;
            }
        } else {
#pragma unroll
            for (uint32_t e = 0; e < kSegRows; ++e) {
#pragma unroll
                for (int q = 0; q < 4; ++q) run[q] = fmadd_c(run[q], c.row[e], x[e][q]);
                a[e] = run;
            }
        }
        tot[buf][wave][lane] = run;
        __syncthreads();
        u32x4 before = carry;
#pragma unroll
        for (uint32_t w = 0; w < kSegWaves; ++w) {
            const u32x4 t = tot[buf][w][lane];
            if (w == wave) before = carry;
#pragma unroll
            for (int q = 0; q < 4; ++q) carry[q] = fmin_p(carry[q] + t[q]);
        }
#pragma unroll
        for (uint32_t e = 0; e < kSegRows; ++e) {
#pragma unroll
            for (int q = 0; q < 4; ++q) a[e][q] = fmin_p(a[e][q] + before[q]);
            const uint32_t j = jw + e < N ? jw + e : N - 1;
            if constexpr (FIRST)
                __builtin_nontemporal_store(a[e], reinterpret_cast<u32x4*>(t3 + (size_t)j * kSegVec));
            else
                __builtin_nontemporal_store((u32x4_w)a[e], reinterpret_cast<u32x4_w*>(out + (size_t)j * nvec + vb));
        }
        jw += kSegStep;
    };
    // two register sets in turn; segments are an even number of steps, so that
    // no step's loads are conditional
    for (uint32_t t = 0; t < L / kSegStep; t += 2) {
        step(cur, nxt, 0);
        step(nxt, cur, 1);
    }
}

// ---------------------------------------------------------------------------
// Syndrome of short blocks (N <= 16384): one 1024-thread workgroup per
// vector, the work arrays in LDS (syn_block.h).
// ---------------------------------------------------------------------------
constexpr int kSynThreads = 1024;
constexpr int kSynMaxU = 16;
static_assert((size_t)kSynThreads * kSynMaxU == kSynScratchAbove, "LDS syndrome covers the scratch-free range");
using namespace synseg;

template <bool SPARSE, int U>
__global__ __launch_bounds__(kSynThreads) void syn_wg(uint32_t k, uint32_t r, const uint32_t* __restrict__ pi1,
                                                      const uint32_t* __restrict__ pi2,
                                                      const uint32_t* __restrict__ v1,
                                                      const uint32_t* __restrict__ v2,
                                                      const uint32_t* __restrict__ vin,
                                                      const uint32_t* __restrict__ idx,
                                                      const uint32_t* __restrict__ val, uint32_t t,
                                                      const uint32_t* __restrict__ X, uint32_t* __restrict__ out) {
    __shared__ uint32_t lds[syn::lds_words<U, kSynThreads>()];
    syn::syn_block<SPARSE, U, kSynThreads, false>(blockIdx.x, k, r, pi1, pi2, v1, v2, vin, idx, val, t, X, out, lds);
}

// ---------------------------------------------------------------------------
// Multi-workgroup syndrome (several workgroups per vector).  The length-N work array
// is cut into segments, one workgroup each, of kSegLen positions or, with four
// stripes (seg_shape), of four times as many, in three launches; the second may
// run beside the row gathers of a preparation (prepare.hip), and the
// decode/verify of long blocks has its own first and second launch with the same
// parts (client.hip):
//   p1: a = suffix sum of the input (the carry into a segment is the sum of the
//       input beyond it: for sparse input a sum over the t terms, for dense
//       input a reduction of the tail), then b[pi2[j]] = v2[j] a[j]; p1 also
//       resets p2's look-back state
//   p2: c = suffix sum of b, then d[pi1[j]] = v1[j] c[j].  The carry into a
//       segment is the sum of the later segments' sums: every workgroup
//       publishes its segment's sum and reads the later ones (a single-pass
//       scan with look-back).  Segments are handed out by a ticket counter
//       from the last one down, so a workgroup only ever waits for segments
//       taken by workgroups that started before it.
//   p3: out[i] = (X[i] +) sum_{q<r} d[i r + q]
// b and d live in the global scratch (count x 2N words), followed by the
// look-back state: per vector one ticket word and one status word per segment
// (bit 32 set once the segment's sum, in the low 31 bits, is published).
// ---------------------------------------------------------------------------
template <bool SPARSE, int NS>
__global__ __launch_bounds__(kSegThreads) void syn_p1(const SegArgs a) {
    __shared__ SegLds<NS> lds;
    uint32_t c, vy, sg;
    seg_place(a, blockIdx.x, blockIdx.y, gridDim.x, &vy, &sg);
    if (vy >= a.vend[a.S - 1]) return;
    const SegSet& S = seg_set(a, vy, &c);
    if (sg >= seg_count<NS>(S.k * S.r)) return;
    seg_first<SPARSE, NS>(S, c, sg, lds);
}

template <int NS>
__global__ __launch_bounds__(kSegThreads) void syn_p2(const SegArgs a) {
    __shared__ SegLds<NS> lds;
    seg_second_scatter<NS>(a, blockIdx.x, blockIdx.y, gridDim.x, lds);
}

__global__ __launch_bounds__(256) void syn_p3(const SegArgs a) {
    uint32_t c, vy, chunk;
    seg_place(a, blockIdx.x, blockIdx.y, gridDim.x, &vy, &chunk);
    if (vy >= a.vend[a.S - 1]) return;
    const SegSet& S = seg_set(a, vy, &c);
    const uint32_t N = S.k * S.r;
    const uint32_t i = chunk * 256 + threadIdx.x;
    if (i >= S.k) return;
    const uint32_t* dbuf = S.work + (size_t)c * 2 * N + N;
    uint32_t s = 0;
    for (uint32_t q = 0; q < S.r; ++q) s = fadd(s, dbuf[(size_t)i * S.r + q]);  // R: fold blocks of r
    if (S.X) s = fadd(S.X[(size_t)c * S.k + i], s);
    S.out[(size_t)c * S.k + i] = s;
}

template <bool SPARSE>
hipError_t launch_p1(const SegArgs& a, const SegShape& h, hipStream_t s) {
    const dim3 grid(h.gx, h.rows);
    if (h.stripes == 4)
        hipLaunchKernelGGL((syn_p1<SPARSE, 4>), grid, dim3(kSegThreads), 0, s, a);
    else
        hipLaunchKernelGGL((syn_p1<SPARSE, 1>), grid, dim3(kSegThreads), 0, s, a);
    return hipGetLastError();
}

// The three launches over sets of one input kind (sparse or dense).
template <bool SPARSE>
hipError_t launch_seg_sets(SegArgs a, hipStream_t s) {
    const SegShape h = seg_shape(a);
    if (h.rows == 0) return hipSuccess;
    if (h.rows > kMaxVectors) return hipErrorInvalidValue;
    hipError_t e = launch_p1<SPARSE>(a, h, s);
    if (e != hipSuccess) return e;
    const dim3 grid(h.gx, h.rows);
    if (h.stripes == 4)
        hipLaunchKernelGGL((syn_p2<4>), grid, dim3(kSegThreads), 0, s, a);
    else
        hipLaunchKernelGGL((syn_p2<1>), grid, dim3(kSegThreads), 0, s, a);
    e = hipGetLastError();
    return e == hipSuccess ? launch_seg_last(a, h, s) : e;
}

template <bool SPARSE>
hipError_t launch_syn(const mvk_code& c, const uint32_t* v, const uint32_t* idx, const uint32_t* val, uint32_t t,
                      uint32_t count, const uint32_t* X, uint32_t* scratch, uint32_t* out, hipStream_t s) {
    if (count == 0) return hipSuccess;
    const size_t N = (size_t)c.k * c.r;
    if (N <= (size_t)kSynThreads * kSynMaxU) {
        // short blocks: one workgroup per vector, everything in LDS
        const dim3 grid(count), block(kSynThreads);
        const size_t U = (N + kSynThreads - 1) / kSynThreads;
#define MVK_SYN(EV)                                                                                        \
    hipLaunchKernelGGL((syn_wg<SPARSE, EV>), grid, block, 0, s, c.k, c.r, c.pi1, c.pi2, c.v1, c.v2, v, idx, val, \
                       t, X, out)
        if (U <= 4) MVK_SYN(4);
        else if (U <= 8) MVK_SYN(8);
        else if (U <= 12) MVK_SYN(12);
        else MVK_SYN(16);
#undef MVK_SYN
        return hipGetLastError();
    }
    SegArgs a{};
    a.S = 1;
    a.vend[0] = count;
    a.set[0] = SegSet{c.pi1, c.pi2, c.v1, c.v2, v, idx, val, X, out, scratch, c.k, c.r, t, count};
    return launch_seg_sets<SPARSE>(a, s);
}

// W (m x n) -> WT (n x m) in tiles of T x T: a thread takes 4 x 4 blocks (one
// word from each of four rows, transposed in registers), so both sides move
// words, T consecutive bytes per row of a tile; what is left at the edges goes
// byte by byte.  T is 128, or 64 where tiles of 128 do not fill the chip.  (11008
// x 4096: 16 us, against 65 with byte loads and stores.)
template <uint32_t T>
__global__ __launch_bounds__(256) void transpose_i8(const int8_t* __restrict__ W, uint32_t m, uint32_t n,
                                                    int8_t* __restrict__ WT) {
    __shared__ uint32_t tile[T][T / 4 + 1];  // [column][group of four rows]
    const uint32_t r0 = blockIdx.y * T, c0 = blockIdx.x * T;
    const bool whole = r0 + T <= m && c0 + T <= n;  // (uniform)
#pragma unroll
    for (uint32_t b = 0; b < T * T / 4096; ++b) {
        const uint32_t cg = threadIdx.x % (T / 4), rg = threadIdx.x / (T / 4) + 1024 / T * b;  // groups of four columns, rows
        uint32_t w[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t row = r0 + 4 * rg + i, col = c0 + 4 * cg;
            if (whole || (row < m && col + 4 <= n)) {
                w[i] = *reinterpret_cast<const u32_b*>(W + (size_t)row * n + col);
            } else {
                w[i] = 0;
                for (uint32_t e = 0; e < 4; ++e)
                    if (row < m && col + e < n) w[i] |= (uint32_t)(uint8_t)W[(size_t)row * n + col + e] << (8 * e);
            }
        }
        // v_perm_b32(S0, S1, sel): selector bytes 0..3 pick bytes of S1, 4..7 of S0
        const uint32_t a0 = __builtin_amdgcn_perm(w[1], w[0], 0x05010400u);  // w0.0 w1.0 w0.1 w1.1
        const uint32_t a1 = __builtin_amdgcn_perm(w[1], w[0], 0x07030602u);  // w0.2 w1.2 w0.3 w1.3
        const uint32_t b0 = __builtin_amdgcn_perm(w[3], w[2], 0x05010400u);
        const uint32_t b1 = __builtin_amdgcn_perm(w[3], w[2], 0x07030602u);
        tile[4 * cg + 0][rg] = __builtin_amdgcn_perm(b0, a0, 0x05040100u);
        tile[4 * cg + 1][rg] = __builtin_amdgcn_perm(b0, a0, 0x07060302u);
        tile[4 * cg + 2][rg] = __builtin_amdgcn_perm(b1, a1, 0x05040100u);
        tile[4 * cg + 3][rg] = __builtin_amdgcn_perm(b1, a1, 0x07060302u);
    }
    __syncthreads();
#pragma unroll
    for (uint32_t b = 0; b < T * T / 1024; ++b) {
        const uint32_t rg = threadIdx.x % (T / 4), c = threadIdx.x / (T / 4) + 1024 / T * b;
        const uint32_t w = tile[c][rg], col = c0 + c, row = r0 + 4 * rg;
        if (whole || (col < n && row + 4 <= m)) {
            *reinterpret_cast<u32_b*>(WT + (size_t)col * m + row) = w;
        } else if (col < n) {
            for (uint32_t e = 0; e < 4; ++e)
                if (row + e < m) WT[(size_t)col * m + row + e] = (int8_t)(w >> (8 * e));
        }
    }
}

__global__ void fill_u32(uint32_t* p, size_t count, uint32_t value) {
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < count; i += (size_t)gridDim.x * blockDim.x)
        p[i] = value;
}

}  // namespace

size_t encT_seg_words(size_t N, size_t nvec) {
    const size_t L = enc_seg_len(N, nvec);
    return 2 * ((N + L - 1) / L) * nvec;
}

// Plan of the segmented encoding of an int8 matrix: 32 segments (62 queries, one
// launch of the server product; 64 segments measured 10% longer at 11008 x
// 4096).  It pays where t3 no longer fits the memory-side cache: 2048 x 2048, r
// = 3 (t3 of 50 MB) takes 174 us against 152 on the three-pass form, 4096 x
// 4096 (201 MB) 341 to 380 against 416 to 431; with M's rows not whole aligned
// granules the product takes four launches (4095 x 4097: 561 us against 517),
// eight for rows above 16384 and sixteen above 32768.  A launch costs about 0.5
// us per million entries of M, and the passes saved 2.8 us per million positions,
// r times as many: up to 4 r launches (2051 x 65537, r = 1, sixteen: 3496 us against
// 1707; 2051 x 33001, r = 3, sixteen: 2378 against 2129; 4099 x 30001, r = 1,
// eight: 1634 against 1375; 2051 x 20001, r = 3, eight: 1245 against 1542).
// Fewer vectors than 2048 make too few workgroups (11008 x 256: 306 us against
// 178 with 128 segments).
namespace {
constexpr uint32_t kEncSegs = 32;
constexpr size_t kEncSegsAbove = (size_t)192 << 20, kEncSegsAboveAny = (size_t)400 << 20;  // bytes of t3
constexpr uint32_t kEncReadings = 4;  // readings of M per r
struct EncPlan {
    uint32_t nseg, L, nq, ntile, npad;  // npad: positions the passes read (whole segments, two more steps)
    size_t o_pos, o_row1, o_row2, o_c1, o_c1off, o_c2, o_idx, o_val, o_qry, o_off, o_syn, o_srv, o_t3, bytes;
    ServerEvalPlan srv;
};
bool enc_i8_plan(uint32_t k, uint32_t r, uint32_t nvec, bool rows_aligned, EncPlan* out) {
    const size_t N = (size_t)k * r, unit = 2 * kSegStep;  // (an even number of steps per segment)
    if (k > MVK_MAX_N || nvec < 2048 || N < kEncSegs * unit) return false;
    if (4 * N * nvec < (rows_aligned ? kEncSegsAbove : kEncSegsAboveAny)) return false;
    EncPlan p{};
    p.ntile = ceil_div(nvec, kSegVec);
    p.L = (uint32_t)((N + kEncSegs * unit - 1) / (kEncSegs * unit) * unit);
    p.nseg = (uint32_t)((N + p.L - 1) / p.L);
    p.nq = p.nseg - 1;
    if (!rows_aligned && server_any_launches(nvec, k, 2 * p.nq) > kEncReadings * r) return false;
    p.srv = server_eval_plan(nvec, k, 2 * p.nq, MVK_PATH_AUTO, false, rows_aligned);
    size_t b = 0;
    auto take = [&](size_t bytes) {
        const size_t at = b;
        b += (bytes + 255) & ~(size_t)255;
        return at;
    };
    p.o_pos = take(4 * N);
    p.npad = p.nseg * p.L + 2 * kSegStep;
    p.o_row1 = take(4 * (size_t)p.npad);
    p.o_row2 = take(4 * (size_t)p.npad);
    p.o_c1 = take(4 * (size_t)p.npad);
    p.o_c1off = take(4 * (size_t)p.npad);
    p.o_c2 = take(4 * (size_t)p.npad);
    p.o_idx = take(4 * (size_t)p.nq);
    p.o_val = take(4 * (size_t)p.nq);
    p.o_qry = take(4 * (size_t)2 * p.nq * k);
    p.o_off = take(4 * (size_t)2 * p.nq * nvec);
    p.o_syn = take(syn_scratch_bytes(p.nq, N));
    p.o_srv = take(p.srv.ws_bytes);
    p.o_t3 = take(4 * N * kSegVec * p.ntile);
    p.bytes = b;
    *out = p;
    return true;
}

}  // namespace

bool enc_i8_scratch(uint32_t k, uint32_t r, uint32_t nvec, bool rows_aligned, size_t* bytes, size_t* ctrl_words) {
    EncPlan p;
    if (!enc_i8_plan(k, r, nvec, rows_aligned, &p)) return false;
    *bytes = p.bytes;
    *ctrl_words = p.srv.ctrl_words;
    return true;
}

hipError_t launch_enc_i8(const mvk_code& c, const int8_t* M, const int8_t* in, uint32_t nvec, void* scratch,
                         size_t scratch_bytes, uint32_t* counters, uint32_t* out, hipStream_t s) {
    EncPlan p;
    if (!enc_i8_plan(c.k, c.r, nvec, c.k % 16 == 0 && (uintptr_t)M % 16 == 0, &p) || p.bytes > scratch_bytes)
        return hipErrorInvalidValue;
    const uint32_t N = c.k * c.r;
    char* ws = reinterpret_cast<char*>(scratch);
    auto at = [&](size_t o) { return reinterpret_cast<uint32_t*>(ws + o); };
    hipLaunchKernelGGL(enc_prep, dim3(ceil_div(p.npad, 256)), dim3(256), 0, s, N, p.npad, c.r, p.L, p.nq, c.pi1,
                       c.pi2, c.v1, c.v2, at(p.o_pos), at(p.o_row1), at(p.o_row2), at(p.o_c1), at(p.o_c1off),
                       at(p.o_c2), at(p.o_idx), at(p.o_val));
    hipLaunchKernelGGL(enc_dq, dim3(ceil_div(c.k, 256), ceil_div(p.nq, kDqPer)), dim3(256), 0, s, c.k, c.r, N, p.L,
                       p.nq, at(p.o_pos), c.v1, at(p.o_qry));
    hipError_t e = launch_syn_sparse(c, at(p.o_idx), at(p.o_val), 1, p.nq, nullptr, at(p.o_syn),
                                     at(p.o_qry) + (size_t)p.nq * c.k, s);
    if (e != hipSuccess) return e;
    e = launch_server_eval(M, nvec, c.k, at(p.o_qry), 2 * p.nq, at(p.o_off), MVK_PATH_AUTO, false, ws + p.o_srv,
                           counters, s);
    if (e != hipSuccess) return e;
    const dim3 grid(p.ntile * p.nseg), block(kSegWaves * 64);
    hipLaunchKernelGGL(enc_seg<true>, grid, block, 0, s, N, p.L, p.nseg, p.ntile, at(p.o_row1), at(p.o_c1),
                       at(p.o_c1off), in, nvec, at(p.o_off), at(p.o_t3), nullptr);
    hipLaunchKernelGGL(enc_seg<false>, grid, block, 0, s, N, p.L, p.nseg, p.ntile, at(p.o_row2), at(p.o_c2), nullptr,
                       nullptr, nvec, at(p.o_off) + (size_t)p.nq * nvec, at(p.o_t3), out);
    return hipGetLastError();
}

hipError_t launch_encT_u32(const mvk_code& c, const uint32_t* in, size_t ld_in, size_t vs_in, uint32_t nvec,
                           uint32_t* t3, uint32_t* seg, uint32_t* out, size_t ld_out, size_t vs_out, hipStream_t s) {
    return launch_encT<uint32_t>(c, in, ld_in, vs_in, nvec, t3, seg, out, ld_out, vs_out, s);
}

hipError_t launch_encT_i8(const mvk_code& c, const int8_t* in, size_t ld_in, size_t vs_in, uint32_t nvec,
                          uint32_t* t3, uint32_t* seg, uint32_t* out, size_t ld_out, size_t vs_out, hipStream_t s) {
    return launch_encT<int8_t>(c, in, ld_in, vs_in, nvec, t3, seg, out, ld_out, vs_out, s);
}

size_t syn_sets_scratch_bytes(const SynSet* sets, uint32_t S) {
    size_t b = 0;
    for (uint32_t i = 0; i < S; ++i) b += (syn_seg_bytes(sets[i].count, (size_t)sets[i].c->k * sets[i].c->r) + 255) & ~(size_t)255;
    return b;
}

namespace synseg {
SegShape seg_shape(SegArgs& a) {
    SegShape h{0, 0, 1, 0};
    uint32_t maxN = 0;
    uint64_t segs = 0;  // workgroups with one stripe each
    for (uint32_t i = 0; i < a.S; ++i) {
        const uint32_t N = a.set[i].k * a.set[i].r;
        segs += (uint64_t)seg_count<1>(N) * a.set[i].count;
        maxN = N > maxN ? N : maxN;
        h.maxk = a.set[i].k > h.maxk ? a.set[i].k : h.maxk;
    }
    const uint32_t nv = a.S ? a.vend[a.S - 1] : 0u;
    // placed by XCD: whole eights, and a rest of six or more (its empty places
    // return at once; fewer vectors would leave XCDs idle); where lengths differ so
    // much that one XCD would get over 3/2 of its share, the whole eights of fewer
    // sets (a preparation with 15 vectors of one segment and six of 136: 58.3 us
    // with the first 16 placed, 51.0 with the first eight; with ten of 56 segments
    // and four of two: 28.1 and 25.6)
    const auto balanced = [&](uint32_t by) {
        uint64_t load[kXcds] = {}, sum = 0, most = 0;
        for (uint32_t i = 0, v = 0; i < a.S && v < by; v += a.set[i++].count) {
            const uint32_t count = a.set[i].count < by - v ? a.set[i].count : by - v;
            const uint64_t seg = seg_count<1>(a.set[i].k * a.set[i].r);
            for (uint32_t x = 0; x < kXcds; ++x)  // (the vectors from v on go to the XCDs in turn)
                load[(v + x) % kXcds] += seg * (count / kXcds + (x < count % kXcds ? 1u : 0u));
        }
        for (uint64_t l : load) sum += l, most = l > most ? l : most;
        return 2 * kXcds * most <= 3 * sum;
    };
    a.by_xcd = (nv + 2) / kXcds * kXcds;
    if (a.by_xcd > kMaxVectors) a.by_xcd = nv / kXcds * kXcds;
    for (uint32_t i = a.S; i-- > 0 && !balanced(a.by_xcd);) a.by_xcd = (i ? a.vend[i - 1] : 0u) / kXcds * kXcds;
    h.rows = nv > a.by_xcd ? nv : a.by_xcd;
    // four stripes per workgroup where one each would be more workgroups than
    // the chip holds at once (eight per compute unit)
    h.stripes = segs > 2048 ? 4u : 1u;
    h.gx = h.stripes == 4 ? seg_count<4>(maxN) : seg_count<1>(maxN);
    return h;
}

hipError_t launch_seg_first(const SegArgs& a, const SegShape& h, hipStream_t s) {
    return launch_p1<true>(a, h, s);
}

hipError_t launch_seg_last(const SegArgs& a, const SegShape& h, hipStream_t s) {
    hipLaunchKernelGGL(syn_p3, dim3(ceil_div(h.maxk, 256u), h.rows), dim3(256), 0, s, a);
    return hipGetLastError();
}
}  // namespace synseg

bool synseg::seg_args(const SynSet* sets, uint32_t S, uint32_t* scratch, size_t scratch_bytes, SegArgs* out) {
    if (S > kMaxSynSets) return false;
    // the sets' work regions lie one after another: the scratch must hold them all
    if (syn_sets_scratch_bytes(sets, S) > scratch_bytes) return false;
    SegArgs a{};
    uint32_t nv = 0;
    char* w = reinterpret_cast<char*>(scratch);
    for (uint32_t i = 0; i < S; ++i) {
        const SynSet& d = sets[i];
        const size_t N = (size_t)d.c->k * d.c->r;
        if (d.count == 0) continue;
        a.set[a.S] = SegSet{d.c->pi1, d.c->pi2, d.c->v1, d.c->v2, nullptr, d.idx, d.val, nullptr, d.out,
                            reinterpret_cast<uint32_t*>(w), d.c->k, d.c->r, d.t, d.count};
        nv += d.count;
        a.vend[a.S++] = nv;
        w += (syn_seg_bytes(d.count, N) + 255) & ~(size_t)255;
    }
    *out = a;
    return nv <= kMaxVectors;
}

hipError_t launch_syn_sets(const SynSet* sets, uint32_t S, uint32_t* scratch, size_t scratch_bytes, hipStream_t s) {
    SegArgs a;
    return seg_args(sets, S, scratch, scratch_bytes, &a) ? launch_seg_sets<true>(a, s) : hipErrorInvalidValue;
}

hipError_t launch_syn_dense(const mvk_code& c, const uint32_t* v, uint32_t count, uint32_t* scratch, uint32_t* out,
                            hipStream_t s) {
    return launch_syn<false>(c, v, nullptr, nullptr, 0u, count, nullptr, scratch, out, s);
}

hipError_t launch_syn_sparse(const mvk_code& c, const uint32_t* idx, const uint32_t* val, uint32_t t,
                             uint32_t count, const uint32_t* X, uint32_t* scratch, uint32_t* out, hipStream_t s) {
    return launch_syn<true>(c, nullptr, idx, val, t, count, X, scratch, out, s);
}

hipError_t launch_transpose_i8(const int8_t* W, uint32_t m, uint32_t n, int8_t* WT, hipStream_t s) {
    if (m == 0 || n == 0) return hipSuccess;
    if ((uint64_t)ceil_div(n, 128) * ceil_div(m, 128) >= 256)
        hipLaunchKernelGGL(transpose_i8<128>, dim3(ceil_div(n, 128), ceil_div(m, 128)), dim3(256), 0, s, W, m, n, WT);
    else
        hipLaunchKernelGGL(transpose_i8<64>, dim3(ceil_div(n, 64), ceil_div(m, 64)), dim3(256), 0, s, W, m, n, WT);
    return hipGetLastError();
}

hipError_t launch_fill_u32(uint32_t* p, size_t count, uint32_t value, hipStream_t s) {
    if (count == 0) return hipSuccess;
    size_t blocks = (count + 255) / 256;
    if (blocks > 4096) blocks = 4096;
    hipLaunchKernelGGL(fill_u32, dim3((uint32_t)blocks), dim3(256), 0, s, p, count, value);
    return hipGetLastError();
}

}  // namespace mvk
