// Clusters, octree traversal and compressed list encoding (Sec. II-A, II-B,
// II-C).
//
// One wavefront builds the list of one super-cluster (64 particles = 8
// i-clusters of 8).
//
// Traversal: depth-first from the root with an LDS stack; at an internal node
// 64 lanes test up to 8 children against 8 boxes of the super-cluster and
// push the survivors in reverse key order, so leaves come out in key order
// and the list is sorted without a sort (Sec. II-A). The leaves' candidate
// j-clusters collect 64 at a time, one per lane, and are tested against the
// boxes of the super-cluster's particles 8 at a time; the survivors join an
// LDS queue, whose batches of 64 j-particles arrive with one load per field
// while the previous batch is tested. Box tests are conservative under FP32
// rounding (rounding is monotone), so they never drop a pair the exact test
// keeps; the masks are exact.
//
// Pair tests. The matrix cores evaluate all 64 x 64 squared distances of a
// batch from split half-precision coordinates, with a bound E on their error;
// a tile with a distance more than E below its squared radius is set, one with
// none within E of it is clear, and the few left open (and the tiles of a
// cluster with itself) are decided by the exact FP32 formula, so the list does
// not depend on the filter. The former vector tests of the tiles whose boxes
// met cost 8 vector instructions per 64 pairs and about 6,100 of a
// super-cluster's 10,900; now a 64 x 64 block costs some 235. Both were bound
// by vector issue and latency: 0.63 -> 0.53 ms on 2,097,152 uniform particles
// (half list, cluster size 8), 1.74 -> 1.52 ms on the 4,000,037-particle 1/r
// sphere (full list).
//
// The list is staged in 64-entry chunks with its encoded size computed on the
// fly (a super-cluster's first chunk is its own, later ones come from 64
// striped counters), a prefix sum places the super-clusters in order, and a
// second kernel writes masks and nibble segments.
#include <cstring>
#include <type_traits>
#include <utility>

#include "internal.h"

namespace sfcnl {
namespace {

// Lambdas of the traversal kernel are always inlined: a lambda left as a call
// takes the kernel's argument block by reference, which then lives in
// scratch memory, and every pointer from it is loaded through scratch.
#define SFC_INLINE __attribute__((always_inline))

// One wavefront (one super-cluster) per block for the traversal and the
// encoder: a block's resources are released only when its slowest wave ends,
// and super-clusters differ in work; measured 10 % faster than four.
constexpr int kWavesPerBlock = 1;
constexpr uint32_t kStrictFrom = 128;  // tested clusters after which few listed ones matter (k_traverse's strict tests)
constexpr int kStackCap = 148;  // 1 + 7 * 21 records at most
constexpr int kSegCap = 80;     // words of one 64-value segment: 2 + (64 + 512 + 7) / 8
constexpr int kQueueCap = 128;  // queued candidates (a ring): fewer than 16 left over, one box step adds at most 64
constexpr uint32_t kUnstaged = 0xFFFFFFFFu;  // sc_nj of a list that found no staging room

__device__ __forceinline__ unsigned xcd_remap(unsigned b, unsigned g) {
    // blocks are dealt round-robin to the 8 XCDs; give each XCD a contiguous
    // range of super-clusters so neighbouring ones share its L2
    const unsigned per = g / 8, rem = g % 8, x = b % 8, i = b / 8;
    return x < rem ? x * (per + 1) + i : rem * (per + 1) + (x - rem) * per + i;
}

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Boxes carry .w of lo = largest radius inside. True if some particle pair
// across the two boxes could satisfy d2 < max(h_i, h_j)^2.
template <bool kPbc>
__device__ __forceinline__ bool boxes_near_p(float4 alo, float4 ahi, float4 blo, float4 bhi, const Period &per) {
    float gx = axis_gap<kPbc>(blo.x - ahi.x, alo.x - bhi.x, per.L[0]);
    float gy = axis_gap<kPbc>(blo.y - ahi.y, alo.y - bhi.y, per.L[1]);
    float gz = axis_gap<kPbc>(blo.z - ahi.z, alo.z - bhi.z, per.L[2]);
    float gxx = gx * gx;
    float d2 = __builtin_fmaf(gz, gz, __builtin_fmaf(gy, gy, gxx));
    float ra = alo.w * alo.w, rb = blo.w * blo.w;
    return d2 < fmaxf(ra, rb);
}
// per is wave-uniform: super-clusters that need no wrapping take the open test
template <bool kPbc = false>
__device__ __forceinline__ bool boxes_near(float4 alo, float4 ahi, float4 blo, float4 bhi, const Period &per = Period{}) {
    if (kPbc && per.on()) return boxes_near_p<true>(alo, ahi, blo, bhi, per);
    return boxes_near_p<false>(alo, ahi, blo, bhi, per);
}

// Position for absent particles: any distance to it overflows to +inf.
constexpr float kFar = 3.0e38f;

__device__ __forceinline__ uint32_t nibbles_of(uint32_t v) { return (32u - (uint32_t)__clz((int)v) + 3u) >> 2; }

// ---------------------------------------------------------------------------
// Clusters: bounding boxes and radius maxima, input checks.
// ---------------------------------------------------------------------------
template <int CS, bool kVec>
__global__ __launch_bounds__(256) void k_cluster_bbox(int64_t n, const float *__restrict__ x,
                                                      const float *__restrict__ y, const float *__restrict__ z,
                                                      const float *__restrict__ h, float4 *__restrict__ bbox,
                                                      uint32_t *status, SegTable seg) {
    int64_t c = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (c >= (n + CS - 1) / CS) return;
    // batched systems: particles from pend on are padding (NaN, ignored by
    // fminf / fmaxf and never checked)
    int64_t pend = n;
    if (seg.on()) {
        const int sy = seg.sc_sys[c * CS / kScSize];
        pend = (int64_t)seg.pbase[sy] + seg.count[sy];
    }
    // a whole cluster of 16-byte-aligned fields comes as CS / 4 float4 loads
    // per field (one request per 16 bytes instead of one per 4); the last,
    // partial cluster or unaligned fields read each particle from a clamped
    // index; all loads are in flight together
    float px[CS], py[CS], pz[CS], ph[CS];
    if (kVec && c * CS + CS <= n) {
        const float4 *x4 = reinterpret_cast<const float4 *>(x) + c * (CS / 4);
        const float4 *y4 = reinterpret_cast<const float4 *>(y) + c * (CS / 4);
        const float4 *z4 = reinterpret_cast<const float4 *>(z) + c * (CS / 4);
        const float4 *h4 = reinterpret_cast<const float4 *>(h) + c * (CS / 4);
#pragma unroll
        for (int q = 0; q < CS / 4; q++) {
            const float4 vx = x4[q], vy = y4[q], vz = z4[q], vh = h4[q];
            px[4 * q] = vx.x, px[4 * q + 1] = vx.y, px[4 * q + 2] = vx.z, px[4 * q + 3] = vx.w;
            py[4 * q] = vy.x, py[4 * q + 1] = vy.y, py[4 * q + 2] = vy.z, py[4 * q + 3] = vy.w;
            pz[4 * q] = vz.x, pz[4 * q + 1] = vz.y, pz[4 * q + 2] = vz.z, pz[4 * q + 3] = vz.w;
            ph[4 * q] = vh.x, ph[4 * q + 1] = vh.y, ph[4 * q + 2] = vh.z, ph[4 * q + 3] = vh.w;
        }
    } else {
#pragma unroll
        for (int k = 0; k < CS; k++) {
            const int64_t p = c * CS + k;
            const int64_t q = p < n ? p : n - 1;
            px[k] = x[q];
            py[k] = y[q];
            pz[k] = z[q];
            ph[k] = h[q];
        }
    }
    float4 lo = make_float4(INFINITY, INFINITY, INFINITY, 0.0f);
    float4 hi = make_float4(-INFINITY, -INFINITY, -INFINITY, 0.0f);
    uint32_t bad = 0;
#pragma unroll
    for (int k = 0; k < CS; k++) {
        const int64_t p = c * CS + k;
        if (p < n) {
            const bool pad = p >= pend;
            if (!pad && !(isfinite(px[k]) && isfinite(py[k]) && isfinite(pz[k]))) bad |= 1u;
            if (!pad && !(isfinite(ph[k]) && ph[k] > 0.0f)) bad |= 2u;
            lo.x = fminf(lo.x, px[k]);
            lo.y = fminf(lo.y, py[k]);
            lo.z = fminf(lo.z, pz[k]);
            lo.w = fmaxf(lo.w, ph[k]);
            hi.x = fmaxf(hi.x, px[k]);
            hi.y = fmaxf(hi.y, py[k]);
            hi.z = fmaxf(hi.z, pz[k]);
        }
    }
    bbox[2 * c] = lo;
    bbox[2 * c + 1] = hi;
    if (bad) atomicOr(&status[kStInputErr], bad);
}

// ---------------------------------------------------------------------------
// Traversal
// ---------------------------------------------------------------------------
struct TravArgs {
    int64_t n;
    uint32_t nsc, nclu;
    int compress;
    const float *x, *y, *z, *h;
    const float4 *bbox;
    const float4 *cs_box;  // octree child slots (slot 0 = root)
    const uint4 *cs_rec;
    const float4 *lvl1;    // kDirect: boxes of 8 clusters (nullable; cs_box is then the root box alone)
    uint32_t nslots;       // capacity of the slot arrays
    SegTable seg;          // batched systems (empty for one system)
    Period per;            // periodic axes (used by the kPbc kernels)
    const uint32_t *active;  // nullable: super-clusters with active[s] == 0 get an empty list
    // nullable: a counting list for the flagged particles only (own radius):
    // pairs d2 < h_i^2 for i with p_active[i] != 0; node, cluster and j radii
    // are ignored, so the octree's boxes need no refit when only radii change
    const uint8_t *p_active;
    const uint32_t *gate;  // nullable: every list empty when *gate <= gate_max
    uint32_t gate_max;
    // staging: 64-entry chunks; chunk s is super-cluster s's first, longer
    // lists continue in chunks nsc + id taken from the stripe counters
    // (take_chunk); chunk_next links a list's chunks in order
    uint32_t *list_j;
    uint16_t *list_m;
    uint32_t *chunk_next;
    uint32_t nshared;      // shared chunks (ids 0 .. nshared - 1)
    uint32_t *chunk_ctr;   // the stripe counters that hand them out; word 1 of each line holds the stripe's longest list (zeroed before the build)
    uint32_t *sc_nj, *sc_words;
    uint32_t *status;
};

// Node tests pair child l / 8 with the box of super-cluster particles
// [8g, 8g + 8), g = l % 8 (for CS = 16 the box of the i-cluster holding them).
template <int CS>
struct Shape {
    static constexpr int kNsub = kScSize / CS;  // i-clusters per super-cluster
    static constexpr int kMaskBytes = kNsub > 8 ? 2 : 1;
    static constexpr uint32_t kFull = (1u << kNsub) - 1u;
};

__device__ __forceinline__ void box_union(float4 &lo, float4 &hi, float4 blo, float4 bhi) {
    lo.x = fminf(lo.x, blo.x);
    lo.y = fminf(lo.y, blo.y);
    lo.z = fminf(lo.z, blo.z);
    lo.w = fmaxf(lo.w, blo.w);
    hi.x = fmaxf(hi.x, bhi.x);
    hi.y = fmaxf(hi.y, bhi.y);
    hi.z = fmaxf(hi.z, bhi.z);
}

constexpr uint32_t kNoChunk = 0xFFFFFFFFu;

// A shared staging chunk for super-cluster s: from stripe s % kChunkStripes,
// else from the next stripes while one is used up; kNoChunk once all are
// (every one of the nshared ids is taken). Called by one lane.
__device__ uint32_t take_chunk(uint32_t *ctr, uint32_t nshared, uint32_t s) {
    for (uint32_t t = 0; t < (uint32_t)kChunkStripes; t++) {
        const uint32_t k = (s + t) % kChunkStripes;
        if (k >= nshared) continue;  // an empty stripe
        const uint32_t cap = (nshared - k + kChunkStripes - 1) / kChunkStripes;
        const uint32_t i = atomicAdd(&ctr[k * kStripeWords], 1u);
        if (i < cap) return k + kChunkStripes * i;
    }
    return kNoChunk;
}

// Bit k of the result: byte k of b is nonzero.
__device__ __forceinline__ uint32_t nonzero_bytes(uint64_t b) {
    b |= b >> 4;
    b |= b >> 2;
    b |= b >> 1;
    b &= 0x0101010101010101ull;
    return (uint32_t)((b * 0x0102040810204080ull) >> 56);
}

// f(std::integral_constant<int, i>{}) for i = 0 .. N - 1
template <int N, typename F, int... I>
__device__ __forceinline__ void static_for_impl(F &&f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F &&f) {
    static_for_impl<N>(f, std::make_integer_sequence<int, N>{});
}

// v of lane P of the quad (DPP quad_perm broadcast). With all rows and banks
// enabled and bound_ctrl set, the compiler folds the move into the consuming
// instruction's first operand, so the broadcast costs no instruction.
template <int P>
__device__ __forceinline__ float quad_bcast(float v) {
    return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), P * 0x55, 0xF, 0xF, true));
}

// v of lane P of the group of CS lanes (a quad or a row; the same fold)
template <int CS, int P>
__device__ __forceinline__ float group_bcast(float v) {
    if constexpr (CS == 4)
        return quad_bcast<P>(v);
    else
        return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x150 + P, 0xF, 0xF, true));  // row_newbcast
}

// max of two squared radii (both >= +0): the integer order of their bit
// patterns is their order, and the integer max needs no canonicalisation
__device__ __forceinline__ float max_sq(float u, float v) {
    return __int_as_float(max(__float_as_int(u), __float_as_int(v)));
}

// ---------------------------------------------------------------------------
// The matrix-core filter of the exact tests. For 32 i-particles (rows) and 32
// j-particles (columns), one v_mfma_f32_32x32x16_f16 gives every pair's
// |x_i|^2 + |x_j|^2 - 2 x_i . x_j minus one of the two squared radii, from
// coordinates taken relative to the super-cluster, scaled by a power of two
// and split into two halves each (x = h + l; the l l products are dropped),
// and squares split into three. Slots k of the 16 products A_k B_k:
//   3t .. 3t + 2  (axis t)  A = -2h, -2h, -2l   B = h, l, h
//   9 .. 11                 A = the i-square    B = 1
//   12 .. 14                A = 1               B = the j-square
//   15                      0
// A lane's first four registers hold slots 0-7, the others 8-15.
// ---------------------------------------------------------------------------
typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));
typedef float float16_t __attribute__((ext_vector_type(16)));
typedef uint32_t uint4_t __attribute__((ext_vector_type(4)));

constexpr float kFar16 = 60000.0f;    // values above cannot be split into halves
constexpr uint32_t kInf16 = 0x7C00u;  // an absent particle's square: no pair of it is near
constexpr uint32_t kOnes16 = 0x3C003C00u;

__device__ __forceinline__ uint32_t pack16(float a, float b) {
    const half2_t v = {(_Float16)a, (_Float16)b};
    return __builtin_bit_cast(uint32_t, v);
}
// v rounded to a half. The empty asm keeps the conversion one instruction of its
// own: joined with the arithmetic before it (v_fma_mixlo) it would round v's
// exact value, which near a tie is another half than v's, and a remainder
// v - round16(v) needs the value that is packed.
__device__ __forceinline__ float round16(float v) {
    _Float16 t = (_Float16)v;
    asm("" : "+v"(t));
    return (float)t;
}

// lanes 32-63 of a change places with lanes 0-31 of b
__device__ __forceinline__ void swap_halves(uint32_t &a, uint32_t &b) {
    const auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
    a = r[0];
    b = r[1];
}

// One particle's operand in its own lane (8 registers), with a second form of
// the two registers that hold the square: `row` selects A (rows: square, and
// square minus the squared radius; an absent particle's are infinite) or B.
// After the swaps lane l of plain[0] holds slots 8 (l / 32) .. of particle
// l % 32 and plain[1] those of particle 32 + l % 32; other[] are the registers
// kSquare and kSquare + 1 of the second form.
constexpr int kSquareA = 0, kSquareB = 2;
struct Operands {
    uint4_t plain[2];
    uint32_t other[2][2];
};
template <bool kRow>
__device__ __forceinline__ Operands operands(float x, float y, float z, float sq, float sq_other, bool present) {
    const float hx = round16(x), hy = round16(y), hz = round16(z);
    const float lx = x - hx, ly = y - hy, lz = z - hz;
    const float s0 = round16(sq), s1 = round16(sq - s0), s2 = sq - s0 - s1;
    const float t0 = round16(sq_other), t1 = round16(sq_other - t0), t2 = sq_other - t0 - t1;
    uint32_t r[8], u0, u1;
    if (kRow) {
        r[0] = pack16(-2.0f * hx, -2.0f * hx);
        r[1] = pack16(-2.0f * lx, -2.0f * hy);
        r[2] = pack16(-2.0f * hy, -2.0f * ly);
        r[3] = pack16(-2.0f * hz, -2.0f * hz);
        r[4] = pack16(-2.0f * lz, present ? s0 : INFINITY);
        r[5] = present ? pack16(s1, s2) : 0u;
        r[6] = kOnes16;
        r[7] = kOnes16 & 0xFFFFu;
        u0 = pack16(-2.0f * lz, present ? t0 : INFINITY);
        u1 = present ? pack16(t1, t2) : 0u;
    } else {
        r[0] = pack16(hx, lx);
        r[1] = pack16(hx, hy);
        r[2] = pack16(ly, hy);
        r[3] = pack16(hz, lz);
        r[4] = pack16(hz, 1.0f);
        r[5] = kOnes16;
        r[6] = pack16(s0, s1);
        r[7] = pack16(s2, 0.0f);
        u0 = pack16(t0, t1);
        u1 = pack16(t2, 0.0f);
    }
    constexpr int kS = kRow ? kSquareA : kSquareB;
    uint32_t v0 = r[kS], v1 = r[kS + 1];
#pragma unroll
    for (int k = 0; k < 4; k++) swap_halves(r[k], r[4 + k]);
    swap_halves(v0, u0);
    swap_halves(v1, u1);
    Operands o;
    o.plain[0] = uint4_t{r[0], r[1], r[2], r[3]};
    o.plain[1] = uint4_t{r[4], r[5], r[6], r[7]};
    o.other[0][0] = v0;
    o.other[0][1] = v1;
    o.other[1][0] = u0;
    o.other[1][1] = u1;
    return o;
}

__device__ __forceinline__ float16_t pair_block(uint4_t a, uint4_t b) {
    return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(half8_t, a), __builtin_bit_cast(half8_t, b),
                                                  float16_t{}, 0, 0, 0);
}

// bit k: lane k or k + 32 of a ballot
__device__ __forceinline__ uint32_t fold_halves(uint64_t b) { return (uint32_t)b | (uint32_t)(b >> 32); }

// v of the lane whose index differs as the DPP control says (the moves fold
// into the consuming instruction)
template <int CTRL>
__device__ __forceinline__ uint32_t dpp_u(uint32_t v) {
    return (uint32_t)__builtin_amdgcn_mov_dpp((int)v, CTRL, 0xF, 0xF, true);
}

// The i-cluster masks of a 64 x 64 block's candidates. Bit 8 b + 4 f + g of
// `seen`, lane l: that lane saw a pair of one of the i-particles
// 32 f + 8 g + 4 (l / 32) + {0..3} with j-particle 32 b + l % 32. Lane q gets
// the mask of candidate q (q below 64 / CS; other lanes: unspecified).
template <int CS>
__device__ __forceinline__ uint32_t candidate_mask(uint32_t seen, int lane) {
    // over the lanes of a j-cluster (4, 8 or 16 lanes of a half)
    seen |= dpp_u<0xB1>(seen);  // quad_perm [1, 0, 3, 2]
    seen |= dpp_u<0x4E>(seen);  // quad_perm [2, 3, 0, 1]
    if constexpr (CS >= 8) seen |= dpp_u<0x141>(seen);   // row_half_mirror
    if constexpr (CS == 16) seen |= dpp_u<0x140>(seen);  // row_mirror
    if constexpr (CS == 4) {
        // candidate 8b + c: lanes 4c .. 4c + 3 of the halves; i-cluster 8f + 2g + half
        const int src = 4 * (lane & 7);
        const uint32_t lo = (uint32_t)__shfl((int)seen, src, kWave), hi = (uint32_t)__shfl((int)seen, src + 32, kWave);
        auto spread = [](uint32_t v) {  // bit k to bit 2k
            v = (v | (v << 4)) & 0x0F0Fu;
            v = (v | (v << 2)) & 0x3333u;
            return (v | (v << 1)) & 0x5555u;
        };
        const int sh = lane & 8;  // byte b
        return spread((lo >> sh) & 0xFFu) | (spread((hi >> sh) & 0xFFu) << 1);
    } else {
        uint32_t a = seen, b = seen;
        swap_halves(a, b);
        seen = a | b;  // both halves' rows
        if constexpr (CS == 8) {  // candidate 4b + c: lanes 8c .. 8c + 7; i-cluster 4f + g
            return ((uint32_t)__shfl((int)seen, 8 * (lane & 3), kWave) >> (8 * ((lane >> 2) & 1))) & 0xFFu;
        } else {  // candidate 2b + c: lanes 16c .. 16c + 15; i-cluster 2f + g / 2
            uint32_t v = ((uint32_t)__shfl((int)seen, 16 * (lane & 1), kWave) >> (8 * ((lane >> 1) & 1))) & 0xFFu;
            v = (v | (v >> 1)) & 0x55u;
            v = (v | (v >> 1)) & 0x33u;
            return (v | (v >> 2)) & 0x0Fu;
        }
    }
}

// kDirect: a small system without its octree, kDirect waves of a block sharing
// a super-cluster. Each takes its share of all groups of 8 clusters, tests the
// groups' boxes (lvl1, nullable: every group passes), the clusters' boxes and
// the pairs of what comes near, and leaves the masks in LDS, from which the
// first wave makes the list. The octree's ten dependent launches and the walk's
// chain of node reads by one wave take longer than testing every group, whose
// work grows with n^2. Builds (clusters to pool) in us, octree / this, full
// lists of some 100 neighbours:
//                         uniform      1/r sphere   Plummer      Plummer, equal radii
//   clusters of 8   1,000    86 /  50     81 /  49    106 /  47     89 /  46
//                  32,768   128 /  60    142 /  59    379 / 124    620 / 160
//                 131,072   168 / 135    157 / 134    315 / 232   1241 / 565
//                 196,608   161 / 254    168 / 254    330 / 304   1532 / 900
//   clusters of 4  65,536   171 / 131    154 / 127    398 / 277   1045 / 446
//                 131,072   181 / 539    184 / 524    359 / 639   1456 / 1599
//   clusters of 16 196,608  176 / 164    190 / 172    393 / 282   1506 / 685
//                 262,144   193 / 230    222 / 230    331 / 278   1805 / 859
// (half lists, radii of a uniform guess on the sphere and periodic boxes alike).
// The strict tests of the walk are not needed here: the outskirts of condensed
// systems, whose boxes let most clusters through, are tested by 4 to 8 waves. Group
// boxes (a launch) with 4 waves against 8 waves without, from kDirectFew on, full
// lists: uniform 24,000 56 / 52, 40,000 67 / 73, 65,536 79 / 100; sphere 24,000
// 56 / 51, 40,000 64 / 71, 65,536 83 / 98; Plummer 24,000 143 / 104, 65,536 206 / 174,
// 100,000 236 / 260.
constexpr int kDirectWavesFew = 8, kDirectWavesMany = 4;
constexpr int64_t kDirectFew = 32768;  // particles: above, 4 waves and group boxes
constexpr int64_t direct_max(int cs) { return cs == 4 ? 65536 : (cs == 8 ? 131072 : 196608); }

// Five waves per SIMD: at most 96 VGPRs, and at most 7,680 bytes of LDS (four
// waves: 0.56 against 0.53 ms on the 2M box).
template <int CS, bool kHalf, bool kPbc, int kDirect>
__global__ __launch_bounds__(kWave * (kDirect ? kDirect : kWavesPerBlock)) __attribute__((amdgpu_waves_per_eu(5, 5))) void k_traverse(TravArgs a) {
    using S = Shape<CS>;
    constexpr int kNsub = S::kNsub;
    constexpr int kBatch = kWave / CS;               // candidates per batch of 64 j-particles
    constexpr int kBoxes = kNsub < 8 ? kNsub : 8;    // i-boxes of the box tests (CS = 4: of two clusters each)
    constexpr bool kLaneTiles = CS == 8;
    constexpr int kW = kDirect ? kDirect : kWavesPerBlock;
    __shared__ uint4 s_stack[kDirect ? 1 : kW][kDirect ? 1 : kStackCap];
    __shared__ uint32_t s_queue[kW][kQueueCap];
    __shared__ float4 s_box[kW][2 * kBoxes];
    __shared__ uint2 s_ent[kDirect ? 1 : kW][kBatch];
    using Mask = typename std::conditional<CS == 4, uint16_t, uint8_t>::type;
    __shared__ uint32_t s_grp[kDirect ? kW : 1][kDirect ? kWave : 1];
    extern __shared__ uint32_t s_dyn[];  // kDirect: every cluster's mask
    Mask *const s_mask = reinterpret_cast<Mask *>(s_dyn);
    __shared__ uint4_t s_a[kW][4][kWave];  // the filter's i-operands: less[0], less[1], plain[0], plain[1]
    const int lane = sfc_lane();
    const int w = threadIdx.x / kWave;
    // wave-uniform: keep the super-cluster index (and all derived from it) scalar
    const uint32_t s = (uint32_t)__builtin_amdgcn_readfirstlane(
        (int)(kDirect ? xcd_remap(blockIdx.x, gridDim.x) : xcd_remap(blockIdx.x, gridDim.x) * kWavesPerBlock + w));
    if (s >= a.nsc) return;
    if (kDirect) {
        const uint32_t words = (a.nclu * (uint32_t)sizeof(Mask) + 3u) / 4u;
        for (uint32_t k = threadIdx.x; k < words; k += kW * kWave) s_dyn[k] = 0u;
        __syncthreads();
    } else if ((a.active && !a.active[s]) || (a.gate && *a.gate <= a.gate_max)) {  // no list for this super-cluster
        if (sfc_lane() == 0) {
            a.sc_nj[s] = 0;
            a.sc_words[s] = 0;
        }
        return;
    }
    const int64_t n = a.n;
    const bool gather = !kDirect && a.p_active != nullptr;
    const uint32_t own_c0 = s * kNsub;   // first i-cluster of this super-cluster
    const uint32_t own_p0 = s * kScSize; // and its first particle
    // i-particle `lane`; absent ones are put far away so that no test accepts them
    bool big = false;  // a radius reaches half a period
    float ix, iy, iz, ih2;
    bool ipresent;
    {
        const int64_t i = (int64_t)own_p0 + lane;
        const bool v = i < n;
        const int64_t ic = v ? i : n - 1;
        ix = a.x[ic];
        iy = a.y[ic];
        iz = a.z[ic];
        float hh = a.h[ic];
        if (kPbc) big = v && !(hh < a.per.hmin);
        ipresent = v && ix + iy + iz == ix + iy + iz;  // (a batch's padding is NaN)
        if (gather) ipresent = ipresent && a.p_active[ic];  // counting list: flagged particles only
        if (!v) ix = iy = iz = kFar;
        ih2 = v && (!gather || a.p_active[ic]) ? hh * hh : 0.0f;
    }
    if (kPbc && sfc_ballot(big) && lane == 0) atomicOr(&a.status[kStInputErr], 8u);

    constexpr bool half = kHalf;
    // node tests: the box of super-cluster particles [8g, 8g + 8), g = lane % 8
    // (for CS = 16 the box of their i-cluster)
    float4 glo = make_float4(INFINITY, INFINITY, INFINITY, 0.0f), ghi = make_float4(-INFINITY, -INFINITY, -INFINITY, 0.0f);
    {
        const int g = lane & 7;
        const uint32_t c0 = own_c0 + (CS == 4 ? 2 * g : (CS == 8 ? g : (g >> 1)));
        if (c0 < a.nclu) {
            glo = a.bbox[2 * (size_t)c0];
            ghi = a.bbox[2 * (size_t)c0 + 1];
        }
        if (CS == 4 && c0 + 1 < a.nclu) box_union(glo, ghi, a.bbox[2 * (size_t)c0 + 2], a.bbox[2 * (size_t)c0 + 3]);
    }
    if (gather) {
        // radii of the boxes: the largest flagged radius inside (a radius 0
        // box passes no test): a maximum over the particles of each box
        float r = ih2;
        constexpr int kSpan = CS == 16 ? 16 : 8;
#pragma unroll
        for (int d = 1; d < kSpan; d <<= 1) r = fmaxf(r, __shfl_xor(r, d, kWave));
        glo.w = __builtin_sqrtf(__shfl(r, CS == 16 ? 16 * ((lane & 7) >> 1) : 8 * (lane & 7), kWave));
    }
    // (for CS = 16 lanes 2k and 2k + 1 hold the same box)
    if (CS == 16 ? (lane & 1) == 0 && lane < 2 * kBoxes : lane < kBoxes) {
        const int k = CS == 16 ? lane >> 1 : lane;
        s_box[w][2 * k] = glo;
        s_box[w][2 * k + 1] = ghi;
    }

    // Periodic axes: a pair can take an image one period away only if the
    // super-cluster lies within the largest search radius R of the far face
    // of the particles' span (a direct difference above L - R). Otherwise
    // every minimum image is the direct one and the super-cluster runs the
    // open-boundary tests; the margin on R keeps the decision on the safe side
    // of FP32 rounding, so no accepted pair changes.
    bool wraps = false;
    float span_c[3] = {0.0f, 0.0f, 0.0f};  // the super-cluster's box centre
    float reach2[3] = {0.0f, 0.0f, 0.0f};  // its half width and R: how far a j-particle's image matters
    int nimages = 1;  // a wrapping super-cluster so wide that a second image of a j-particle can matter: 8
    float wrap_err = 0.0f;
    if (kPbc) {
        float slo[3] = {glo.x, glo.y, glo.z}, shi[3] = {ghi.x, ghi.y, ghi.z};
        float r = glo.w;  // full build: replaced by the largest radius of all
#pragma unroll
        for (int d = 1; d < 8; d <<= 1) {  // (the boxes repeat every 8 lanes)
#pragma unroll
            for (int t = 0; t < 3; t++) {
                slo[t] = fminf(slo[t], __shfl_xor(slo[t], d, 64));
                shi[t] = fmaxf(shi[t], __shfl_xor(shi[t], d, 64));
            }
            r = fmaxf(r, __shfl_xor(r, d, 64));
        }
        const float4 rlo = a.cs_box[0], rhi = a.cs_box[1];  // root box: the particles' span
        if (!gather) r = fmaxf(r, rlo.w);  // pairs use max(h_i, h_j)
        const float plo[3] = {rlo.x, rlo.y, rlo.z}, phi[3] = {rhi.x, rhi.y, rhi.z};
        bool w_lane = false, far_lane = false;
#pragma unroll
        for (int t = 0; t < 3; t++) {
            if (a.per.L[t] < INFINITY) {
                const float reach = a.per.L[t] - 1.0001f * r - 1e-5f * a.per.L[t];
                w_lane = w_lane || !(phi[t] - slo[t] <= reach) || !(shi[t] - plo[t] <= reach);
                // the image nearest to the box's centre is the minimum image of
                // every pair within R if half the box and R stay inside half
                // a period
                span_c[t] = 0.5f * slo[t] + 0.5f * shi[t];
                reach2[t] = 1.0001f * (fmaxf(shi[t] - span_c[t], span_c[t] - slo[t]) + r);
                far_lane = far_lane || !(reach2[t] < 0.4999f * a.per.L[t]);
                wrap_err = fmaxf(wrap_err, a.per.L[t]);
            }
        }
        wraps = sfc_ballot(w_lane) != 0;
        if (wraps && sfc_ballot(far_lane)) nimages = 8;
    }
    const Period per = wraps ? a.per : Period{};

    // The filter's frame: positions relative to the middle particle, scaled so
    // that the super-cluster and a radius around it fill +-64 or so
    const int mid = sfc_popc(sfc_ballot(ix + iy + iz == ix + iy + iz && (int64_t)own_p0 + lane < n)) >> 1;
    // (a wrapping super-cluster: on a periodic axis relative to its box's centre)
    float cx = sfc_readlane_f(ix, mid), cy = sfc_readlane_f(iy, mid), cz = sfc_readlane_f(iz, mid);
    if (kPbc && wraps) {
        cx = a.per.L[0] < INFINITY ? span_c[0] : cx;
        cy = a.per.L[1] < INFINITY ? span_c[1] : cy;
        cz = a.per.L[2] < INFINITY ? span_c[2] : cz;
    }
    float sc, sc2;        // scale and its square
    float range;          // bound on the scaled squares that the filter takes
    float err_sq, err_0;  // its error bound's coefficients
    float h2_min;         // smallest squared radius of the super-cluster's particles
    {
        float dx = ix - cx, dy = iy - cy, dz = iz - cz;
        float m = ipresent ? fmaxf(__builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx)), ih2) : 0.0f;
        m = sfc_wave_max(m);
        int k = 6 - ((__builtin_amdgcn_frexp_expf(m) + 1) >> 1);
        k = k < -60 ? -60 : (k > 60 ? 60 : k);
        sc = ldexpf(1.0f, k);
        sc2 = ldexpf(1.0f, 2 * k);
        const float reach_i = __builtin_sqrtf(m * sc2) * 1.0001f;  // a bound on the scaled |x_i| and h_i
        dx *= sc;
        dy *= sc;
        dz *= sc;
        const float sq = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
        // infinite coordinates: every pair goes to the exact tests
        const bool serves = reach_i < 128.0f;
        range = serves ? kFar16 : -1.0f;
        ipresent = ipresent && serves;
        if (!ipresent) dx = dy = dz = 0.0f;
        const Operands A = operands<true>(dx, dy, dz, sq, sq - ih2 * sc2, ipresent);
        s_a[w][2][lane] = A.plain[0];
        s_a[w][3][lane] = A.plain[1];
        uint4_t f0 = A.plain[0], f1 = A.plain[1];
        f0[kSquareA] = A.other[0][0];
        f0[kSquareA + 1] = A.other[0][1];
        f1[kSquareA] = A.other[1][0];
        f1[kSquareA + 1] = A.other[1][1];
        s_a[w][0][lane] = f0;
        s_a[w][1][lane] = f1;
        // the smallest squared radius: j-particles with none above it need no
        // test of their own (a counting list's never do)
        h2_min = sfc_wave_min(ipresent && !gather ? ih2 : INFINITY);
        // E = |x_j|^2 err_sq + h_j^2 2^-17 + err_0 (see test_batch), scaled; N^2 is
        // at most 2 (reach_i^2 + |x_j|^2), 128 N at most N^2 + 64^2, and so on
        const float werr = wraps ? wrap_err * sc * 0x1p-19f : 0.0f;  // times N, at most (N^2 + 128^2) / 256
        err_sq = 0x1p-15f + werr * 0x1p-7f;
        err_0 = reach_i * reach_i * err_sq + 0x1p-4f + werr * 64.0f;
    }

    float inf = INFINITY;
    asm("" : "+v"(inf));  // kept in a register (see test_batch)

    // stack of node records {first, end, child count (0 = leaf), first child
    // slot}; a node is pushed only after its box passed the test
    uint4 *stack = s_stack[kDirect ? 0 : w];
    uint32_t *queue = s_queue[w];
    int sp = 0;
    // the tree of this super-cluster's system; list entries are cluster
    // indices relative to the system's first cluster
    uint32_t jbase = 0;
    if (kDirect) {
        // no tree
    } else if (a.seg.on()) {
        const int sy = a.seg.sc_sys[s];
        jbase = a.seg.pbase[sy] / CS;
        if (lane == 0) stack[0] = a.seg.roots[sy];
    } else {
        if (lane == 0) stack[0] = a.cs_rec[0];  // root
    }
    sp = 1;
    wave_sync();

    uint32_t nj = 0, prevj = 0xFFFFFFFFu, seg_words = 0;
    // entries collect in lane (index % 64) of ej / em and leave 64 at a time
    // into the next staging chunk: one coalesced store each, and the
    // compressed size of the 64-entry segment (first difference from the
    // previous segment's last index; difference 1: no nibble, up to 9: one,
    // else one plus its hex digits)
    uint32_t ej = 0, em = 0;
    uint32_t chunk = s;        // chunk being filled
    bool staged = true;        // false once the shared chunks ran out
    auto flush = [&](uint32_t cnt) SFC_INLINE {
        if (nj > cnt) {  // beyond the first chunk: take a shared one
            uint32_t id = kNoChunk;
            if (lane == 0 && staged) id = take_chunk(a.chunk_ctr, a.nshared, s);
            id = (uint32_t)__builtin_amdgcn_readfirstlane((int)id);
            if (id != kNoChunk) {
                if (lane == 0) a.chunk_next[chunk] = a.nsc + id;
                chunk = a.nsc + id;
            } else {
                if (lane == 0) atomicAdd(&a.status[kStChunks], 1u);  // a request left unserved (sizes the retry)
                staged = false;
            }
        }
        if (staged && (uint32_t)lane < cnt) {
            a.list_j[(size_t)chunk * kWave + lane] = ej;
            a.list_m[(size_t)chunk * kWave + lane] = (uint16_t)em;
        }
        const uint32_t up = sfc_prev_lane(ej);
        const uint32_t v = ej - (lane == 0 ? prevj : up);
        const uint32_t nib = (uint32_t)lane < cnt ? (v == 1u ? 0u : (v <= 9u ? 1u : 1u + nibbles_of(v))) : 0u;
        const uint32_t tot = sfc_readlane(sfc_incl_scan(nib), kWave - 1);
        seg_words += 2u + (tot + 7u) / 8u;
        prevj = sfc_readlane(ej, (int)cnt - 1);
    };

    // The queue of candidate j-clusters whose boxes came near (a ring);
    // batches of kBatch leave it in order. Lane (q, p) = (lane / CS, lane % CS)
    // takes particle p of the batch's candidate q: the loads read a clamped
    // index unconditionally, so the next batch's stay in flight while the
    // current batch is tested (a load behind a branch, or one whose value is
    // used at once, ends with a wait).
    uint32_t qh = 0, qt = 0;
    struct JLoad {
        float x, y, z, h;
    };
    const uint32_t n_last = (uint32_t)(n - 1);
    auto load_batch = [&](uint32_t b0, uint32_t cnt, JLoad &f) SFC_INLINE {
        const uint32_t q = (uint32_t)(lane / CS);
        const uint32_t p = queue[(b0 + (q < cnt ? q : 0u)) % kQueueCap] * CS + (uint32_t)(lane & (CS - 1));
        const uint32_t pc = p < n_last ? p : n_last;
        f.x = a.x[pc];
        f.y = a.y[pc];
        f.z = a.z[pc];
        f.h = a.h[pc];
    };

    // The exact FP32 tests of the tiles set in `aq` (lane q: i-cluster mask of
    // the batch's candidate q, cluster `cj`); returns the mask of those holding
    // a pair. Only the tiles that the filter left open come here: pairs within
    // its error of the radius, and the tiles of an i-cluster with itself. They
    // read their particles from memory again (few tiles: LDS copies of every
    // batch would cost more, and a wave per SIMD). Absent particles are far
    // away with a zero radius, as are a counting list's j radii and those of
    // unflagged i-particles.
    // Cluster size 8: a round gives one tile to each group of 8 lanes; lane
    // (g, l) takes i-particle l of its tile and steps through the 8
    // j-particles of its candidate, two of which it holds while the quad's
    // other lanes supply the rest (DPP operands).
    __shared__ uint32_t s_tile[kW][kLaneTiles ? 64 : 1];
    __shared__ uint64_t s_hits[kW][kLaneTiles ? 8 : 1];
    if constexpr (kLaneTiles) s_tile[w][lane] = 0u;  // entries past a batch's tiles: some valid tile
    auto particle = [&](uint32_t p, bool i_side) SFC_INLINE {
        const bool v = p < (uint64_t)n;
        const uint32_t pc = v ? p : (uint32_t)(n - 1);
        float hh = a.h[pc];
        if (gather && (!i_side || !a.p_active[pc])) hh = 0.0f;
        return make_float4(v ? a.x[pc] : kFar, v ? a.y[pc] : kFar, v ? a.z[pc] : kFar, v ? hh * hh : 0.0f);
    };
    auto exact_tiles = [&](uint32_t aq, uint32_t cj) SFC_INLINE -> uint32_t {
        if constexpr (kLaneTiles) {
            const int g = lane >> 3, l = lane & 7;
            const uint32_t am = (uint32_t)__shfl((int)aq, g, kWave);
            const bool bit = (am >> l) & 1u;
            const uint64_t W = sfc_ballot(bit);
            const int T = sfc_popc(W);
            const uint32_t k = __builtin_amdgcn_mbcnt_hi((uint32_t)(W >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)W, 0u));
            if (bit) s_tile[w][k] = (uint32_t)(l | (g << 3));  // tile k: its i-cluster and candidate
            wave_sync();
            // s_hits[r]: round r's ballot (byte g: group g, i.e. tile 8r + g,
            // saw a pair); bytes of tiles past T are never read
            for (int r = 0; 8 * r < T; r++) {
                const uint32_t tv = s_tile[w][8 * r + g];  // tiles past T: an older tile, results unread
                const uint32_t ci = own_c0 + (tv & 7u), c = (uint32_t)__shfl((int)cj, (int)(tv >> 3), kWave);
                const float4 ip = particle(8u * ci + (uint32_t)l, true);
                const float4 ja = particle(8u * c + (uint32_t)(l & 3), false), jz = particle(8u * c + 4u + (uint32_t)(l & 3), false);
                constexpr uint64_t kBytes = 0x0101010101010101ull;
                const uint64_t same = sfc_ballot(ci == c);
                uint64_t t = 0;
                static_for<8>([&](auto pc) SFC_INLINE {
                    constexpr int p = decltype(pc)::value;
                    const float4 &jq = p < 4 ? ja : jz;
                    float dx = quad_bcast<p & 3>(jq.x) - ip.x;
                    float dy = quad_bcast<p & 3>(jq.y) - ip.y;
                    float dz = quad_bcast<p & 3>(jq.z) - ip.z;
                    if (kPbc && wraps) wave_min_image(dx, dy, dz, a.per);
                    const float dxx = dx * dx;
                    const float d2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dxx));
                    // lane (g, l): i = l and j = p of the same cluster; the half
                    // list keeps j > i, the full list all but i = j
                    const uint64_t keep = half ? ~same | (((1ull << p) - 1ull) * kBytes) : ~(same & ((1ull << p) * kBytes));
                    t |= sfc_ballot(d2 < max_sq(quad_bcast<p & 3>(jq.w), ip.w)) & keep;
                });
                if (lane == 0) s_hits[w][r] = t;
            }
            wave_sync();
            // W's bit of rank k: tile k, byte k % 8 of round k / 8
            const uint32_t hw = reinterpret_cast<const uint32_t *>(s_hits[w])[(k >> 2) & 15u];
            const uint64_t R = sfc_ballot(bit && ((hw >> (8 * (k & 3u))) & 0xFFu) != 0u);
            return lane < kBatch ? (uint32_t)(R >> ((8 * lane) & 63)) & 0xFFu : 0u;
        } else {
            // candidate by candidate, whose particles a quad (CS = 4) or a row
            // (CS = 16) holds and hands round as DPP operands. CS = 4: all
            // i-clusters at once, lane l with i-particle l, as a candidate that
            // leaves one tile open mostly leaves all that are not set. CS = 16:
            // the open tiles one by one, row g from the candidate's particle 4g
            // on, so that four steps make the 16 x 16 pairs (all four i-clusters
            // at once: 16 steps). The i-particles come from the lanes that loaded
            // them, but are read again where registers are short (CS = 4,
            // periodic boxes), and nothing is loaded ahead: held values spilled.
            // us, by single tiles with both sides read from memory / now, half lists
            // at 200 neighbours: 200,000 particles in 200 clumps, clusters of 4 / 16,
            // 515 / 213 and 209 / 186 (clusters of 4 before the filter: 330);
            // 2,000,000 uniform, clusters of 4 686 / 684, periodic 920 / 889,
            // clusters of 16 661 / 648, periodic 858 / 849. With clusters of 8
            // the rounds above are 3 to 20 % faster.
            constexpr bool kHeld = CS == 16 && !kPbc;
            const uint32_t rot = CS == 16 ? 4u * ((uint32_t)lane >> 4) : 0u;
            float4 ih = {};
            if (kHeld) ih = particle(own_p0 + (uint32_t)lane, true);
            uint32_t out = 0;
            for (uint64_t todo = sfc_ballot(aq != 0u); todo; todo &= todo - 1ull) {
                const int q = __builtin_ctzll(todo);
                const uint32_t c = sfc_readlane(cj, q), am = sfc_readlane(aq, q);
                const float4 jp = particle(c * CS + (((uint32_t)lane + rot) & (uint32_t)(CS - 1)), false);
                // lane's i-particle against particle p of its quad or row, bit by bit
                auto near = [&](const float4 &ip, auto pc) SFC_INLINE -> uint64_t {
                    constexpr int p = decltype(pc)::value;
                    float dx = group_bcast<CS, p>(jp.x) - ip.x;
                    float dy = group_bcast<CS, p>(jp.y) - ip.y;
                    float dz = group_bcast<CS, p>(jp.z) - ip.z;
                    if (kPbc && wraps) wave_min_image(dx, dy, dz, a.per);
                    const float dxx = dx * dx;
                    const float d2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dxx));
                    return sfc_ballot(d2 < max_sq(group_bcast<CS, p>(jp.w), ip.w));
                };
                uint32_t got = 0;
                if constexpr (CS == 16) {
                    const uint32_t il = (uint32_t)lane & 15u;
                    for (uint32_t m = am; m; m &= m - 1u) {
                        const uint32_t t = (uint32_t)__builtin_ctz(m);
                        float4 ip;
                        if (kHeld) {
                            const int from = (int)((16u * t + il) << 2);
                            ip.x = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(ih.x)));
                            ip.y = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(ih.y)));
                            ip.z = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(ih.z)));
                            ip.w = __int_as_float(__builtin_amdgcn_ds_bpermute(from, __float_as_int(ih.w)));
                        } else {
                            ip = particle(own_p0 + 16u * t + il, true);
                        }
                        uint64_t hits = 0;
                        static_for<4>([&](auto pc) SFC_INLINE {
                            uint64_t r = near(ip, pc);
                            // the half list keeps j > i, the full list all but i = j
                            const uint32_t jl = rot + (uint32_t)decltype(pc)::value;
                            if (c == own_c0 + t) r &= sfc_ballot(half ? jl > il : jl != il);
                            hits |= r;
                        });
                        if (hits) got |= 1u << t;
                    }
                } else {
                    uint32_t pi = own_p0 + (uint32_t)lane;
                    asm volatile("" : "+v"(pi));  // (or the load is moved out of the loop)
                    const float4 ip = particle(pi, true);
                    const bool own = c - own_c0 < (uint32_t)kNsub;
                    uint64_t hits = 0;  // bit l: i-particle l has a pair
                    static_for<CS>([&](auto pc) SFC_INLINE {
                        uint64_t r = near(ip, pc);
                        const uint32_t pj = c * CS + (uint32_t)decltype(pc)::value;
                        if (own) r &= sfc_ballot(half ? pj > pi : pj != pi);
                        hits |= r;
                    });
                    // lane k: i-cluster k's particles
                    const bool hit = lane < kNsub && ((hits >> ((lane * CS) & 63)) & ((1ull << CS) - 1ull)) != 0ull;
                    got = (uint32_t)sfc_ballot(hit) & am;
                }
                out = lane == q ? got : out;
            }
            return out;
        }
    };

    // One batch: the filter decides every pair of the 64 x 64 block whose
    // squared distance is not within E of the larger squared radius. E bounds
    // the filter's error: with N >= |x_i| + |x_j| (scaled, so N is about 128),
    // the split coordinates and dropped products leave 2^-18.4 N^2, the FP32
    // accumulation of 16 products 2^-18.8 N^2, the rounding of x - c and of the
    // exact formula 2^-21 N^2, and halves too small for their normal range
    // (below 2^-14) 2^-11.4 N; 2^-16 N max(N, 128) + 2^-17 h_j^2 covers them with
    // room, and on a wrapping axis the roundings of x - c and of the image add
    // at most 2^-20.6 N L. A j-particle beyond the halves' range (or NaN: a
    // batch's padding), or any when an i-particle is, has E = inf: all its
    // pairs are open. Lanes without a particle hold some
    // particle of the same cluster or of an unused candidate again, which
    // changes no mask.
    auto test_batch = [&](const JLoad &f, uint32_t cnt) SFC_INLINE {
        const float hh = gather ? 0.0f : f.h;
        const float h2 = hh * hh;
        const bool both = sfc_ballot(h2 > h2_min) != 0;  // some max(h_i, h_j) may be h_j
        uint32_t seen_any = 0;
        uint64_t open_any[2] = {0, 0};  // lane l: j-particle l % 32 of either half has a pair within E of a radius
        uint64_t bad_any = 0;
        // Images of the batch: the nearest to the frame's centre; in a box only
        // a few radii wide also the second nearest on each periodic axis
        // (image bit t: axis t), where some j-particle's can reach. A pair is
        // near in one image if and only if it is near in its minimum image, as
        // every radius is below half a period.
        for (int img = 0; img < (kPbc ? nimages : 1); img++) {
            float dx = f.x - cx, dy = f.y - cy, dz = f.z - cz;
            if (kPbc && wraps) {
                dx = min_image(dx, a.per.L[0], a.per.hL[0]);
                dy = min_image(dy, a.per.L[1], a.per.hL[1]);
                dz = min_image(dz, a.per.L[2], a.per.hL[2]);
                if (img) {
                    if (img & 1) dx -= copysignf(a.per.L[0], dx);
                    if (img & 2) dy -= copysignf(a.per.L[1], dy);
                    if (img & 4) dz -= copysignf(a.per.L[2], dz);
                    const bool near = !((img & 1) && fabsf(dx) > reach2[0]) && !((img & 2) && fabsf(dy) > reach2[1]) &&
                                      !((img & 4) && fabsf(dz) > reach2[2]);
                    if (!sfc_ballot(near)) continue;
                }
            }
            dx *= sc;
            dy *= sc;
            dz *= sc;
            const float sq = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dx * dx));
            const float h2s = h2 * sc2;
            const bool bad = !(sq + h2s < range);
            float E = __builtin_fmaf(sq, err_sq, __builtin_fmaf(h2s, 0x1p-17f, err_0));
            E = bad ? INFINITY : E;
            Operands B = operands<false>(dx, dy, dz, sq, sq - h2s, true);
            uint32_t e0 = (uint32_t)__float_as_int(E), e1 = e0;
            swap_halves(e0, e1);  // e0: E of j-particle l % 32 of the first half, e1: of the second
            uint32_t seen = 0;  // candidate_mask's bits, the first one pushed ends highest
            static_for<2>([&](auto bc) SFC_INLINE {
                constexpr int b = decltype(bc)::value;
                const float Eb = __int_as_float((int)(b ? e1 : e0));
                // least d^2 - max(h_i, h_j)^2 of the group's four pairs; one block's
                // sums at a time (two would spill). (v_min3 from the register inf
                // on: a minimum of two sums alone would first quiet both)
                float x[2][4];
                static_for<2>([&](auto fc) SFC_INLINE {
                    constexpr int fh = decltype(fc)::value;
                    __builtin_amdgcn_sched_barrier(0);
                    const float16_t u = pair_block(s_a[w][fh][lane], B.plain[b]);  // d^2 - h_i^2
                    static_for<4>([&](auto gc) SFC_INLINE {
                        constexpr int g = decltype(gc)::value;
                        x[fh][g] = fminf(fminf(inf, u[4 * g]), u[4 * g + 1]);
                        x[fh][g] = fminf(fminf(x[fh][g], u[4 * g + 2]), u[4 * g + 3]);
                    });
                });
                if (both) {
                    B.plain[b][kSquareB] = B.other[b][0];
                    B.plain[b][kSquareB + 1] = B.other[b][1];
                    static_for<2>([&](auto fc) SFC_INLINE {
                        constexpr int fh = decltype(fc)::value;
                        __builtin_amdgcn_sched_barrier(0);
                        const float16_t v = pair_block(s_a[w][2 + fh][lane], B.plain[b]);  // d^2 - h_j^2
                        static_for<4>([&](auto gc) SFC_INLINE {
                            constexpr int g = decltype(gc)::value;
                            x[fh][g] = fminf(fminf(x[fh][g], v[4 * g]), v[4 * g + 1]);
                            x[fh][g] = fminf(fminf(x[fh][g], v[4 * g + 2]), v[4 * g + 3]);
                        });
                    });
                }
                __builtin_amdgcn_sched_barrier(0);
                float near = inf;
                static_for<8>([&](auto kc) SFC_INLINE {
                    constexpr int k = decltype(kc)::value;
                    const float v = x[k / 4][k % 4];
                    near = fminf(near, fabsf(v));
                    // the sign of x + E joins from the right (v_alignbit)
                    seen = __builtin_amdgcn_alignbit(seen, (uint32_t)__float_as_int(v + Eb), 31u);
                });
                open_any[b] |= sfc_ballot(!(near > Eb));
            });
            __builtin_amdgcn_sched_barrier(0);
            seen_any |= seen;
            bad_any |= sfc_ballot(bad);  // (bit l: j-particle l)
        }
        uint32_t mq = candidate_mask<CS>(__brev(seen_any) >> 16, lane);
        // lane q: candidate q of the batch; its tiles left open
        const uint32_t cj = queue[(qh + (uint32_t)(lane < (int)cnt ? lane : 0)) % kQueueCap];
        const bool used = lane < (int)cnt;
        const uint32_t rel = cj - own_c0;  // below kNsub: our own i-cluster rel
        uint32_t aq = 0;
        if (open_any[0] | open_any[1]) {
            const uint64_t oj = (uint64_t)fold_halves(open_any[0]) | ((uint64_t)fold_halves(open_any[1]) << 32);
            constexpr uint64_t kMine = (1ull << CS) - 1ull;
            const int sh = (lane * CS) & 63;
            if ((bad_any >> sh) & kMine) mq = 0;  // not even a number
            if (used && ((oj >> sh) & kMine)) aq = ~mq & S::kFull;
        }
        if (used && rel < (uint32_t)kNsub) {
            const uint32_t own = 1u << rel;
            if (half) {  // i-clusters after the candidate have no j > i in it
                mq &= own - 1u;
                aq &= own - 1u;
            } else {
                mq &= ~own;
            }
            aq |= own;
        }
        if (sfc_ballot(aq != 0u)) mq |= exact_tiles(aq, cj);
        // the candidates with a nonempty mask join the list in queue order
        // (lane (nj + rank) % 64 of ej / em)
        if (!used) mq = 0u;
        if constexpr (kDirect) {
            if (mq) s_mask[cj] = (Mask)mq;
            return;
        }
        const uint64_t ne = sfc_ballot(mq != 0u);
        if (ne) {
            const uint32_t c = (uint32_t)sfc_popc(ne);
            if (mq) s_ent[kDirect ? 0 : w][__builtin_amdgcn_mbcnt_lo((uint32_t)ne, 0u)] = make_uint2(cj - jbase, mq);
            wave_sync();
            const uint32_t base = nj & (kWave - 1);
            const uint32_t first = c < kWave - base ? c : kWave - base;
            const uint32_t d = (uint32_t)lane - base;
            if (d < first) {
                const uint2 e = s_ent[kDirect ? 0 : w][d];
                ej = e.x;
                em = e.y;
            }
            nj += first;
            if ((nj & (kWave - 1)) == 0) flush(kWave);
            if (c > first) {
                if ((uint32_t)lane < c - first) {
                    const uint2 e = s_ent[kDirect ? 0 : w][first + lane];
                    ej = e.x;
                    em = e.y;
                }
                nj += c - first;
            }
            wave_sync();  // the next batch rewrites s_ent
        }
    };

    // Candidate clusters of the leaves collect one per lane (cn of them, the
    // current leaf's from pos to pos_end next); 64 at a time are tested against
    // the boxes of the super-cluster's particles 8 at a time (their boxes from
    // LDS), the survivors join the queue in order and its whole batches are
    // tested.
    const uint64_t lt = sfc_lt_mask();
    if constexpr (kDirect) {
        // the waves take the groups of 8 clusters by turns, 64 at a time
        const uint32_t c_first = half ? own_c0 : 0u;  // (j-clusters wholly before i: no j > i)
        const uint32_t g_first = c_first / 8u, ngrp = (a.nclu + 7u) / 8u;
        for (uint32_t k0 = 0; g_first + k0 * kW + (uint32_t)w < ngrp; k0 += kWave) {
            const uint32_t g = g_first + (k0 + (uint32_t)lane) * kW + (uint32_t)w;
            bool gin = g < ngrp;
            if (a.lvl1) {
                const float4 l = a.lvl1[2 * (size_t)(gin ? g : 0u)], u = a.lvl1[2 * (size_t)(gin ? g : 0u) + 1];
                bool hit = false;
#pragma unroll
                for (int k = 0; k < kBoxes; k++)
                    hit = hit | boxes_near<kPbc>(s_box[w][2 * k], s_box[w][2 * k + 1], l, u, per);
                gin = gin && hit;
            }
            const uint64_t gs = sfc_ballot(gin);
            const uint32_t ng = (uint32_t)sfc_popc(gs);
            if (gin) s_grp[w][sfc_popc(gs & lt)] = g;
            wave_sync();
            for (uint32_t e0 = 0; e0 < ng; e0 += 8) {
                const uint32_t e = e0 + (uint32_t)(lane >> 3);
                const uint32_t c = 8u * s_grp[w][e < ng ? e : 0u] + (uint32_t)(lane & 7);
                const bool in = e < ng && c < a.nclu && c >= c_first;
                const float4 l = a.bbox[2 * (size_t)(in ? c : 0u)], u = a.bbox[2 * (size_t)(in ? c : 0u) + 1];
                bool hit = false;
#pragma unroll
                for (int k = 0; k < kBoxes; k++)
                    hit = hit | boxes_near<kPbc>(s_box[w][2 * k], s_box[w][2 * k + 1], l, u, per);
                const uint64_t sv = sfc_ballot(hit && in);
                if (hit && in) queue[(qt + (uint32_t)sfc_popc(sv & lt)) % kQueueCap] = c;
                qt += (uint32_t)sfc_popc(sv);
                wave_sync();
                for (; qt - qh >= (uint32_t)kBatch; qh += kBatch) {
                    JLoad f;
                    load_batch(qh, kBatch, f);
                    test_batch(f, kBatch);
                }
            }
            wave_sync();  // the next groups overwrite s_grp
        }
        if (qt != qh) {
            JLoad f;
            load_batch(qh, qt - qh, f);
            test_batch(f, qt - qh);
        }
        __syncthreads();
        if (w != 0) return;
        // the list: 64 clusters at a time, those with a mask to the lanes that
        // follow the entries so far (lane e % 64 for entry e)
        for (uint32_t c0 = c_first; c0 < a.nclu; c0 += kWave) {
            const uint32_t c = c0 + (uint32_t)lane;
            const uint32_t m = c < a.nclu ? s_mask[c] : 0u;
            const uint64_t ne = sfc_ballot(m != 0u);
            if (ne == 0) continue;
            const uint32_t cnt = (uint32_t)sfc_popc(ne), base = nj & (kWave - 1), below = (uint32_t)sfc_popc(ne & lt);
            const uint32_t to = (base + (m ? below : cnt + (uint32_t)lane - below)) & (kWave - 1);  // a permutation
            const uint32_t pj = (uint32_t)__builtin_amdgcn_ds_permute((int)(to << 2), (int)c);
            const uint32_t pm = (uint32_t)__builtin_amdgcn_ds_permute((int)(to << 2), (int)m);
            const uint32_t first = cnt < kWave - base ? cnt : kWave - base;
            const uint32_t d = (uint32_t)lane - base;
            if (d < first) {
                ej = pj;
                em = pm;
            }
            nj += first;
            if ((nj & (kWave - 1)) == 0) flush(kWave);
            if (cnt > first) {
                if ((uint32_t)lane < cnt - first) {
                    ej = pj;
                    em = pm;
                }
                nj += cnt - first;
            }
        }
    } else {
    uint32_t cand = 0, cn = 0, pos = 0, pos_end = 0;
    // Eight particles in the outskirts of a condensed system have a box that
    // holds its core, and the boxes let thousands of clusters through that no
    // particle's own sphere comes near. Where few of the tested clusters joined
    // the list, nodes and clusters are also tested against the particles one by
    // one. (16 systems, half of them Plummer spheres: a traversal at converged
    // radii 1.12 -> 0.39 ms, as its outermost super-clusters walked for 1 ms;
    // the 1/r sphere of 4,000,037 particles 1439 -> 1143 us. From 128 clusters
    // on with one in four listed: 512 and 2048 clusters 1209 and 1440 us for
    // the sphere; one in two costs uniform systems 5 %. Short lists meet the rule
    // where it pays little: half lists of a sphere of 1,000,000 at 30 neighbours
    // 278 us against 259 without, at 60 277, by the tests before the filter 266
    // and 293. One in eight gives 248 there, but 507 instead of 445 us for a
    // Plummer sphere of 200,000 at 200 neighbours.)
    bool strict = false;
    // does one of the `count` particles from p0 on come near the box?
    auto any_near = [&](uint32_t p0, uint32_t count, const float4 &lo, const float4 &hi) SFC_INLINE {
        bool near = false;
#pragma unroll 1
        for (uint32_t k = 0; k < count; k++) {
            const uint32_t pc = p0 + k < n_last ? p0 + k : n_last;
            float4 q = make_float4(a.x[pc], a.y[pc], a.z[pc], a.h[pc]);
            if (gather && !a.p_active[pc]) q.w = 0.0f;
            near = near || (q.w >= 0.0f && boxes_near<kPbc>(q, q, lo, hi, per));  // (NaN: a batch's padding)
        }
        return near;
    };
    for (bool more = true; more;) {
        if (pos < pos_end) {
            const uint32_t room = kWave - cn, left = pos_end - pos;
            const uint32_t take = left < room ? left : room;
            const uint32_t d = (uint32_t)lane - cn;
            if (d < take) cand = pos + d;
            cn += take;
            pos += take;
            if (cn < (uint32_t)kWave) continue;
        } else if (sp > 0) {
            sp--;
            const uint4 rv = stack[sp];
            const uint32_t nfirst = (uint32_t)__builtin_amdgcn_readfirstlane((int)rv.x);
            const uint32_t nend = (uint32_t)__builtin_amdgcn_readfirstlane((int)rv.y);
            const uint32_t nchild = (uint32_t)__builtin_amdgcn_readfirstlane((int)rv.z);
            const uint32_t cslot = (uint32_t)__builtin_amdgcn_readfirstlane((int)rv.w);
            if (nend > (uint64_t)n || nfirst >= nend || cslot + nchild > a.nslots) {  // only on a broken tree
                if (lane == 0) atomicOr(&a.status[kStTree], 16u);
                sp = 0;
                continue;
            }
            if (nchild == 0) {  // a leaf: its clusters not collected yet (pos_end: all before are)
                const uint32_t c0 = nfirst / CS;
                pos = c0 > pos_end ? c0 : pos_end;
                if (half && pos < own_c0) pos = own_c0;  // j-clusters wholly before i: no j > i
                const uint32_t e = (nend - 1) / CS + 1;
                pos_end = e > pos_end ? e : pos_end;
                continue;
            }
            // lane (ch, g): child ch = lane / 8 of the node against group g's box
            const int ch = lane >> 3;
            const bool act = ch < (int)nchild;
            // unconditional loads from a clamped slot (an internal node has
            // at least one child), then the select
            const uint32_t slot = cslot + (uint32_t)(act ? ch : 0);
            const float4 l = a.cs_box[2 * (size_t)slot];
            const float4 hi = a.cs_box[2 * (size_t)slot + 1];
            const uint4 crec = a.cs_rec[slot];
            const float4 lo = make_float4(l.x, l.y, l.z, gather ? 0.0f : l.w);  // own radius only when counting
            // a half list never needs a node that ends before the super-cluster
            const int gb = CS == 16 ? (lane & 7) >> 1 : lane & 7;
            bool hit = act && boxes_near<kPbc>(s_box[w][2 * gb], s_box[w][2 * gb + 1], lo, hi, per) &&
                       (!half || crec.y > own_p0);
            if (strict) hit = hit && any_near(own_p0 + 8u * (uint32_t)(lane & 7), 8u, lo, hi);
            const uint32_t keep = nonzero_bytes(sfc_ballot(hit));
            const int cnt = __popc(keep);
            if (sp + cnt > kStackCap) {  // cannot happen in a valid octree (depth <= 21)
                if (lane == 0) atomicOr(&a.status[kStTree], 8u);
                sp = 0;
                continue;
            }
            if ((lane & 7) == 0 && ((keep >> ch) & 1u)) {
                const int r = __popc(keep & ((1u << ch) - 1u));
                stack[sp + cnt - 1 - r] = crec;  // first child on top
            }
            sp += cnt;
            wave_sync();
            continue;
        } else {
            more = false;  // the last box step, then the rest of the queue
        }
        if (cn) {
            const float4 l = a.bbox[2 * (size_t)cand], u = a.bbox[2 * (size_t)cand + 1];  // (lanes past cn: an older candidate)
            const float4 blo = make_float4(l.x, l.y, l.z, gather ? 0.0f : l.w);  // own radius only when counting
            bool hit = false;
#pragma unroll
            for (int k = 0; k < kBoxes; k++)
                hit = hit | boxes_near<kPbc>(s_box[w][2 * k], s_box[w][2 * k + 1], blo, u, per);
            hit = hit && (uint32_t)lane < cn;
            if (strict && sfc_ballot(hit)) hit = hit && any_near(own_p0, kWave, blo, u);
            cn = 0;
            const uint64_t sv = sfc_ballot(hit);
            if (hit) queue[(qt + (uint32_t)sfc_popc(sv & lt)) % kQueueCap] = cand;
            qt += (uint32_t)sfc_popc(sv);
            wave_sync();
        }
        uint32_t total = qt - qh;  // whole batches, but at the end
        if (more) total = total / kBatch * kBatch;
        if (total == 0) continue;
        JLoad f;
        load_batch(qh, total < (uint32_t)kBatch ? total : (uint32_t)kBatch, f);
        while (total) {
            const uint32_t cnt = total < (uint32_t)kBatch ? total : (uint32_t)kBatch;
            const JLoad c = f;
            total -= cnt;
            if (total) load_batch(qh + cnt, total < (uint32_t)kBatch ? total : (uint32_t)kBatch, f);
            test_batch(c, cnt);
            qh += cnt;
        }
        strict = qh > kStrictFrom && nj < qh / 4;
    }
    }
    if (nj & (kWave - 1)) flush(nj & (kWave - 1));
    if (lane == 0) {
        const uint32_t mwords = (nj * S::kMaskBytes + 3u) / 4u;
        a.sc_nj[s] = staged ? nj : kUnstaged;
        a.sc_words[s] = staged ? mwords + (a.compress ? seg_words : nj) : 0u;
        atomicMax(&a.chunk_ctr[(s % kChunkStripes) * kStripeWords + 1], nj);  // longest list, per stripe
        if (!staged) atomicOr(&a.status[kStScratch], 1u);
    }
}

// ---------------------------------------------------------------------------
// Encoder: masks, then raw indices or 64-wide nibble segments.
// ---------------------------------------------------------------------------
struct EncArgs {
    uint32_t nsc;
    int compress;
    int mask_bytes;  // 2 for 16 i-clusters per super-cluster, else 1
    const uint32_t *list_j;  // staging chunks (see TravArgs)
    const uint16_t *list_m;
    const uint32_t *chunk_next;
    const uint32_t *sc_nj, *sc_off;  // sc_off has nsc + 1 entries (kSum: sc_words, the words of each list)
    uint32_t *sc_info;
    uint32_t *pool;
    uint64_t pool_words;
    const uint32_t *chunk_ctr;  // the traversal's stripe counters
    uint32_t nshared;
    uint32_t *status;
};

// kSum: every wave adds up the words of the lists before its own (up to
// kSumLists of them) instead of reading prefix sums, which take a
// launch of 3 us (32,768 particles: encoder and scan 10.9 -> 5.7 us).
constexpr uint32_t kSumLists = 1024;

__device__ __forceinline__ uint32_t sum_words(const uint32_t *words, uint32_t n) {
    uint32_t v = 0;
    for (uint32_t k = (uint32_t)sfc_lane(); k < n; k += kWave) v += words[k];
    return sfc_readlane(sfc_incl_scan(v), kWave - 1);
}

template <bool kSum>
__global__ __launch_bounds__(kWave * kWavesPerBlock) void k_encode(EncArgs a) {
    __shared__ uint32_t s_seg[kWavesPerBlock][kSegCap];
    const int lane = sfc_lane();
    const int w = threadIdx.x / kWave;
    // wave-uniform: keep the super-cluster index (and all derived from it) scalar
    const uint32_t s = (uint32_t)__builtin_amdgcn_readfirstlane((int)(xcd_remap(blockIdx.x, gridDim.x) * kWavesPerBlock + w));
    // the pool total (the scan's last entry) into the status block, the
    // shared staging chunks taken added to the requests left unserved (a
    // stripe counter runs past its share when a request probes it full), and
    // the longest list over the stripes' maxima
    if (blockIdx.x == 0 && w == 0) {
        uint32_t taken = 0, longest = 0;
        if ((uint32_t)lane < (uint32_t)kChunkStripes) {
            longest = a.chunk_ctr[lane * kStripeWords + 1];
            if ((uint32_t)lane < a.nshared) {
                const uint32_t cap = (a.nshared - lane + kChunkStripes - 1) / kChunkStripes;
                taken = min(a.chunk_ctr[lane * kStripeWords], cap);
            }
        }
        const uint32_t tot = sfc_readlane(sfc_incl_scan(taken), kWave - 1);
        const uint32_t pool = kSum ? sum_words(a.sc_off, a.nsc) : a.sc_off[a.nsc];
#pragma unroll
        for (int d = 1; d < kWave; d <<= 1) longest = max(longest, (uint32_t)__shfl_xor((int)longest, d, kWave));
        if (lane == 0) {
            a.status[kStTotalLo] = pool;
            a.status[kStChunks] += tot;
            a.status[kStMaxNj] = max(a.status[kStMaxNj], longest);
        }
    }
    if (s >= a.nsc) return;
    const uint32_t nj = a.sc_nj[s];
    const uint32_t off = kSum ? sum_words(a.sc_off, s) : a.sc_off[s];
    const uint32_t words = kSum ? a.sc_off[s] : a.sc_off[s + 1] - off;
    // a list that could not be staged or stored is recorded as empty (the
    // status block reports it), so that a pass launched regardless never
    // reads past the pool
    const bool fits = nj != kUnstaged && (uint64_t)off + words <= a.pool_words;
    if (lane == 0) {
        a.sc_info[2 * s] = off;
        a.sc_info[2 * s + 1] = fits ? nj : 0u;
        if (nj != kUnstaged && !fits) atomicOr(&a.status[kStPoolOverflow], 1u);
    }
    if (!fits) return;
    const uint32_t mwords = (nj * (uint32_t)a.mask_bytes + 3u) / 4u;
    uint32_t *mout = a.pool + off;
    uint32_t *out = mout + mwords;
    uint32_t *seg = s_seg[w];
    const uint64_t lt = sfc_lt_mask();
    uint32_t prevj = 0xFFFFFFFFu;
    uint32_t chunk = s;
    for (uint32_t b0 = 0; b0 < nj; b0 += kWave) {
        const uint32_t cnt = nj - b0 < (uint32_t)kWave ? nj - b0 : (uint32_t)kWave;
        const bool valid = (uint32_t)lane < cnt;
        // every lane of a 64-entry chunk is inside the staging arrays: the
        // loads go out unconditionally, the select follows
        const uint32_t jl = a.list_j[(size_t)chunk * kWave + lane];
        const uint32_t ml = (uint32_t)a.list_m[(size_t)chunk * kWave + lane];
        const uint32_t j = valid ? jl : 0u;
        const uint32_t m = valid ? ml : 0u;
        if (b0 + kWave < nj) chunk = a.chunk_next[chunk];
        // masks of this block: 4 (or 2) consecutive entries per word
        if (a.mask_bytes == 1) {
            uint32_t v = m << (8 * (lane & 3));
            v |= __shfl_xor(v, 1, 64);
            v |= __shfl_xor(v, 2, 64);
            if ((lane & 3) == 0 && (uint32_t)lane < cnt) mout[b0 / 4 + lane / 4] = v;
        } else {
            uint32_t v = m << (16 * (lane & 1));
            v |= __shfl_xor(v, 1, 64);
            if ((lane & 1) == 0 && (uint32_t)lane < cnt) mout[b0 / 2 + lane / 2] = v;
        }
        if (!a.compress) {
            if (valid) out[b0 + lane] = j;
            continue;
        }
        uint32_t jprev = sfc_prev_lane(j);
        if (lane == 0) jprev = prevj;
        const uint32_t v = j - jprev;
        const bool nonone = valid && v != 1u;
        const uint64_t mk = sfc_ballot(nonone);
        const bool small = v <= 9u;
        const uint32_t nn = nibbles_of(v);
        const uint32_t ndata = (nonone && !small) ? nn : 0u;
        const uint32_t info = small ? v + 6u : nn - 1u;
        const uint32_t ninfo = (uint32_t)sfc_popc(mk);
        const uint32_t ipos = (uint32_t)sfc_popc(mk & lt);
        const uint32_t incl = sfc_incl_scan(ndata);
        const uint32_t dpos = ninfo + incl - ndata;
        const uint32_t total_nib = ninfo + sfc_readlane(incl, kWave - 1);
        const uint32_t segw = 2u + (total_nib + 7u) / 8u;
        for (uint32_t q = lane; q < segw; q += kWave) seg[q] = 0u;
        wave_sync();
        if (lane == 0) {
            seg[0] = (uint32_t)mk;
            seg[1] = (uint32_t)(mk >> 32);
        }
        if (nonone) {
            atomicOr(&seg[2 + ipos / 8], info << (4 * (ipos % 8)));
            for (uint32_t d = 0; d < ndata; d++) {
                const uint32_t nib = (v >> (4 * (ndata - 1 - d))) & 0xFu;
                const uint32_t t = dpos + d;
                atomicOr(&seg[2 + t / 8], nib << (4 * (t % 8)));
            }
        }
        wave_sync();
        for (uint32_t q = lane; q < segw; q += kWave) out[q] = seg[q];
        wave_sync();
        out += segw;
        prevj = sfc_readlane(j, (int)cnt - 1);
    }
}

struct NlistWs {
    Octree tree;
    uint32_t nchunks;     // staging chunks: nsc first ones, then the shared ones
    uint32_t *list_j;
    uint16_t *list_m;
    uint32_t *chunk_next;
    uint32_t *sc_nj, *sc_words, *sc_off;
    uint32_t *sc_active;  // per super-cluster counts / flags for restricted rebuilds (h-iteration)
    uint32_t *sc_scan;    // their prefix sum (nsc + 1)
    uint8_t *p_active;    // per particle flags for restricted rebuilds
    void *scan_tmp;
    uint32_t *plist;      // the flagged particles, compacted
};

// Staging chunks per super-cluster (on average): max_j_per_sc rounded up to
// whole 64-entry chunks.
inline int64_t staging_chunks(int max_j_per_sc) { return ((int64_t)max_j_per_sc + kWave - 1) / kWave; }

void carve_nlist(Carver &cv, NlistWs &ws, int64_t n, const sfcnl_nlist_opts &o, int nsys = 1) {
    const uint32_t nsc = (uint32_t)((n + kScSize - 1) / kScSize);
    octree_carve(cv, ws.tree, n, o.leaf_bucket, nsys, o.cluster_size);
    ws.nchunks = nsc * (uint32_t)staging_chunks(o.max_j_per_sc);
    ws.list_j = cv.take<uint32_t>((size_t)ws.nchunks * kWave);
    ws.list_m = cv.take<uint16_t>((size_t)ws.nchunks * kWave);
    ws.chunk_next = cv.take<uint32_t>(ws.nchunks);
    ws.sc_nj = cv.take<uint32_t>(nsc);
    ws.sc_words = cv.take<uint32_t>(nsc);
    ws.sc_off = cv.take<uint32_t>((size_t)nsc + 1);
    ws.sc_active = cv.take<uint32_t>(nsc);
    ws.sc_scan = cv.take<uint32_t>((size_t)nsc + 1);
    ws.p_active = cv.take<uint8_t>((size_t)n);
    ws.scan_tmp = cv.take<char>(scan_tmp_bytes(nsc));
    ws.plist = cv.take<uint32_t>((size_t)n);
}

template <int CS, bool kPbc, int kDirect>
void launch_direct(int half, unsigned nsc, hipStream_t st, const TravArgs &ta) {
    const size_t lds = align_up((size_t)ta.nclu * (CS == 4 ? 2 : 1), 16);
    if (half)
        k_traverse<CS, true, kPbc, kDirect><<<nsc, kWave * kDirect, lds, st>>>(ta);
    else
        k_traverse<CS, false, kPbc, kDirect><<<nsc, kWave * kDirect, lds, st>>>(ta);
}

template <int CS, bool kPbc>
void launch_traverse_cs(int half, bool direct, unsigned nsc, hipStream_t st, const TravArgs &ta) {
    if (direct) {
        if (ta.n <= kDirectFew)
            launch_direct<CS, kPbc, kDirectWavesFew>(half, nsc, st, ta);
        else
            launch_direct<CS, kPbc, kDirectWavesMany>(half, nsc, st, ta);
        return;
    }
    const unsigned gb = blocks_for(nsc, kWavesPerBlock);
    if (half)
        k_traverse<CS, true, kPbc, 0><<<gb, kWave * kWavesPerBlock, 0, st>>>(ta);
    else
        k_traverse<CS, false, kPbc, 0><<<gb, kWave * kWavesPerBlock, 0, st>>>(ta);
}

template <bool kPbc>
void launch_traverse(int cs, int half, bool direct, unsigned nsc, hipStream_t st, const TravArgs &ta) {
    if (cs == 4)
        launch_traverse_cs<4, kPbc>(half, direct, nsc, st, ta);
    else if (cs == 16)
        launch_traverse_cs<16, kPbc>(half, direct, nsc, st, ta);
    else
        launch_traverse_cs<8, kPbc>(half, direct, nsc, st, ta);
}

// Periodic axes: the particles must span less than one period (the root box
// of the octree holds the exact extent).
__global__ void k_check_span(const float4 *__restrict__ root_box, Period per, uint32_t *status) {
    const float4 lo = root_box[0], hi = root_box[1];
    const bool bad = !(hi.x - lo.x < per.L[0]) || !(hi.y - lo.y < per.L[1]) || !(hi.z - lo.z < per.L[2]);
    if (bad) atomicOr(&status[kStInputErr], 8u);
}

int check_opts(sfcnl_ctx ctx, const sfcnl_nlist_opts *o) {
    if (!o) return set_err(ctx, SFCNL_E_ARG, "null options");
    if (o->cluster_size != 4 && o->cluster_size != 8 && o->cluster_size != 16)
        return set_err(ctx, SFCNL_E_ARG, "cluster_size %d not supported (4, 8, 16)", o->cluster_size);
    if (o->compress != 0 && o->compress != 1) return set_err(ctx, SFCNL_E_ARG, "compress must be 0 or 1");
    if (o->half != 0 && o->half != 1) return set_err(ctx, SFCNL_E_ARG, "half must be 0 or 1");
    if (o->leaf_bucket < 8 || o->leaf_bucket > 256)
        return set_err(ctx, SFCNL_E_ARG, "leaf_bucket %d outside [8, 256]", o->leaf_bucket);
    if (o->max_j_per_sc < 1) return set_err(ctx, SFCNL_E_ARG, "max_j_per_sc must be positive");
    if (!period_ok(o->period)) return set_err(ctx, SFCNL_E_ARG, "period must be 3 finite values >= 0");
    return SFCNL_OK;
}

}  // namespace
}  // namespace sfcnl

using namespace sfcnl;

int sfcnl::clusters_impl(sfcnl_ctx ctx, int64_t n, const float *x, const float *y, const float *z, const float *h,
                         int cs, float *bbox, const SegTable &seg) {
    if (n == 0) return SFCNL_OK;
    const int64_t nclu = (n + cs - 1) / cs;
    prof_mark(ctx, kStageClusters, false);
    float4 *b4 = reinterpret_cast<float4 *>(bbox);
    const unsigned g = blocks_for(nclu, 256);
    const bool vec = ((reinterpret_cast<uintptr_t>(x) | reinterpret_cast<uintptr_t>(y) |
                       reinterpret_cast<uintptr_t>(z) | reinterpret_cast<uintptr_t>(h)) & 15u) == 0;
    hipStream_t st = ctx->stream;
    if (cs == 4) {
        if (vec) k_cluster_bbox<4, true><<<g, 256, 0, st>>>(n, x, y, z, h, b4, ctx->d_status, seg);
        else k_cluster_bbox<4, false><<<g, 256, 0, st>>>(n, x, y, z, h, b4, ctx->d_status, seg);
    } else if (cs == 16) {
        if (vec) k_cluster_bbox<16, true><<<g, 256, 0, st>>>(n, x, y, z, h, b4, ctx->d_status, seg);
        else k_cluster_bbox<16, false><<<g, 256, 0, st>>>(n, x, y, z, h, b4, ctx->d_status, seg);
    } else {
        if (vec) k_cluster_bbox<8, true><<<g, 256, 0, st>>>(n, x, y, z, h, b4, ctx->d_status, seg);
        else k_cluster_bbox<8, false><<<g, 256, 0, st>>>(n, x, y, z, h, b4, ctx->d_status, seg);
    }
    SFCNL_LAUNCHED(ctx);
    prof_mark(ctx, kStageClusters, true);
    return SFCNL_OK;
}

extern "C" int build_clusters(sfcnl_ctx ctx, int64_t n, const float *d_x, const float *d_y, const float *d_z,
                              const float *d_h, int cluster_size, float *d_bbox_out) {
    if (!ctx) return SFCNL_E_ARG;
    if (n < 0 || n >= (int64_t(1) << 31)) return set_err(ctx, SFCNL_E_ARG, "build_clusters: n out of range");
    if (cluster_size != 4 && cluster_size != 8 && cluster_size != 16)
        return set_err(ctx, SFCNL_E_ARG, "build_clusters: cluster_size %d not supported (4, 8, 16)", cluster_size);
    if (n == 0) return SFCNL_OK;
    if (!d_x || !d_y || !d_z || !d_h || !d_bbox_out) return set_err(ctx, SFCNL_E_ARG, "build_clusters: null pointer");
    return clusters_impl(ctx, n, d_x, d_y, d_z, d_h, cluster_size, d_bbox_out, SegTable{});
}

size_t sfcnl::nlist_ws_bytes(int64_t n, const sfcnl_nlist_opts &o, int nsys) {
    Carver cv{nullptr, 0};
    NlistWs ws;
    carve_nlist(cv, ws, n, o, nsys);
    return align_up(cv.used, 256) + 256;
}

extern "C" int build_nlist_workspace(int64_t n, const sfcnl_nlist_opts *opts, size_t *ws_bytes) {
    if (n < 0 || !ws_bytes || !opts || check_opts(nullptr, opts)) return SFCNL_E_ARG;
    *ws_bytes = nlist_ws_bytes(n, *opts, 1);
    return SFCNL_OK;
}

int sfcnl::read_status(sfcnl_ctx ctx) {
    SFCNL_HIP(ctx, hipMemcpyAsync(ctx->h_status, ctx->d_status, kStWords * sizeof(uint32_t), hipMemcpyDeviceToHost,
                                  ctx->stream));
    SFCNL_HIP(ctx, hipStreamSynchronize(ctx->stream));
    return SFCNL_OK;
}

sfcnl::ActiveWs sfcnl::nlist_ws_active(void *d_ws, int64_t n, const sfcnl_nlist_opts &o, int nsys) {
    Carver cv{reinterpret_cast<char *>(d_ws), 0};
    NlistWs ws;
    carve_nlist(cv, ws, n, o, nsys);
    return ActiveWs{ws.sc_active, ws.sc_scan, ws.p_active, ws.scan_tmp, ws.plist, ws.tree.cs_box, ws.tree.cs_rec,
                    ws.tree.node_cap};
}

int sfcnl::nlist_build_impl(sfcnl_ctx ctx, int64_t n, const uint64_t *d_keys, const float *d_x, const float *d_y,
                            const float *d_z, const float *d_h, const float *d_bbox, const sfcnl_nlist_opts &o,
                            void *d_ws, size_t ws_bytes, uint32_t *d_sc_info, uint32_t *d_pool, size_t pool_bytes,
                            const SegTable &seg, bool readback, size_t *h_used_bytes, int64_t *h_max_nj,
                            const uint32_t *active, const uint8_t *p_active, TreeUse tree, const uint32_t *gate,
                            uint32_t gate_max) {
    if ((active || p_active) && o.half)
        return set_err(ctx, SFCNL_E_ARG, "build_nlist: a restricted rebuild needs the full list");
    const Period per = make_period(o.period);
    if (per.on() && seg.on()) return set_err(ctx, SFCNL_E_ARG, "batched lists take open boundaries only");
    const int nsys = seg.on() ? seg.nsys : 1;
    Carver cv{reinterpret_cast<char *>(d_ws), 0};
    NlistWs ws;
    carve_nlist(cv, ws, n, o, nsys);
    if (cv.used > ws_bytes) return set_err(ctx, SFCNL_E_ARG, "build_nlist: workspace %zu < %zu bytes", ws_bytes, cv.used);
    const uint32_t nsc = (uint32_t)((n + kScSize - 1) / kScSize);
    const int cs = o.cluster_size;
    const uint32_t nclu = (uint32_t)((n + cs - 1) / cs);
    hipStream_t st = ctx->stream;

    // the status words and stripe counters start at zero: cleared by a new
    // octree's first launch, else by a fill
    uint32_t *const st_clear = ctx->d_status + kStPoolOverflow;
    const int st_nclear = kStatusAlloc - kStPoolOverflow;
    int rc = SFCNL_OK;
    // small systems need no octree for their lists
    const bool direct = n <= direct_max(cs) && !seg.on() && !active && !p_active && !gate;
    const bool kept = tree == kTreeKeep;
    if (tree == kTreeNone && !direct) tree = kTreeNew;
    if (tree == kTreeBoxes && direct) tree = kTreeNone;  // (its radii are read by walks of whole lists only)
    if (tree != kTreeNew) {
        rc = fill_u32(ctx, st_clear, st_nclear, 0);
        if (rc) return rc;
    }
    const float4 *const boxes = reinterpret_cast<const float4 *>(d_bbox);
    const float4 *lvl1 = nullptr, *root = ws.tree.cs_box;
    if (!kept) prof_mark(ctx, kStageOctree, false);
    const bool levels = direct && (n > kDirectFew || per.on());  // a direct list's box levels
    if (tree == kTreeNew || tree == kTreeBoxes) {
        rc = tree == kTreeNew
                 ? octree_build(ctx, ws.tree, d_keys, d_x, d_y, d_z, d_h, boxes, seg, st_clear, st_nclear)
                 : octree_geometry(ctx, ws.tree, d_x, d_y, d_z, d_h, boxes, seg);
        if (rc) return rc;
    } else if (levels) {
        rc = box_levels_build(ctx, ws.tree, boxes, nullptr);
        if (rc) return rc;
    }
    if (levels) {  // (an octree comes with them)
        if (ws.tree.nboxlvl > 0) lvl1 = ws.tree.boxlvl[0];
        root = ws.tree.nboxlvl > 0 ? ws.tree.boxlvl[ws.tree.nboxlvl - 1] : boxes;
    }
    if (per.on() && !kept) {
        k_check_span<<<1, 1, 0, st>>>(root, per, ctx->d_status);
        SFCNL_LAUNCHED(ctx);
    }
    if (!kept) prof_mark(ctx, kStageOctree, true);

    TravArgs ta;
    ta.n = n;
    ta.nsc = nsc;
    ta.nclu = nclu;
    ta.compress = o.compress;
    ta.x = d_x;
    ta.y = d_y;
    ta.z = d_z;
    ta.h = d_h;
    ta.bbox = reinterpret_cast<const float4 *>(d_bbox);
    ta.cs_box = direct ? root : ws.tree.cs_box;
    ta.lvl1 = lvl1;
    ta.cs_rec = ws.tree.cs_rec;
    ta.nslots = ws.tree.node_cap;
    ta.seg = seg;
    ta.per = per;
    ta.active = active;
    ta.p_active = p_active;
    ta.gate = gate;
    ta.gate_max = gate_max;
    ta.list_j = ws.list_j;
    ta.list_m = ws.list_m;
    ta.chunk_next = ws.chunk_next;
    ta.nshared = ws.nchunks - nsc;
    ta.chunk_ctr = ctx->d_status + kStWords;
    ta.sc_nj = ws.sc_nj;
    ta.sc_words = ws.sc_words;
    ta.status = ctx->d_status;
    const unsigned gb = blocks_for(nsc, kWavesPerBlock);
    prof_mark(ctx, kStageTraverse, false);
    if (per.on())
        launch_traverse<true>(cs, o.half, direct, nsc, st, ta);
    else
        launch_traverse<false>(cs, o.half, direct, nsc, st, ta);
    SFCNL_LAUNCHED(ctx);
    prof_mark(ctx, kStageTraverse, true);
    prof_mark(ctx, kStageEncode, false);
    const bool sum = nsc <= kSumLists;
    if (!sum) {
        rc = scan_u32(ctx, ws.sc_words, ws.sc_off, nsc, ws.sc_off + nsc, ws.scan_tmp);
        if (rc) return rc;
    }

    EncArgs ea;
    ea.nsc = nsc;
    ea.compress = o.compress;
    ea.mask_bytes = cs == 4 ? 2 : 1;
    ea.list_j = ws.list_j;
    ea.list_m = ws.list_m;
    ea.chunk_next = ws.chunk_next;
    ea.sc_nj = ws.sc_nj;
    ea.sc_off = sum ? ws.sc_words : ws.sc_off;
    ea.sc_info = d_sc_info;
    ea.pool = d_pool;
    ea.pool_words = pool_bytes / 4;
    ea.chunk_ctr = ctx->d_status + kStWords;
    ea.nshared = ws.nchunks - nsc;
    ea.status = ctx->d_status;
    if (sum)
        k_encode<true><<<gb, kWave * kWavesPerBlock, 0, st>>>(ea);
    else
        k_encode<false><<<gb, kWave * kWavesPerBlock, 0, st>>>(ea);
    SFCNL_LAUNCHED(ctx);
    prof_mark(ctx, kStageEncode, true);
    if (!readback) return SFCNL_OK;

    rc = read_status(ctx);
    if (rc) return rc;
    return nlist_status(ctx, ctx->h_status, pool_bytes, o.max_j_per_sc, nsc, h_used_bytes, h_max_nj);
}

// Sizes and errors of a build from its copied status block.
int sfcnl::nlist_status(sfcnl_ctx ctx, const uint32_t *hs, size_t pool_bytes, int max_j_per_sc, uint32_t nsc,
                        size_t *h_used_bytes, int64_t *h_max_nj) {
    int rc;
    *h_used_bytes = (size_t)hs[kStTotalLo] * 4;
    *h_max_nj = hs[kStMaxNj];
    if (hs[kStInputErr]) {
        uint32_t e = hs[kStInputErr];
        rc = fill_u32(ctx, ctx->d_status + kStInputErr, 1, 0);
        if (rc) return rc;
        return set_err(ctx, SFCNL_E_INPUT,
                       "input error flags 0x%x (1: non-finite position, 2: bad radius, 4: bad permutation, "
                       "8: positions span a period or a radius reaches half of it)", e);
    }
    if (hs[kStTree]) return set_err(ctx, SFCNL_E_HIP, "internal error: octree invariant broken (0x%x)", hs[kStTree]);
    if (hs[kStScratch]) {
        *h_max_nj = staging_fit(hs, nsc);
        return set_err(ctx, SFCNL_E_CAPACITY, "staging list of max_j_per_sc %d too small: %lld holds the lists",
                       max_j_per_sc, (long long)*h_max_nj);
    }
    if (hs[kStPoolOverflow])
        return set_err(ctx, SFCNL_E_CAPACITY, "pool of %zu bytes < %zu needed", pool_bytes, *h_used_bytes);
    return SFCNL_OK;
}

extern "C" int build_nlist(sfcnl_ctx ctx, int64_t n, const uint64_t *d_keys, const float *d_x, const float *d_y,
                           const float *d_z, const float *d_h, const float *d_bbox, const sfcnl_nlist_opts *opts,
                           void *d_ws, size_t ws_bytes, uint32_t *d_sc_info, uint32_t *d_pool, size_t pool_bytes,
                           size_t *h_used_bytes, int64_t *h_max_nj) {
    if (!ctx) return SFCNL_E_ARG;
    int rc = check_opts(ctx, opts);
    if (rc) return rc;
    if (n < 0 || n >= (int64_t(1) << 31)) return set_err(ctx, SFCNL_E_ARG, "build_nlist: n out of range");
    if (!h_used_bytes || !h_max_nj) return set_err(ctx, SFCNL_E_ARG, "build_nlist: null result pointer");
    *h_used_bytes = 0;
    *h_max_nj = 0;
    if (n == 0) return SFCNL_OK;
    if (!d_keys || !d_x || !d_y || !d_z || !d_h || !d_bbox || !d_ws || !d_sc_info || (!d_pool && pool_bytes))
        return set_err(ctx, SFCNL_E_ARG, "build_nlist: null pointer");
    return nlist_build_impl(ctx, n, d_keys, d_x, d_y, d_z, d_h, d_bbox, *opts, d_ws, ws_bytes, d_sc_info, d_pool,
                            pool_bytes, SegTable{}, true, h_used_bytes, h_max_nj, nullptr, nullptr, kTreeNone);
}

// The async build's status to the host: word k (zero when `zero`) with the
// build's number in the high half, as one 64-bit store (single-copy atomic),
// so the host knows each word's build without a fence between the stores.
// One wave.
__global__ void k_post_status(const uint32_t *__restrict__ status, uint64_t *out, uint32_t seq, int zero) {
    const int t = threadIdx.x;
    if (t < kStWords) {
        const uint32_t v = zero ? 0u : status[t];
        __hip_atomic_store(out + t, ((uint64_t)seq << 32) | v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
    }
}

// The async build's bookkeeping: the status block posted behind the work
// (a kernel instead of a copy and an event, whose barrier would stall the
// stream), numbered so that the result call knows it when it arrives.
static int mark_pending(sfcnl_ctx ctx, int64_t n, const sfcnl_nlist_opts *opts, size_t pool_bytes) {
    ctx->pend_seq = ctx->pend_seq + 1u ? ctx->pend_seq + 1u : 1u;  // 0: nothing posted yet
    k_post_status<<<1, kWave, 0, ctx->stream>>>(ctx->d_status, ctx->d_pend, ctx->pend_seq, n > 0 ? 0 : 1);
    SFCNL_LAUNCHED(ctx);
    ctx->pend = 1;
    ctx->pend_pool_bytes = pool_bytes;
    ctx->pend_max_j = opts->max_j_per_sc;
    ctx->pend_nsc = (uint32_t)((n + kScSize - 1) / kScSize);
    return SFCNL_OK;
}

extern "C" int build_nlist_async(sfcnl_ctx ctx, int64_t n, const uint64_t *d_keys, const float *d_x,
                                 const float *d_y, const float *d_z, const float *d_h, const float *d_bbox,
                                 const sfcnl_nlist_opts *opts, void *d_ws, size_t ws_bytes, uint32_t *d_sc_info,
                                 uint32_t *d_pool, size_t pool_bytes) {
    if (!ctx) return SFCNL_E_ARG;
    ctx->pend = 0;
    int rc = check_opts(ctx, opts);
    if (rc) return rc;
    if (n < 0 || n >= (int64_t(1) << 31)) return set_err(ctx, SFCNL_E_ARG, "build_nlist_async: n out of range");
    if (n > 0 && (!d_keys || !d_x || !d_y || !d_z || !d_h || !d_bbox || !d_ws || !d_sc_info || (!d_pool && pool_bytes)))
        return set_err(ctx, SFCNL_E_ARG, "build_nlist_async: null pointer");
    if (n > 0) {
        size_t used;
        int64_t maxnj;
        rc = nlist_build_impl(ctx, n, d_keys, d_x, d_y, d_z, d_h, d_bbox, *opts, d_ws, ws_bytes, d_sc_info, d_pool,
                              pool_bytes, SegTable{}, false, &used, &maxnj, nullptr, nullptr, kTreeNone);
        if (rc) return rc;
    }
    return mark_pending(ctx, n, opts, pool_bytes);
}

extern "C" int build_nlist_result(sfcnl_ctx ctx, size_t *h_used_bytes, int64_t *h_max_nj) {
    if (!ctx) return SFCNL_E_ARG;
    if (!h_used_bytes || !h_max_nj) return set_err(ctx, SFCNL_E_ARG, "build_nlist_result: null result pointer");
    *h_used_bytes = 0;
    *h_max_nj = 0;
    if (!ctx->pend) return set_err(ctx, SFCNL_E_ARG, "build_nlist_result: no build_nlist_async pending");
    ctx->pend = 0;
    // wait until every status word carries the build's number; every 256
    // rounds the stream's state is asked: an error ends the wait, and an idle
    // stream means the post has run (its stores are visible by then)
    const uint32_t seq = ctx->pend_seq;
    uint32_t hs[kStWords];
    for (uint32_t spin = 1;; spin++) {
        int have = 0;
        for (int k = 0; k < kStWords; k++) {
            const uint64_t v = __atomic_load_n(&ctx->h_pend[k], __ATOMIC_ACQUIRE);
            hs[k] = (uint32_t)v;
            have += (uint32_t)(v >> 32) == seq;
        }
        if (have == kStWords) break;
        if (spin % 256u) continue;
        const hipError_t e = hipStreamQuery(ctx->stream);
        if (e == hipErrorNotReady) continue;
        if (e != hipSuccess) return set_err(ctx, SFCNL_E_HIP, "build_nlist_result: %s", hipGetErrorString(e));
        for (int k = 0; k < kStWords; k++) {
            const uint64_t v = __atomic_load_n(&ctx->h_pend[k], __ATOMIC_ACQUIRE);
            if ((uint32_t)(v >> 32) != seq)
                return set_err(ctx, SFCNL_E_HIP, "build_nlist_result: the stream is idle but the build's status did not arrive");
            hs[k] = (uint32_t)v;
        }
        break;
    }
    return nlist_status(ctx, hs, ctx->pend_pool_bytes, ctx->pend_max_j, ctx->pend_nsc, h_used_bytes, h_max_nj);
}
