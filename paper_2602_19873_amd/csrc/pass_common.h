// Pieces shared by the list passes (the SPH density pass and the
// Lennard-Jones + Coulomb pass): the wave-level decoder of one compressed
// segment (Sec. II-B), the XCD-aware block order, the lane roles that map
// list tiles onto a wavefront, DPP sums inside lane groups, and the wave's
// i-box that the periodic batch test (far_from_box) takes.
#pragma once
#include "internal.h"

namespace sfcnl {
namespace passk {

constexpr int kWavesPerBlock = 4;
// Position for absent particles: any distance to it overflows to +inf.
constexpr float kFar = 3.0e38f;

__device__ __forceinline__ unsigned xcd_remap(unsigned b, unsigned g) {
    const unsigned per = g / 8, rem = g % 8, x = b % 8, i = b / 8;
    return x < rem ? x * (per + 1) + i : rem * (per + 1) + (x - rem) * per + i;
}

__device__ __forceinline__ uint32_t nibble_at(const uint8_t *stream, uint32_t t) {
    return (uint32_t)(stream[t >> 1] >> ((t & 1u) * 4u)) & 0xFu;
}

// Decodes one segment of `cnt` differences at pool[p..] whose previous index
// is prevj; lane k returns index k (lanes >= cnt return garbage). Advances p
// past the segment.
__device__ __forceinline__ uint32_t decode_segment(const uint32_t *__restrict__ pool, uint32_t &p, uint32_t cnt,
                                                   uint32_t prevj) {
    const int lane = sfc_lane();
    const uint32_t lo = pool[p], hi = pool[p + 1];
    const uint64_t m = ((uint64_t)hi << 32) | lo;
    const uint8_t *stream = reinterpret_cast<const uint8_t *>(pool + p + 2);
    const bool valid = (uint32_t)lane < cnt;
    const bool nonone = valid && ((m >> lane) & 1ull);
    const uint32_t ninfo = (uint32_t)sfc_popc(m);
    uint32_t v = 1u, nd = 0u;
    if (nonone) {
        const uint32_t inf = nibble_at(stream, (uint32_t)sfc_popc(m & sfc_lt_mask()));
        if (inf >= 8u)
            v = inf - 6u;
        else
            nd = inf + 1u;
    }
    const uint32_t incl = sfc_incl_scan(nd);
    if (nd) {
        uint32_t t = ninfo + incl - nd;
        v = 0u;
        for (uint32_t d = 0; d < nd; d++) v = (v << 4) | nibble_at(stream, t + d);
    }
    const uint32_t total_nib = ninfo + sfc_readlane(incl, kWave - 1);
    p += 2u + (total_nib + 7u) / 8u;
    return prevj + sfc_incl_scan(valid ? v : 0u);
}

// i-particle held in register k by a lane (the traversal's lane roles):
// CS = 8: 8k + lane / 8; CS = 4 and 16: 16k + lane / 4.
template <int CS>
__device__ __forceinline__ int ipart(int k, int lane) {
    return CS == 8 ? 8 * k + (lane >> 3) : 16 * k + (lane >> 2);
}

constexpr int kPassSplitMax = 8;

// Moves the list entries (mask, j-cluster) of the lanes with `keep` up, in
// their order; cnt becomes their number.
__device__ __forceinline__ void sfc_compact(bool keep, uint32_t &mv, uint32_t &jv, uint32_t &cnt) {
    const uint64_t has = sfc_ballot(keep);
    const int rest = sfc_popc(has);
    const int below = (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(has >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)has, 0u));
    const int to = (keep ? below : rest + sfc_lane() - below) << 2;  // a permutation of the lanes
    mv = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)mv);
    jv = (uint32_t)__builtin_amdgcn_ds_permute(to, (int)jv);
    cnt = (uint32_t)rest;
}

// Wavefronts that share a super-cluster's list. With one each, a pass takes
// as long as its longest list until some thousand super-clusters fill the GPU.
// A full list is split by i-clusters (every part decodes it and evaluates its
// own clusters' tiles), so a particle's sum has one order whatever the split;
// a half list, whose sums meet in atomics in any case, by its entries. Limits
// where more parts stop paying; us with 1 / 2 / 4 / 8 parts (d density pass,
// f force pass, uniform systems and lattices):
//   full, clusters of 8:  d  32768: 117 / 88 / 68 / 58     f  32768: 84 / 63 / 44 / 38
//                         d  65536: 126 / 101 / 86 / 101   f  97336: 105 / 87 / 77 / 93
//                         d 131072: 125 / 132 / 136 / 165  f 262144: 126 / 142 / 157 / 196
//   full, clusters of 4:  d  65536: 152 / 121 / 100        f 125000: 139 / 129 / 122
//   half, clusters of 8:  d  32768: 108 / 65 / 43 / 35     f  64000: 120 / 73 / 50 / 51
//                         d 262144: 140 / 114 / 109 / 140  f 262144: 142 / 115 / 114 / 146
//                         d 800000: 276 / 260 / 281        f 729000: 252 / 236 / 254 / 364
//                         d 2097152: 581 / 590 / 665       f 4096000: 1144 / 1197 / 1378
//   half, clusters of 4:  d  65536: 265 / 145 / 86 / 67    f 125000: 223 / 133 / 91 / 91
//                         d 800000: 501 / 422 / 403        f 262144: 248 / 185 / 153 / 163
// (clusters of 16 behave as clusters of 4; their full lists have four
// i-registers to share out). Lists of few entries gain less, and the largest
// shared ones lose: half, clusters of 8, density pass in us with 1 / 2 / 4 parts
//   at 10 neighbours (30 entries)  120000: 37 / 29 / 30  262000: 43 / 40 / 46  1048000: 94 / 101 / 132
//   at 30 neighbours (42 entries)  120000: 49 / 37 / 36  262000: 59 / 51 / 54  1048000: 133 / 138 / 167
//   at 60 neighbours (56 entries)  120000: 64 / 45 / 43  262000: 79 / 67 / 67  1048000: 178 / 180 / 209
// The rule does not see the lists. (Parts that end at once where a list is short
// cost as much: idle wavefronts of a block hold its LDS, blocks of one wavefront
// starve the dispatch.)
inline uint32_t pass_split(int cs, bool half, int64_t nsc) {
    if (!half) return nsc <= 512 && cs == 8 ? 8u : (nsc <= 1600 ? 4u : 1u);
    if (nsc <= (cs == 8 ? 800 : 1600)) return 8u;
    if (nsc <= (cs == 8 ? 4096 : 16384)) return 4u;
    return cs == 8 && nsc <= 16384 ? 2u : 1u;
}

// Super-cluster and part of this wavefront: a block holds several
// super-clusters (split 1) or the parts of one.
__device__ __forceinline__ uint32_t wave_sc(uint32_t split, uint32_t &part) {
    const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const uint32_t b = (uint32_t)xcd_remap(blockIdx.x, gridDim.x);
    part = split > 1 ? w : 0u;
    return split > 1 ? b : b * (blockDim.x / kWave) + w;
}

// Cross-lane sums inside groups of 4, 8 or 16 consecutive lanes with DPP
// (quad swaps, then the mirrored half row, then the mirrored row): every lane
// of a group ends with the group total.
template <int CTRL>
__device__ __forceinline__ float dpp_f(float v) {
    return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ int dpp_i(int v) {
    return __builtin_amdgcn_update_dpp(0, v, CTRL, 0xF, 0xF, false);
}
template <int kLanes>
__device__ __forceinline__ void group_sum(float &f, int &c) {
    f += dpp_f<0xB1>(f);  // quad_perm [1, 0, 3, 2]
    c += dpp_i<0xB1>(c);
    f += dpp_f<0x4E>(f);  // quad_perm [2, 3, 0, 1]
    c += dpp_i<0x4E>(c);
    if (kLanes >= 8) {
        f += dpp_f<0x141>(f);  // row_half_mirror
        c += dpp_i<0x141>(c);
    }
    if (kLanes == 16) {
        f += dpp_f<0x140>(f);  // row_mirror
        c += dpp_i<0x140>(c);
    }
}

template <int kLanes>
__device__ __forceinline__ void group_sum(float &f) {
    f += dpp_f<0xB1>(f);
    f += dpp_f<0x4E>(f);
    if (kLanes >= 8) f += dpp_f<0x141>(f);
    if (kLanes == 16) f += dpp_f<0x140>(f);
}

// Lane roles of the symmetric pass (the i-particles in the low lane bits, so
// that a j-particle's sum over the i side stays inside a DPP row):
//   CS = 8:  lane = 8 jl + il; register k holds i-particle 8k + il;
//   CS = 4:  lane = 16 jl + 4q + il; register k holds i-particle 16k + 4q + il
//            (i-cluster 4k + q);
//   CS = 16: lane = 16 jq + il; register k holds i-particle 16k + il; the
//            lane takes j-particles 4t + jq.
template <int CS>
__device__ __forceinline__ int ipart_sym(int k, int lane) {
    return CS == 8 ? 8 * k + (lane & 7) : 16 * k + (lane & 15);
}

template <int kNreg>
__device__ __forceinline__ void wave_range(const float (&v)[kNreg], float &lo, float &hi) {
    lo = v[0];
    hi = v[0];
#pragma unroll
    for (int k = 1; k < kNreg; k++) {
        lo = fminf(lo, v[k]);
        hi = fmaxf(hi, v[k]);
    }
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        lo = fminf(lo, __shfl_xor(lo, d, kWave));
        hi = fmaxf(hi, __shfl_xor(hi, d, kWave));
    }
    // wave-uniform: scalar registers
    lo = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, lo)));
    hi = __builtin_bit_cast(float, __builtin_amdgcn_readfirstlane(__builtin_bit_cast(int, hi)));
}
template <int kNreg>
__device__ __forceinline__ IBox ibox_of(const float (&ix)[kNreg], const float (&iy)[kNreg], const float (&iz)[kNreg]) {
    IBox b;
    wave_range<kNreg>(ix, b.lo[0], b.hi[0]);
    wave_range<kNreg>(iy, b.lo[1], b.hi[1]);
    wave_range<kNreg>(iz, b.lo[2], b.hi[2]);
    return b;
}

}  // namespace passk
}  // namespace sfcnl
