// Compressed 1x1 list: the combination of the index compression with a full
// neighbour list that the paper leaves as future work (Sec. V). Row i holds
// particle i's neighbours in the pair set (j != i, d2 < max(h_i, h_j)^2) in
// ascending order, encoded as the index stream of a super-cluster list
// without masks (differences from -1, nibble segments of 64 values,
// Sec. II-B/II-C); rows follow each other in particle order.
//
// Build: from a full cluster list. One wavefront takes 8 consecutive particles
// (one cluster of 8, two of 4, half of one of 16): it decodes their
// super-cluster's list 64 entries at a time, keeps the entries whose mask holds
// one of their i-clusters (a ballot compaction into LDS), and fetches the
// particles of 64 / CS of those j-clusters at a time, one per lane; each of the
// 8 particles then tests all 64 with the exact FP32 pair formula and appends the
// survivors (already in ascending order) to its pending buffer in LDS, and a
// segment is encoded whenever 64 are pending. A sizing run and a writing run
// around a prefix sum place the rows deterministically. (One wavefront per
// particle decoded the list and fetched the candidates 8 times as often, and
// placed the nibbles one LDS atomic at a time: sizing 729 -> 331 us, writing
// 893 -> 521 us for 500,009 uniform particles of ~240 neighbours.)
//
// Pass: one wavefront per row brings the row's words into LDS with one or two
// coalesced loads, decodes 64 neighbours per step from there and evaluates each
// lane's pair once, a step's particles loading while the next one is decoded; no
// tile of a cluster pair is wasted. (Decoding from memory, every step waited in
// turn for its bitmask, its info nibbles, its data nibbles and its particles: 517
// -> 292 us for 500,009 particles; 8 rows per wavefront from one staging: 314.)
#include "internal.h"
#include "pass_common.h"
#include "row_stage.h"

namespace sfcnl {
namespace {

using namespace passk;

constexpr int kSegCap = 80;  // words of one 64-value segment: 2 + (64 + 512 + 7) / 8

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

__device__ __forceinline__ uint32_t nibbles_of(uint32_t v) { return (32u - (uint32_t)__clz((int)v) + 3u) >> 2; }

struct RowArgs {
    int64_t n;
    const uint32_t *sc_info, *pool;  // the full cluster list
    const float *x, *y, *z, *h;
    Period per;
    int compress;                    // encoding of the rows
    uint32_t *row_words;             // sizing run: words of each row
    const uint32_t *row_off;         // writing run: prefix sum of row_words (n + 1)
    uint32_t *row_info;              // writing run: {word offset, count} per particle
    uint32_t *out;
    uint64_t out_words;
    uint32_t *status;
};

// Rows per wavefront of the build: a wavefront of 8 shares most, but takes as
// long as its rows need one after another, so small systems, which leave the GPU
// half empty, take 4 or 1. Builds in us with 1 / 4 / 8, uniform systems at 200
// neighbours, lists of clusters of 8 (of 4 and 16 alike to within 10 %, the
// limits the same):
//   particles      nibble segments      raw indices
//      8,000         69 /  76 /  95       64 /  66 /  77
//     11,000         77 /  79 / 100       72 /  69 /  82
//     32,000        126 / 115 / 121      114 /  96 /  98
//    110,000        352 / 258 / 262      316 / 206 / 202
//    160,000        470 / 330 / 325      421 / 255 / 241
//    500,009      1,465 / 930 / 861    1,365 / 708 / 625
// (At 50 neighbours nibble segments 52 / 53 / 60, 83 / 72 / 74 and 202 / 145 / 142
// at 8,000, 32,000 and 110,000. Decoding and testing 8 times, a row per wavefront
// without the present encoder, took 71, 138, 386 and 1,620 at 8,000, 32,000,
// 110,000 and 500,009.)
constexpr int64_t kRows4Min = 12000, kRows8Min = 128000;

// The nibbles of v from its most significant hex digit on, the first in the low
// bits (nd digits, v > 0).
__device__ __forceinline__ uint32_t digits_first(uint32_t v, uint32_t nd) {
    v <<= 4u * (8u - nd);                                              // the first digit on top
    v = __builtin_bswap32(v);                                          // bytes, then the nibbles in them, reversed
    return ((v >> 4) & 0x0F0F0F0Fu) | ((v & 0x0F0F0F0Fu) << 4);
}

// ORs `bits` (fewer than 9 nibbles) into the nibble stream at words[] from
// nibble t on.
__device__ __forceinline__ void put_nibbles(uint32_t *words, uint32_t t, uint32_t bits) {
    const uint64_t b = (uint64_t)bits << (4u * (t & 7u));
    atomicOr(&words[t >> 3], (uint32_t)b);
    if ((uint32_t)(b >> 32)) atomicOr(&words[(t >> 3) + 1u], (uint32_t)(b >> 32));
}

template <int CS, int kRows, bool kCompIn, bool kWrite, bool kPbc>
__global__ __launch_bounds__(kWave) void k_rows(RowArgs a) {
    constexpr int kPerStep = kWave / CS;  // candidate j-clusters tested per step
    __shared__ uint32_t s_cand[kWave];
    __shared__ uint32_t s_pend[kRows][2 * kWave];
    __shared__ uint32_t s_seg[kSegCap + 1];
    const int lane = sfc_lane();
    const uint64_t lt = sfc_lt_mask();
    const uint32_t n = (uint32_t)a.n;
    const uint32_t grp = xcd_remap(blockIdx.x, gridDim.x);
    const uint32_t i0 = grp * kRows;
    if (i0 >= n) return;
    const uint32_t rows = n - i0 < (uint32_t)kRows ? n - i0 : (uint32_t)kRows;
    const uint32_t s = i0 / kScSize, g = (i0 % kScSize) / 8u;
    // entries with a mask bit of one of our i-clusters
    const uint32_t pick = CS == 4 ? 3u << (2 * g) : (CS == 8 ? 1u << g : 1u << (g >> 1));
    // the rows' particles, wave-uniform (rows past the end: the last particle
    // again, whose pairs are dropped)
    float xi[kRows], yi[kRows], zi[kRows], hi2[kRows];
    {
        const uint32_t p = i0 + ((uint32_t)lane < rows ? (uint32_t)lane : rows - 1u);
        const float px = a.x[p], py = a.y[p], pz = a.z[p], ph = a.h[p];
#pragma unroll
        for (int r = 0; r < kRows; r++) {
            xi[r] = sfc_readlane_f(px, r);
            yi[r] = sfc_readlane_f(py, r);
            zi[r] = sfc_readlane_f(pz, r);
            const float h = sfc_readlane_f(ph, r);
            hi2[r] = h * h;
        }
    }
    const uint32_t off = a.sc_info[2 * s], nj = a.sc_info[2 * s + 1];
    const uint8_t *mbytes = reinterpret_cast<const uint8_t *>(a.pool + off);
    const uint16_t *mshorts = reinterpret_cast<const uint16_t *>(a.pool + off);
    uint32_t p = off + (nj * (CS == 4 ? 2u : 1u) + 3u) / 4u;

    // row state in lane r: words and neighbours emitted, the last neighbour
    // emitted (differences start from -1), and where the row goes
    uint32_t st_words = 0, st_count = 0, st_prev = 0xFFFFFFFFu, st_off = 0;
    uint32_t fits = 0;  // rows that fit the pool
    if (kWrite) {
        uint32_t end = 0;
        if ((uint32_t)lane < rows) {
            st_off = a.row_off[i0 + lane];
            end = a.row_off[i0 + lane + 1];
        }
        fits = (uint32_t)sfc_ballot((uint32_t)lane < rows && (uint64_t)end <= a.out_words);
        if (fits == 0) {
            if ((uint32_t)lane < rows) {
                a.row_info[2 * (size_t)(i0 + lane)] = st_off;
                a.row_info[2 * (size_t)(i0 + lane) + 1] = 0u;
            }
            if (lane == 0) atomicOr(&a.status[kStPoolOverflow], 1u);
            return;
        }
    }
    // emits the first m pending neighbours of row r as one segment (or raw words)
    auto flush = [&](uint32_t r, uint32_t m) __attribute__((always_inline)) {
        const bool valid = (uint32_t)lane < m;
        const uint32_t j = s_pend[r][lane];  // (lanes past m: unused)
        const uint32_t words = sfc_readlane(st_words, (int)r);
        uint32_t add = m;
        if (a.compress) {
            const uint32_t prev = sfc_readlane(st_prev, (int)r);
            const uint32_t up = sfc_prev_lane(j);
            const uint32_t v = j - (lane == 0 ? prev : up);
            const bool nonone = valid && v != 1u;
            const uint64_t mk = sfc_ballot(nonone);
            const bool small = v <= 9u;
            const uint32_t nn = nibbles_of(v);
            const uint32_t ndata = (nonone && !small) ? nn : 0u;
            const uint32_t ninfo = (uint32_t)sfc_popc(mk);
            const uint32_t incl = sfc_incl_scan(ndata);
            const uint32_t total_nib = ninfo + sfc_readlane(incl, kWave - 1);
            add = 2u + (total_nib + 7u) / 8u;
            if (kWrite && ((fits >> r) & 1u)) {
                uint32_t *out = a.out + sfc_readlane(st_off, (int)r) + words;
                s_seg[lane] = 0u;
                if (lane < kSegCap + 1 - kWave) s_seg[kWave + lane] = 0u;
                wave_sync();
                if (nonone) {
                    const uint32_t info = small ? v + 6u : nn - 1u;
                    put_nibbles(s_seg + 2, (uint32_t)sfc_popc(mk & lt), info);
                    if (!small) put_nibbles(s_seg + 2, ninfo + incl - ndata, digits_first(v, nn));
                }
                wave_sync();
                const uint32_t lo = (uint32_t)mk, hi = (uint32_t)(mk >> 32);
                for (uint32_t q = (uint32_t)lane; q < add; q += kWave) out[q] = q == 0 ? lo : (q == 1 ? hi : s_seg[q]);
                wave_sync();
            }
        } else if (kWrite && ((fits >> r) & 1u)) {
            if (valid) a.out[sfc_readlane(st_off, (int)r) + words + lane] = j;
        }
        const uint32_t lastj = sfc_readlane(j, (int)m - 1);
        const bool mine = (uint32_t)lane == r;
        st_prev = mine ? lastj : st_prev;
        st_words += mine ? add : 0u;
        st_count += mine ? m : 0u;
    };

    uint32_t npend[kRows];
#pragma unroll
    for (int r = 0; r < kRows; r++) npend[r] = 0;
    uint32_t prevj = 0xFFFFFFFFu;  // decoding state of the cluster list
    for (uint32_t b0 = 0; b0 < nj; b0 += kWave) {
        const uint32_t cntb = nj - b0 < (uint32_t)kWave ? nj - b0 : (uint32_t)kWave;
        uint32_t jv;
        if (kCompIn)
            jv = decode_segment(a.pool, p, cntb, prevj);
        else
            jv = (uint32_t)lane < cntb ? a.pool[p + b0 + lane] : 0u;
        uint32_t mv = 0u;
        if ((uint32_t)lane < cntb) mv = CS == 4 ? (uint32_t)mshorts[b0 + lane] : (uint32_t)mbytes[b0 + lane];
        prevj = sfc_readlane(jv, (int)cntb - 1);
        // the entries whose mask holds one of our i-clusters, in list (ascending) order
        const bool sel = (mv & pick) != 0u;
        const uint64_t bsel = sfc_ballot(sel);
        const uint32_t ncand = (uint32_t)sfc_popc(bsel);
        wave_sync();  // the last block's reads of s_cand are done
        if (sel) s_cand[sfc_popc(bsel & lt)] = jv;
        wave_sync();
        struct JLoad {
            float x, y, z, h;
            uint32_t j;
        };
        // lane (q, p): particle p of candidate k0 + q; the loads read a clamped
        // index and the next step's stay in flight behind this one's tests
        auto load = [&](uint32_t k0, JLoad &f) __attribute__((always_inline)) {
            const uint32_t kk = k0 + (uint32_t)(lane / CS);
            f.j = kk < ncand ? s_cand[kk] * CS + (uint32_t)(lane % CS) : n;
            const uint32_t jc = f.j < n ? f.j : n - 1u;
            f.x = a.x[jc];
            f.y = a.y[jc];
            f.z = a.z[jc];
            f.h = a.h[jc];
        };
        if (ncand == 0) continue;
        JLoad nx;
        load(0, nx);
        for (uint32_t k0 = 0; k0 < ncand; k0 += kPerStep) {
            const JLoad f = nx;
            if (k0 + kPerStep < ncand) load(k0 + kPerStep, nx);
            const bool valid = f.j < n;
            const float hj2 = f.h * f.h;
            const uint32_t jr = f.j - i0;  // below kRows: our own particle jr
            uint32_t full = 0;  // rows with a segment pending
#pragma unroll
            for (int r = 0; r < kRows; r++) {
                float dx = f.x - xi[r];
                float dy = f.y - yi[r];
                float dz = f.z - zi[r];
                if (kPbc) wave_min_image(dx, dy, dz, a.per);
                const float dxx = dx * dx;
                const float d2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dxx));
                const bool in = (int)valid & (int)(d2 < fmaxf(hi2[r], hj2)) & (int)(jr != (uint32_t)r);
                const uint64_t b = sfc_ballot(in);
                if (in) s_pend[r][npend[r] + __builtin_amdgcn_mbcnt_hi((uint32_t)(b >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)b, 0u))] = f.j;
                npend[r] += (uint32_t)sfc_popc(b);
                full |= npend[r] >= (uint32_t)kWave ? 1u << r : 0u;
            }
            if (full) {
                wave_sync();
                for (uint32_t todo = full; todo; todo &= todo - 1u) {
                    const uint32_t r = (uint32_t)__builtin_ctz(todo);
                    flush(r, kWave);
                    s_pend[r][lane] = s_pend[r][kWave + lane];  // (a lane reads before any writes)
                    wave_sync();
                }
#pragma unroll
                for (int r = 0; r < kRows; r++) npend[r] -= ((full >> r) & 1u) * (uint32_t)kWave;
            }
        }
    }
    wave_sync();
#pragma unroll 1
    for (uint32_t r = 0; r < rows; r++) {
        uint32_t m = npend[0];
#pragma unroll
        for (int k = 1; k < kRows; k++) m = r == (uint32_t)k ? npend[k] : m;
        if (m) flush(r, m);
    }
    if ((uint32_t)lane < rows) {
        if (kWrite) {
            const bool ok = (fits >> lane) & 1u;
            a.row_info[2 * (size_t)(i0 + lane)] = st_off;
            a.row_info[2 * (size_t)(i0 + lane) + 1] = ok ? st_count : 0u;  // a row that did not fit is empty, reported
            if (!ok) atomicOr(&a.status[kStPoolOverflow], 1u);
        } else {
            a.row_words[i0 + lane] = st_words;
        }
    }
}

struct RowPassArgs {
    int64_t n;
    const uint32_t *row_info, *pool;
    const float *x, *y, *z, *h, *m;
    Period per;
    float *rho;
    int32_t *nnb;
};

// As decode_segment, from the words at w[p..] (LDS or memory); the last word
// read is the segment's last.
template <typename W>
__device__ __forceinline__ uint32_t decode_row_segment(W w, uint32_t &p, uint32_t cnt, uint32_t prevj) {
    const int lane = sfc_lane();
    const uint64_t m = ((uint64_t)w[p + 1] << 32) | w[p];
    const bool valid = (uint32_t)lane < cnt;
    const bool nonone = valid && ((m >> lane) & 1ull);
    const uint32_t ninfo = (uint32_t)sfc_popc(m);
    uint32_t v = 1u, nd = 0u;
    if (nonone) {
        const uint32_t t = (uint32_t)sfc_popc(m & sfc_lt_mask());
        const uint32_t inf = (w[p + 2 + (t >> 3)] >> (4u * (t & 7u))) & 0xFu;
        if (inf >= 8u)
            v = inf - 6u;
        else
            nd = inf + 1u;
    }
    const uint32_t incl = sfc_incl_scan(nd);
    if (nd) {  // its digits, the first in the low bits
        const uint32_t t = ninfo + incl - nd, sh = 4u * (t & 7u);
        uint64_t b = w[p + 2 + (t >> 3)];
        if ((t & 7u) + nd > 8u) b |= (uint64_t)w[p + 3 + (t >> 3)] << 32;
        v = digits_first((uint32_t)(b >> sh), 8u) >> (4u * (8u - nd));
    }
    const uint32_t total_nib = ninfo + sfc_readlane(incl, kWave - 1);
    p += 2u + (total_nib + 7u) / 8u;
    return prevj + sfc_incl_scan(valid ? v : 0u);
}

// Density and counts from the rows: the own-radius subset of each row.
template <bool kCompress, bool kMass, bool kCount, bool kPbc>
__global__ __launch_bounds__(kWave) void k_pass_rows(RowPassArgs a) {
    __shared__ uint32_t s_words[kCompress ? kStageWords : 1];
    const int lane = sfc_lane();
    const uint32_t n = (uint32_t)a.n;
    const uint32_t i = xcd_remap(blockIdx.x, gridDim.x);
    if (i >= n) return;
    const uint32_t off = a.row_info[2 * (size_t)i], cnt = a.row_info[2 * (size_t)i + 1];
    const float xi = a.x[i], yi = a.y[i], zi = a.z[i], hi = a.h[i];
    const float hi2 = hi * hi;
    const float hinv = 1.0f / hi;
    bool staged = false;
    if (kCompress && i + 1 < n) {  // the next row begins where this one ends
        const uint32_t len = row_stage_words(off, cnt, a.row_info[2 * (size_t)i + 2]);
        staged = len != 0u;
        if (staged) {
            for (uint32_t q = (uint32_t)lane; q < len; q += kWave) s_words[q] = a.pool[off + q];
            wave_sync();
        }
    }
    uint32_t p = staged ? 0u : off;
    uint32_t prevj = 0xFFFFFFFFu;
    float acc = 0.0f;
    uint32_t nb = 0;
    struct Step {
        float x, y, z, m;
    };
    // decodes neighbours b0 .. and loads their particles (lanes past the end:
    // the row's own particle)
    auto next = [&](uint32_t b0, Step &f) __attribute__((always_inline)) {
        const uint32_t c = cnt - b0 < (uint32_t)kWave ? cnt - b0 : (uint32_t)kWave;
        uint32_t jv;
        if (!kCompress) {
            jv = (uint32_t)lane < c ? a.pool[off + b0 + lane] : 0u;
        } else {
            jv = staged ? decode_row_segment((const uint32_t *)s_words, p, c, prevj)
                        : decode_row_segment(a.pool, p, c, prevj);
            prevj = sfc_readlane(jv, (int)c - 1);
        }
        const uint32_t jc = (uint32_t)lane < c ? jv : i;
        f.x = a.x[jc];
        f.y = a.y[jc];
        f.z = a.z[jc];
        f.m = kMass ? a.m[jc] : 1.0f;
    };
    Step nx;
    if (cnt) next(0, nx);
    for (uint32_t b0 = 0; b0 < cnt; b0 += kWave) {
        const Step f = nx;
        if (b0 + kWave < cnt) next(b0 + kWave, nx);
        float dx = f.x - xi;
        float dy = f.y - yi;
        float dz = f.z - zi;
        if (kPbc) wave_min_image(dx, dy, dz, a.per);
        const float dxx = dx * dx;
        const float d2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dxx));
        const bool in = (int)(b0 + (uint32_t)lane < cnt) & (int)(d2 < hi2);
        nb += (uint32_t)sfc_popc(sfc_ballot(in));
        const float q = __builtin_amdgcn_sqrtf(d2) * hinv;
        const float t1 = q - 1.0f;
        const float q2 = q * q;
        const float inner = __builtin_fmaf(3.0f * q2, t1, 0.5f);
        const float outer = -(t1 * t1) * t1;
        const float wq = q < 0.5f ? inner : outer;
        acc = in ? __builtin_fmaf(kMass ? f.m : 1.0f, wq, acc) : acc;
    }
    acc = sfc_wave_reduce(acc, [](float u, float v) { return u + v; });
    if (lane == 0) {
        const float norm = 2.5464790894703255f * hinv * hinv * hinv;  // 8 / pi
        a.rho[i] = norm * __builtin_fmaf(2.0f, acc, kMass ? a.m[i] : 1.0f);
        if (kCount) a.nnb[i] = (int32_t)nb;
    }
}

template <int CS, int kRows, bool kWrite, bool kPbc>
void launch_rows(bool comp_in, hipStream_t st, const RowArgs &a) {
    const unsigned g = blocks_for(a.n, kRows);
    if (comp_in)
        k_rows<CS, kRows, true, kWrite, kPbc><<<g, kWave, 0, st>>>(a);
    else
        k_rows<CS, kRows, false, kWrite, kPbc><<<g, kWave, 0, st>>>(a);
}

template <int kRows, bool kWrite, bool kPbc>
void launch_rows_cs(int cs, bool comp_in, hipStream_t st, const RowArgs &a) {
    if (cs == 4)
        launch_rows<4, kRows, kWrite, kPbc>(comp_in, st, a);
    else if (cs == 16)
        launch_rows<16, kRows, kWrite, kPbc>(comp_in, st, a);
    else
        launch_rows<8, kRows, kWrite, kPbc>(comp_in, st, a);
}

template <bool kWrite>
void launch_rows_any(int cs, bool comp_in, hipStream_t st, const RowArgs &a) {
    const bool pbc = a.per.on();
    if (a.n >= kRows8Min) {
        if (pbc) launch_rows_cs<8, kWrite, true>(cs, comp_in, st, a);
        else launch_rows_cs<8, kWrite, false>(cs, comp_in, st, a);
    } else if (a.n >= kRows4Min) {
        if (pbc) launch_rows_cs<4, kWrite, true>(cs, comp_in, st, a);
        else launch_rows_cs<4, kWrite, false>(cs, comp_in, st, a);
    } else {
        if (pbc) launch_rows_cs<1, kWrite, true>(cs, comp_in, st, a);
        else launch_rows_cs<1, kWrite, false>(cs, comp_in, st, a);
    }
}

template <bool kPbc>
void launch_pass_rows(int variant, unsigned g, hipStream_t st, const RowPassArgs &a) {
    switch (variant) {
        case 7: k_pass_rows<true, true, true, kPbc><<<g, kWave, 0, st>>>(a); break;
        case 6: k_pass_rows<true, true, false, kPbc><<<g, kWave, 0, st>>>(a); break;
        case 5: k_pass_rows<true, false, true, kPbc><<<g, kWave, 0, st>>>(a); break;
        case 4: k_pass_rows<true, false, false, kPbc><<<g, kWave, 0, st>>>(a); break;
        case 3: k_pass_rows<false, true, true, kPbc><<<g, kWave, 0, st>>>(a); break;
        case 2: k_pass_rows<false, true, false, kPbc><<<g, kWave, 0, st>>>(a); break;
        case 1: k_pass_rows<false, false, true, kPbc><<<g, kWave, 0, st>>>(a); break;
        default: k_pass_rows<false, false, false, kPbc><<<g, kWave, 0, st>>>(a); break;
    }
}

__global__ void k_rows_total(const uint32_t *total, uint32_t *status) { status[kStTotalLo] = *total; }

struct RowsWs {
    uint32_t *row_words, *row_off;
    void *scan_tmp;
};

size_t carve_rows(RowsWs &ws, void *base, int64_t n) {
    Carver cv{reinterpret_cast<char *>(base), 0};
    ws.row_words = cv.take<uint32_t>((size_t)n);
    ws.row_off = cv.take<uint32_t>((size_t)n + 1);
    ws.scan_tmp = cv.take<char>(scan_tmp_bytes(n));
    return cv.used;
}

}  // namespace
}  // namespace sfcnl

using namespace sfcnl;

extern "C" int build_rows_workspace(int64_t n, size_t *ws_bytes) {
    if (n < 0 || n >= (int64_t(1) << 31) || !ws_bytes) return SFCNL_E_ARG;
    RowsWs ws;
    *ws_bytes = align_up(carve_rows(ws, nullptr, n), 256) + 256;
    return SFCNL_OK;
}

extern "C" int build_rows(sfcnl_ctx ctx, int64_t n, int cluster_size, int list_compress, const uint32_t *d_sc_info,
                          const uint32_t *d_pool, const float *d_x, const float *d_y, const float *d_z,
                          const float *d_h, int compress, const float *h_period, void *d_ws, size_t ws_bytes,
                          uint32_t *d_row_info, uint32_t *d_row_pool, size_t pool_bytes, size_t *h_used_bytes) {
    if (!ctx) return SFCNL_E_ARG;
    if (n < 0 || n >= (int64_t(1) << 31)) return set_err(ctx, SFCNL_E_ARG, "build_rows: n out of range");
    if (cluster_size != 4 && cluster_size != 8 && cluster_size != 16)
        return set_err(ctx, SFCNL_E_ARG, "build_rows: cluster_size %d not supported", cluster_size);
    if ((list_compress != 0 && list_compress != 1) || (compress != 0 && compress != 1))
        return set_err(ctx, SFCNL_E_ARG, "build_rows: compress flags must be 0 or 1");
    if (!period_ok(h_period)) return set_err(ctx, SFCNL_E_ARG, "build_rows: period must be 3 finite values >= 0");
    if (!h_used_bytes) return set_err(ctx, SFCNL_E_ARG, "build_rows: null result pointer");
    *h_used_bytes = 0;
    if (n == 0) return SFCNL_OK;
    if (!d_sc_info || !d_pool || !d_x || !d_y || !d_z || !d_h || !d_ws || !d_row_info || (!d_row_pool && pool_bytes))
        return set_err(ctx, SFCNL_E_ARG, "build_rows: null pointer");
    RowsWs ws;
    const size_t need = carve_rows(ws, d_ws, n);
    if (need > ws_bytes) return set_err(ctx, SFCNL_E_ARG, "build_rows: workspace %zu < %zu bytes", ws_bytes, need);
    const Period per = make_period(h_period);
    RowArgs a{n, d_sc_info, d_pool, d_x, d_y, d_z, d_h, per, compress, ws.row_words, ws.row_off, d_row_info,
              d_row_pool, pool_bytes / 4, ctx->d_status};
    hipStream_t st = ctx->stream;
    int rc = fill_u32(ctx, ctx->d_status + kStPoolOverflow, 1, 0u);
    if (rc) return rc;
    launch_rows_any<false>(cluster_size, list_compress, st, a);
    SFCNL_LAUNCHED(ctx);
    rc = scan_u32(ctx, ws.row_words, ws.row_off, n, ws.row_off + n, ws.scan_tmp);
    if (rc) return rc;
    launch_rows_any<true>(cluster_size, list_compress, st, a);
    SFCNL_LAUNCHED(ctx);
    k_rows_total<<<1, 1, 0, st>>>(ws.row_off + n, ctx->d_status);
    SFCNL_LAUNCHED(ctx);
    rc = read_status(ctx);
    if (rc) return rc;
    *h_used_bytes = (size_t)ctx->h_status[kStTotalLo] * 4;
    if (ctx->h_status[kStPoolOverflow])
        return set_err(ctx, SFCNL_E_CAPACITY, "build_rows: pool of %zu bytes < %zu needed", pool_bytes, *h_used_bytes);
    return SFCNL_OK;
}

extern "C" int rows_pass(sfcnl_ctx ctx, int64_t n, int compress, const uint32_t *d_row_info,
                         const uint32_t *d_row_pool, const float *d_x, const float *d_y, const float *d_z,
                         const float *d_h, const float *d_m, float *d_rho, int32_t *d_nnb, const float *h_period) {
    if (!ctx) return SFCNL_E_ARG;
    if (n < 0 || n >= (int64_t(1) << 31)) return set_err(ctx, SFCNL_E_ARG, "rows_pass: n out of range");
    if (compress != 0 && compress != 1) return set_err(ctx, SFCNL_E_ARG, "rows_pass: compress must be 0 or 1");
    if (!period_ok(h_period)) return set_err(ctx, SFCNL_E_ARG, "rows_pass: period must be 3 finite values >= 0");
    if (n == 0) return SFCNL_OK;
    if (!d_row_info || !d_row_pool || !d_x || !d_y || !d_z || !d_h || !d_rho)
        return set_err(ctx, SFCNL_E_ARG, "rows_pass: null pointer");
    RowPassArgs a{n, d_row_info, d_row_pool, d_x, d_y, d_z, d_h, d_m, make_period(h_period), d_rho, d_nnb};
    const int variant = (compress ? 4 : 0) | (d_m ? 2 : 0) | (d_nnb ? 1 : 0);
    prof_mark(ctx, kStagePass, false);
    const unsigned g = blocks_for(n, 1);
    if (a.per.on())
        launch_pass_rows<true>(variant, g, ctx->stream, a);
    else
        launch_pass_rows<false>(variant, g, ctx->stream, a);
    SFCNL_LAUNCHED(ctx);
    prof_mark(ctx, kStagePass, true);
    return SFCNL_OK;
}
