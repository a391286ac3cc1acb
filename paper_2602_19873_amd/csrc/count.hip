// The remaining rounds of an h-iteration once few particles still move,
// without a list. A particle's own-radius count depends on its radius alone,
// so its rounds are independent of every other particle's: one wavefront takes
// a particle and repeats count and update until the count is within the
// tolerance or the rounds are over. A count walks the octree of the last full
// build (positions and key ranges are unchanged) with a sphere a little wider
// than the radius, pushing the children whose boxes come within it, and at a
// leaf tests the leaf's particles 64 at a time with the exact FP32 pair
// formula; the squared distances found stay in LDS, where the later rounds,
// whose radii rarely leave that sphere, count from. Counts are exact;
// densities are the sums of the pass in another order.
//
// Bound by the latency of the walk (a chain of dependent box and particle
// loads). A list round or a recount of all moved particles per round walks
// again for each of some 10 (one sphere) to 40 rounds (16 systems), and from
// the tenth round on a round was 90 to 120 us of launches around a few us of
// work: for the whole iteration 1,000,003 particles of a 1/r sphere 4.74 ->
// 3.51 ms, 20,000 1.68 -> 0.82 ms, four systems of up to 100,000 17.2 -> 6.3 ms
// (3.18, 0.44 and 3.3 ms with what came after: shared counters by stripes,
// incomplete counts and lists without an octree).
#include <algorithm>
#include <type_traits>

#include "internal.h"

namespace sfcnl {
namespace {

constexpr int kWavesPerBlock = 4;
constexpr int kStackCap = 160;  // 1 + 7 * 21 pushes at most

__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Half the M4 spline's shape at a pair inside the radius.
__device__ __forceinline__ float spline_half(float d2, float hinv) {
    const float q = __builtin_amdgcn_sqrtf(d2) * hinv;
    const float t1 = q - 1.0f;
    const float q2 = q * q;
    const float inner = __builtin_fmaf(3.0f * q2, t1, 0.5f);
    const float outer = -(t1 * t1) * t1;
    return q < 0.5f ? inner : outer;
}

// Writes the moved particles of super-cluster s to plist[off[s] + rank] and
// clears the outcome words of the finish.
__global__ __launch_bounds__(256) void k_compact_moved(int64_t n, const uint32_t *__restrict__ cnt,
                                                       const uint32_t *__restrict__ off,
                                                       const uint8_t *__restrict__ moved, uint32_t *__restrict__ plist,
                                                       uint32_t *status) {
    const int lane = sfc_lane();
    const uint32_t s = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * kWavesPerBlock + threadIdx.x / kWave));
    const uint32_t nsc = (uint32_t)((n + kScSize - 1) / kScSize);
    if (s == 0 && lane >= kStFinMoved && lane <= kStFinLeft) status[lane] = 0u;
    if (s == 0 && lane < kChunkStripes) status[kStWords + lane * kStripeWords + kStripeFin] = 0u;
    if (s >= nsc || cnt[s] == 0) return;
    const int64_t i = (int64_t)s * kScSize + lane;
    const bool f = i < n && moved[i] != 0;
    const uint64_t b = sfc_ballot(f);
    if (f) plist[off[s] + (uint32_t)sfc_popc(b & sfc_lt_mask())] = (uint32_t)i;
}

struct FinishArgs {
    int64_t n;
    const uint32_t *plist;
    const uint32_t *total;  // listed particles (device word)
    const float *x, *y, *z, *m;
    float *h;
    float2 *br;
    const float4 *cs_box;   // octree child slots (slot 0 = root)
    const uint4 *cs_rec;
    uint32_t nslots;
    int target, tol, rounds;
    uint32_t plenty;  // count that halves a radius (h_plenty)
    SegTable seg;
    Period per;
    float *rho;
    int32_t *nnb;
    uint32_t *status, *sys_rounds;
};

// One wavefront per listed particle, taken from the list as waves become free
// (some particles need two rounds, some forty): list position k 64 + s belongs
// to stripe s, whose waves share a counter (one counter for all, an atomic that
// returns a value per particle, cost 0.5 ms: iteration of 65,536 particles, all
// of them here, 1290 -> 714 us).
template <bool kMass, bool kPbc>
__global__ __launch_bounds__(256) void k_finish_moved(FinishArgs a) {
    __shared__ uint4 s_stack[kWavesPerBlock][kStackCap];
    __shared__ float s_d2[kWavesPerBlock][kKept];
    __shared__ uint32_t s_j[kWavesPerBlock][kMass ? kKept : 1];
    const int lane = sfc_lane();
    const int w = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    const uint32_t total = *a.total;
    const uint32_t nw = gridDim.x * kWavesPerBlock;
    uint4 *stack = s_stack[w];
    float *d2s = s_d2[w];
    uint32_t *js = s_j[w];
    uint32_t t = blockIdx.x * kWavesPerBlock + (uint32_t)w;
    const uint32_t stripe = t % kChunkStripes, members = (nw - stripe + kChunkStripes - 1) / kChunkStripes;
    uint32_t moves = 0, most = 0, left = 0;
    while (t < total) {
        const uint32_t i = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.plist[t]);
        const float xi = a.x[i], yi = a.y[i], zi = a.z[i];
        float hi = a.h[i];
        float2 b = a.br[i];
        const int sy = a.seg.on() ? a.seg.sc_sys[i / kScSize] : 0;
        const uint4 root = a.seg.on() ? a.seg.roots[sy] : a.cs_rec[0];
        float acc = 0.0f;       // m_j times the halved spline shape, summed
        uint32_t kept = 0;      // pairs in d2s: those within kept_r2
        float kept_r2 = -1.0f;
        // Pairs within h2 (returned); with kept_r2 >= 0 also into d2s those
        // within kept_r2, which becomes -1 if they are more than it holds;
        // kAcc: adds the pairs within h2 to acc instead.
        // A walk ends early at a count of `plenty`.
        auto walk = [&](float h2, float hinv, uint32_t plenty, auto acc_c) __attribute__((always_inline)) -> uint32_t {
            constexpr bool kAcc = decltype(acc_c)::value;
            const float r2 = kAcc ? h2 : fmaxf(h2, kept_r2);
            uint32_t cnt = 0;
            kept = kAcc ? kept : 0u;
            wave_sync();  // the last reads of the stack and the kept pairs are done
            if (lane == 0) stack[0] = root;
            int sp = 1;
            wave_sync();
            while (sp > 0 && cnt < plenty) {
                sp--;
                const uint4 rv = stack[sp];
                const uint32_t nfirst = (uint32_t)__builtin_amdgcn_readfirstlane((int)rv.x);
                const uint32_t nend = (uint32_t)__builtin_amdgcn_readfirstlane((int)rv.y);
                const uint32_t nchild = (uint32_t)__builtin_amdgcn_readfirstlane((int)rv.z);
                const uint32_t cslot = (uint32_t)__builtin_amdgcn_readfirstlane((int)rv.w);
                if (nend > (uint64_t)a.n || nfirst >= nend || cslot + nchild > a.nslots) {  // only on a broken tree
                    if (lane == 0) atomicOr(&a.status[kStTree], 16u);
                    break;
                }
                if (nchild == 0) {
                    for (uint32_t p0 = nfirst; p0 < nend; p0 += kWave) {
                        const uint32_t j = p0 + (uint32_t)lane;
                        const bool v = j < nend;
                        const uint32_t jc = v ? j : nfirst;
                        float dx = a.x[jc] - xi;
                        float dy = a.y[jc] - yi;
                        float dz = a.z[jc] - zi;
                        if (kPbc) wave_min_image(dx, dy, dz, a.per);
                        const float dxx = dx * dx;
                        const float d2 = __builtin_fmaf(dz, dz, __builtin_fmaf(dy, dy, dxx));
                        const bool other = v && j != i;
                        const bool in = other && d2 < h2;
                        cnt += (uint32_t)sfc_popc(sfc_ballot(in));
                        if (kAcc) {
                            const float mj = kMass ? (in ? a.m[jc] : 0.0f) : 1.0f;
                            if (in) acc = __builtin_fmaf(mj, spline_half(d2, hinv), acc);
                        } else {
                            const bool near = other && d2 < kept_r2;
                            const uint64_t bal = sfc_ballot(near);
                            if (bal) {
                                const uint32_t to = kept + (uint32_t)sfc_popc(bal & sfc_lt_mask());
                                if (near && to < (uint32_t)kKept) {
                                    d2s[to] = d2;
                                    if (kMass) js[to] = j;
                                }
                                kept += (uint32_t)sfc_popc(bal);
                            }
                        }
                    }
                } else {
                    // lane jl < nchild tests child jl against the sphere
                    const int jl = lane;
                    bool hit = false;
                    uint4 crec = make_uint4(0u, 0u, 0u, 0u);
                    if (jl < (int)nchild) {
                        const uint32_t slot = cslot + (uint32_t)jl;
                        const float4 lo = a.cs_box[2 * (size_t)slot], hb = a.cs_box[2 * (size_t)slot + 1];
                        crec = a.cs_rec[slot];
                        const float gx = axis_gap<kPbc>(lo.x - xi, xi - hb.x, a.per.L[0]);
                        const float gy = axis_gap<kPbc>(lo.y - yi, yi - hb.y, a.per.L[1]);
                        const float gz = axis_gap<kPbc>(lo.z - zi, zi - hb.z, a.per.L[2]);
                        const float gxx = gx * gx;
                        hit = __builtin_fmaf(gz, gz, __builtin_fmaf(gy, gy, gxx)) < r2;
                    }
                    const uint64_t keep = sfc_ballot(hit);
                    const int c = sfc_popc(keep);
                    if (sp + c > kStackCap) {  // cannot happen in a valid octree (depth <= 21)
                        if (lane == 0) atomicOr(&a.status[kStTree], 8u);
                        break;
                    }
                    if (hit) stack[sp + sfc_popc(keep & sfc_lt_mask())] = crec;
                    sp += c;
                    wave_sync();
                }
            }
            if (!kAcc && (kept > (uint32_t)kKept || cnt >= plenty)) kept_r2 = -1.0f;
            wave_sync();
            return cnt;
        };
        uint32_t cnt, r = 0, my_moves = 0;
        float hc;  // the counted radius
        for (;;) {
            hc = hi;
            const float h2 = hc * hc;
            if (h2 <= kept_r2) {  // (kept_r2 = -1: nothing kept)
                cnt = 0;
                for (uint32_t k0 = 0; k0 < kept; k0 += kWave) {
                    const uint32_t k = k0 + (uint32_t)lane;
                    cnt += (uint32_t)sfc_popc(sfc_ballot(k < kept && d2s[k < kept ? k : 0u] < h2));
                }
            } else {
                // no later radius reaches the bracket's upper end
                const float reach = fmaxf(fminf(kReach * hc, b.y), hc);
                kept_r2 = reach * reach;
                // (a count of `plenty` halves the radius whatever it is, so only
                // the last round needs it)
                cnt = walk(h2, 0.0f, r + 1 < (uint32_t)a.rounds ? a.plenty : 0xFFFFFFFFu, std::false_type{});
            }
            const int dev = (int)cnt - a.target;
            if (!(dev > a.tol || dev < -a.tol)) break;
            hi = h_step(hc, (int)cnt, dev, a.target, NAN, b);
            my_moves++;
            r++;
            if (r == (uint32_t)a.rounds) {
                left++;
                break;
            }
        }
        const float hinv = 1.0f / hc;
        if (hc * hc <= kept_r2) {
            for (uint32_t k = (uint32_t)lane; k < kept; k += kWave) {
                const float d2 = d2s[k];
                if (d2 < hc * hc) acc = __builtin_fmaf(kMass ? a.m[js[k]] : 1.0f, spline_half(d2, hinv), acc);
            }
        } else {
            walk(hc * hc, hinv, 0xFFFFFFFFu, std::true_type{});
        }
        acc = sfc_wave_reduce(acc, [](float p, float q) { return p + q; });
        if (lane == 0) {
            const float norm = 2.5464790894703255f * hinv * hinv * hinv;  // 8 / pi
            a.rho[i] = norm * __builtin_fmaf(2.0f, acc, kMass ? a.m[i] : 1.0f);
            a.nnb[i] = (int32_t)cnt;
            a.h[i] = hi;
            a.br[i] = b;
            if (my_moves && a.sys_rounds) atomicMax(&a.sys_rounds[sy], r);
        }
        moves += my_moves;
        most = r > most ? r : most;
        uint32_t next = 0;
        if (lane == 0) next = atomicAdd(&a.status[kStWords + stripe * kStripeWords + kStripeFin], 1u);
        t = (members + (uint32_t)__builtin_amdgcn_readfirstlane((int)next)) * kChunkStripes + stripe;
    }
    if (lane == 0 && most) {
        atomicAdd(reinterpret_cast<unsigned long long *>(&a.status[kStFinMoved]), (unsigned long long)moves);
        atomicMax(&a.status[kStFinRounds], most);
        if (left) atomicAdd(&a.status[kStFinLeft], left);
    }
}

}  // namespace
}  // namespace sfcnl

using namespace sfcnl;

int sfcnl::finish_moved_impl(sfcnl_ctx ctx, int64_t n, const ActiveWs &act, const float *x, const float *y,
                             const float *z, float *h, float2 *br, const float *m, float *rho, int32_t *nnb, int target,
                             int tol, int rounds, const SegTable &seg, const Period &per, uint32_t *sys_rounds,
                             int64_t moved) {
    if (n == 0) return SFCNL_OK;
    const uint32_t nsc = (uint32_t)((n + kScSize - 1) / kScSize);
    hipStream_t st = ctx->stream;
    prof_mark(ctx, kStagePass, false);
    k_compact_moved<<<blocks_for(nsc, kWavesPerBlock), 256, 0, st>>>(n, act.sc, act.scan, act.p, act.plist, ctx->d_status);
    SFCNL_LAUNCHED(ctx);
    FinishArgs a{n, act.plist, act.scan + nsc, x, y, z, m, h, br, act.cs_box, act.cs_rec, act.nslots, target, tol, rounds,
                 h_plenty(target, tol), seg, per, rho, nnb, ctx->d_status, sys_rounds};
    // as many wavefronts as the GPU holds
    const unsigned g = (unsigned)std::min<int64_t>(blocks_for(moved, kWavesPerBlock), 2048);
    if (per.on()) {
        if (m)
            k_finish_moved<true, true><<<g, 256, 0, st>>>(a);
        else
            k_finish_moved<false, true><<<g, 256, 0, st>>>(a);
    } else {
        if (m)
            k_finish_moved<true, false><<<g, 256, 0, st>>>(a);
        else
            k_finish_moved<false, false><<<g, 256, 0, st>>>(a);
    }
    SFCNL_LAUNCHED(ctx);
    prof_mark(ctx, kStagePass, true);
    return SFCNL_OK;
}
