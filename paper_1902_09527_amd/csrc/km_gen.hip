// Incremental MTI steps for any row width: the paper's skipping of the data
// of the points Clause 1 keeps (section III-C: no row of such a point is
// read) where the streaming path (d = 16, k <= 16) does not apply.  Two kernels share the
// structure; which one runs is a rule on d and k (gen_kind):
//   k_inc_vec  d <= 16 and few centroids: one lane per survivor, its row in
//              registers, the MTI scan of the vector path (tighten, Clauses 2
//              and 3 with the running best, direct-form distances);
//   k_inc_mat  otherwise: 32 survivors per wave against blocks of 32
//              centroids on the matrix cores.
//
// Point state: one 32-bit word per point, the cluster in the low bits (7, or
// 8 for k > 128) and in the rest a float32 value v (rounded up) with v + D_a
// an upper bound on the point's distance to its centroid, D_a the cumulative
// drift of its cluster.  A point that Clause 1 keeps costs the read of its
// word; nothing of it is written and its row is not read.
//
// Per wave: tiles of kGenTile points from a block counter; Clause 1 on every
// word; survivors queued in LDS and settled a full batch at a time.  The rows
// of the points whose cluster changed are moved between the block's exact
// fixed-point sums by lanes that share a row (coalesced, the row just read is
// in cache).  At the end a block adds the words it changed to one of
// kGenRows accumulation rows by device atomics; k_update adds those rows to
// the running sums and clears them.
#include <float.h>
#include <limits.h>
#include <stddef.h>
#include <math.h>

#include "kmeans_mti.h"
#include "km_device.h"
#include "km_internal.h"

namespace km {

extern __shared__ __align__(16) unsigned char km_smem[];

namespace {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4u __attribute__((ext_vector_type(4), aligned(4)));   // a 16-byte load from a 4-byte aligned address

// State word with CB cluster bits: v rounded up to a multiple of 2^CB units
// in the last place (for v >= 0 the bit pattern grows, for v < 0 the
// magnitude shrinks).
template <int CB>
__device__ __forceinline__ uint32_t pack_state(float v, int a) {
    constexpr uint32_t M = (1u << CB) - 1u;
    uint32_t b = __float_as_uint(v);
    if (!(b >> 31)) b += M;
    return (b & ~M) | (uint32_t)a;
}
template <int CB>
__device__ __forceinline__ int state_cluster(uint32_t w) { return (int)(w & ((1u << CB) - 1u)); }
template <int CB>
__device__ __forceinline__ float state_value(uint32_t w) { return __uint_as_float(w & ~((1u << CB) - 1u)); }

// v = ub - D_b rounded up.
template <int CB>
__device__ __forceinline__ uint32_t state_of(float ub, float ddn, int b) {
    const float rr = ub - ddn;
    return pack_state<CB>(rr + fabsf(rr) * 0x1p-22f, b);
}

// Whether a launch has nothing to do: the run has stopped (the step is marked
// as not running), or the other form of a recorded first step runs.  One load.
__device__ __forceinline__ bool step_idle(IterState* st, int first, int check) {
    static_assert(offsetof(IterState, done) == offsetof(IterState, t) + 4, "t and done are one load");
    const int2 td = *reinterpret_cast<const int2*>(&st->t);
    const int other = check & ((td.x == 0 ? 1 : 0) ^ first);
    if (!(td.y | other)) return false;
    if (td.y && blockIdx.x == 0 && threadIdx.x == 0) st->active = 0;
    return true;
}

// LDS ordering point inside one wave.
__device__ __forceinline__ void wave_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The listed moves of a wave (entry: point, new cluster in the low and old
// cluster + 1 in the high half; 0 = none): LPR lanes share a row (LPR the
// smallest power of two >= d, at most 64), so the row is read coalesced and
// the LDS atomics of a row fall on distinct banks.
__device__ __forceinline__ void apply_moves(const uint2* ml, int n, const float* __restrict__ X, int d, int AR,
                                            double qscale, uint64_t* acc, int* cnt) {
    const int lane = threadIdx.x & 63;
    const int lg = d > 32 ? 6 : d > 16 ? 5 : d > 8 ? 4 : d > 4 ? 3 : d > 2 ? 2 : d > 1 ? 1 : 0;
    const int m0 = lane & ((1 << lg) - 1), g = lane >> lg, rpp = 64 >> lg;
    constexpr int U = 4;   // rows in flight per lane
    for (int e0 = 0; e0 < n; e0 += U * rpp) {
        uint2 e[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int i = e0 + u * rpp + g;
            e[u] = ml[i < n ? i : 0];
            if (i >= n) e[u].y = 0xffffffffu;
        }
        for (int m = m0; m < d; m += 64) {
            float x[U];
#pragma unroll
            for (int u = 0; u < U; ++u) x[u] = X[(int64_t)e[u].x * d + m];
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (e[u].y == 0xffffffffu) continue;
                const uint64_t v = fixed_bits((double)x[u], qscale);
                const int b = (int)(e[u].y & 0xffffu), o = (int)(e[u].y >> 16) - 1;
                atomicAdd(reinterpret_cast<unsigned long long*>(acc + b * AR + m), (unsigned long long)v);
                if (o >= 0) lds_sub64(acc + o * AR + m, v);
            }
        }
        if (m0 == 0) {
#pragma unroll
            for (int u = 0; u < U; ++u) {
                if (e[u].y == 0xffffffffu) continue;
                const int b = (int)(e[u].y & 0xffffu), o = (int)(e[u].y >> 16) - 1;
                atomicAdd(&cnt[b], 1);
                if (o >= 0) atomicAdd(&cnt[o], -1);
            }
        }
    }
}

// The words of the block's sums that its moves changed, its member counts
// and counters, added to its accumulation row.
__device__ __forceinline__ void flush_block(const Dev& P, const uint64_t* acc, const int* cnt, const uint64_t* bst,
                                            int AR, int nt) {
    const int k = P.k, d = P.d, tid = threadIdx.x;
    unsigned long long* row =
        reinterpret_cast<unsigned long long*>(P.rows + (int64_t)(blockIdx.x % kGenRows) * P.L);
    for (int j = tid / 64; j < k; j += nt / 64)   // a wave per cluster row
        for (int m = tid & 63; m < d; m += 64) {
            const uint64_t v = acc[j * AR + m];
            if (v) atomicAdd(row + (int64_t)j * d + m, (unsigned long long)v);
        }
    for (int j = tid; j < k; j += nt)
        if (cnt[j]) atomicAdd(row + (int64_t)k * d + j, (unsigned long long)(int64_t)cnt[j]);
    if (tid < kNumStat && bst[tid]) atomicAdd(row + (int64_t)k * d + k + tid, (unsigned long long)bst[tid]);
}

}  // namespace

// ---------------------------------------------------------------------------
// One lane per survivor (d <= DP <= 16, k <= kGenVecMaxK).
//
// Bound by vector instructions: about 2 DP + 8 per survivor and centroid (64
// survivors at a time).  Four centroids are formed side by side, since one
// after another each waited for the bound and the table entry of the one
// before.  The general kernel, which it replaces here, read and summed every
// row in every step: 66M x 8, k = 10 took 3.27 ms a step and takes 0.59 ms
// (the survivors' lines and the states are 0.5 ms at 4.8 TB/s).

template <int DP>
__global__ __launch_bounds__(kGenThreads) void k_inc_vec(Dev P_, int first, int check, int nsub) {
    const Dev P = with_scales(P_);
    IterState* st = P.st;
    if (step_idle(st, first, check)) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) st->active = 1;
    const int k = P.k, d = P.d, tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const float ecmax = st->ec_max, gamma = P.gamma;
    const GenVecLds lay = gen_vec_lds(DP, d, k);
    const int AR = lay.ar;
    float* Cs = reinterpret_cast<float*>(km_smem + lay.off_c);
    float* hl = reinterpret_cast<float*>(km_smem + lay.off_h);
    float* thr = reinterpret_cast<float*>(km_smem + lay.off_thr);
    float* ss = reinterpret_cast<float*>(km_smem + lay.off_s);
    float* ecs = reinterpret_cast<float*>(km_smem + lay.off_ec);
    float* ddn = reinterpret_cast<float*>(km_smem + lay.off_ddn);
    uint64_t* acc = reinterpret_cast<uint64_t*>(km_smem + lay.off_acc);
    int* cnt = reinterpret_cast<int*>(km_smem + lay.off_cnt);
    int* tcount = reinterpret_cast<int*>(km_smem + lay.off_misc);
    uint64_t* bst = reinterpret_cast<uint64_t*>(km_smem + lay.off_misc + 16);
    uint2* q = reinterpret_cast<uint2*>(km_smem + lay.off_q) + w * kGenVecQ;
    uint2* ml = reinterpret_cast<uint2*>(km_smem + lay.off_m) + w * 64;

    const int KS = (k + 3) / 4 * 4;   // row stride of the half-distance table: 16-byte rows
    for (int i = tid; i < KS * DP; i += kGenThreads) {
        const int j = i / DP, m = i % DP;
        Cs[i] = j < k && m < d ? P.C32[j * d + m] : 0.f;
    }
    for (int i = tid; i < k * KS; i += kGenThreads) {
        const int r = i / KS, c = i - r * KS;
        hl[i] = c < k ? P.h[r * k + c] : 0.f;
    }
    for (int i = tid; i < k * AR; i += kGenThreads) acc[i] = 0;
    for (int i = tid; i < k; i += kGenThreads) {
        ss[i] = P.s[i];
        thr[i] = first ? 0.f : clause1_thr(P.s[i], P.dhi[i]);
        ecs[i] = P.ec[i];
        ddn[i] = P.ddnf[i];
        cnt[i] = 0;
    }
    if (tid < kNumStat) bst[tid] = 0;
    if (tid == 0) *tcount = 0;
    __syncthreads();

    uint32_t my_changed = 0, my_comp = 0, my_rc = 0, c1w = 0;
    const float gup = (1.0f + gamma) * (1.0f + 0x1p-20f) * kUp;

    // Settles up to 64 survivors, one per lane.
    auto settle = [&](int p, uint32_t ws, bool live) __attribute__((always_inline)) {
        const float* xr = P.X + (int64_t)p * d;
        float x[DP];
#pragma unroll
        for (int m = 0; m < DP; m += 4) {
            if (m + 4 <= d) {   // uniform
                const f32x4u v = *reinterpret_cast<const f32x4u*>(xr + m);
                x[m] = v.x;
                x[m + 1] = v.y;
                x[m + 2] = v.z;
                x[m + 3] = v.w;
            } else {
#pragma unroll
                for (int e = 0; e < 4; ++e) x[m + e] = m + e < d ? xr[m + e] : 0.f;
            }
        }
        auto dist = [&](int j) __attribute__((always_inline)) {
            const float* c = Cs + j * DP;
            float a = 0.f;
#pragma unroll
            for (int m = 0; m < DP; m += 4) {
                const f32x4 cv = *reinterpret_cast<const f32x4*>(c + m);
                const float t0 = x[m] - cv.x, t1 = x[m + 1] - cv.y, t2 = x[m + 2] - cv.z, t3 = x[m + 3] - cv.w;
                a = fmaf(t0, t0, a);
                a = fmaf(t1, t1, a);
                a = fmaf(t2, t2, a);
                a = fmaf(t3, t3, a);
            }
            return a;
        };
        // upper_bound with the hardware square root (2^-20 covers its error).
        auto bound = [&](float D, float ec) __attribute__((always_inline)) {
            return (__builtin_amdgcn_sqrtf(D) * gup + ec) * kUp;
        };
        const int inc = first ? -1 : state_cluster<7>(ws);
        int b = -1;
        float Db = INFINITY, D2 = INFINITY, ub = 0.f;
        uint32_t nc = 0;
        bool scan = live;
        if (!first) {   // tighten: distance to the incumbent (U(u)); within s(a) all others are skipped
            Db = dist(inc);
            b = inc;
            nc = 1;
            ub = bound(Db, ecs[inc]);
            scan = live && ub > ss[inc];
        }
        if (scan) {
            // The MTI scan in ascending order with the running best, four
            // centroids at a time: their distances are formed side by side
            // (independent chains), then taken one after another by the same
            // tests as one at a time; four that every lane skips cost only
            // the tests.
            for (int j0 = 0; j0 < k; j0 += 4) {
                const int b0 = b;
                const f32x4 hv = *reinterpret_cast<const f32x4*>(hl + max(b0, 0) * KS + j0);
                bool need[4];
#pragma unroll
                for (int i = 0; i < 4; ++i)
                    need[i] = j0 + i < k && j0 + i != inc && !(b0 >= 0 && ub <= hv[i]);   // Clause 2/3
                if (!(need[0] | need[1] | need[2] | need[3])) continue;
                float Dj[4];
                bool better = false;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    Dj[i] = need[i] ? dist(j0 + i) : INFINITY;
                    better |= Dj[i] < Db;
                }
                if (__any(better)) {
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        bool use = need[i];
                        if (use && b != b0) use = !(ub <= hl[b * KS + j0 + i]);   // a nearer one was found in between
                        nc += use ? 1u : 0u;
                        if (use && Dj[i] < Db) {
                            D2 = Db;
                            Db = Dj[i];
                            b = j0 + i;
                            ub = bound(Db, ecs[b]);
                        } else if (use && Dj[i] < D2) {
                            D2 = Dj[i];
                        }
                    }
                } else {   // no lane found a nearer one
#pragma unroll
                    for (int i = 0; i < 4; ++i) {
                        nc += need[i] ? 1u : 0u;
                        D2 = fminf(D2, Dj[i]);
                    }
                }
            }
        }
        if (scan && D2 != INFINITY) {
            const float band = 2.f * gamma * (Db + D2) + 4.f * (sqrtf(Db) + sqrtf(D2)) * ecmax + 8.f * ecmax * ecmax;
            if (D2 - Db <= band) {   // near tie: float64 against the master centroids, oracle's tie rule
                int bb = -1;
                double Dbb = INFINITY;
                if (inc >= 0) {
                    Dbb = sqd64(xr, P.C64 + (int64_t)inc * d, d);
                    bb = inc;
                }
                for (int j = 0; j < k; ++j) {
                    if (j == inc) continue;
                    const double Dj = sqd64(xr, P.C64 + (int64_t)j * d, d);
                    if (Dj < Dbb) {
                        Dbb = Dj;
                        bb = j;
                    }
                }
                b = bb;
                ub = f32_up(sqrt(Dbb) * (1.0 + 0x1p-40));
                my_rc += 1;
            }
        }
        if (b < 0) b = 0;   // only for non-finite rows
        const bool moved = live && b != inc;
        if (live) {
            P.w[p] = state_of<7>(ub, ddn[b], b);
            my_comp += nc;
            my_changed += moved ? 1u : 0u;
        }
        const uint64_t mm = __ballot(moved);
        if (mm) {
            if (moved) ml[lanes_below(mm)] = make_uint2((uint32_t)p, (uint32_t)b | ((uint32_t)(inc + 1) << 16));
            wave_sync();
            apply_moves(ml, __popcll(mm), P.X, d, AR, P.qscale, acc, cnt);
            wave_sync();
        }
    };

    const int64_t n = P.n;
    const int tile = 64 * nsub;   // points a wave takes at once
    const int nwt = (int)((n + tile - 1) / tile);
    const int wt_lo = (int)((int64_t)blockIdx.x * nwt / gridDim.x);
    const int wt_hi = (int)((int64_t)(blockIdx.x + 1) * nwt / gridDim.x);
    int qn = 0;
    int wt = wt_lo + w;
    while (wt < wt_hi) {
        const int base = wt * tile;
        uint32_t sv[kGenTile / 64] = {};
#pragma unroll
        for (int c = 0; c < kGenTile / 64; ++c)
            if (c < nsub) sv[c] = P.w[base + 64 * c + lane];   // the state array is padded
        int nxt = 0;
        if (lane == 0) nxt = wt_lo + kGenWaves + atomicAdd(tcount, 1);
        nxt = __builtin_amdgcn_readfirstlane(nxt);
#pragma unroll 1
        for (int c = 0; c < nsub; ++c) {
            const int p = base + 64 * c + lane;
            const bool valid = p < n;
            const uint32_t ws = sv[0];
#pragma unroll
            for (int i = 0; i + 1 < kGenTile / 64; ++i) sv[i] = sv[i + 1];
            if (first) {
                settle(valid ? p : (int)n - 1, 0u, valid);
                continue;
            }
            const bool surv = valid && !(state_value<7>(ws) <= thr[state_cluster<7>(ws)]);
            const uint64_t bm = __ballot(surv);
            c1w += (uint32_t)__popcll(__ballot(valid && !surv));
            if (surv) q[qn + lanes_below(bm)] = make_uint2((uint32_t)p, ws);
            qn += __popcll(bm);
            if (qn >= 64) {
                wave_sync();
                qn -= 64;
                const uint2 e = q[qn + lane];
                settle((int)e.x, e.y, true);
                wave_sync();
            }
        }
        wt = nxt;
    }
    if (qn > 0) {
        wave_sync();
        const uint2 e = q[lane < qn ? lane : 0];
        settle((int)e.x, e.y, lane < qn);
    }

    const uint64_t v0 = wave_sum_u64(my_changed), v1 = wave_sum_u64(my_comp), v3 = wave_sum_u64(my_rc);
    if (lane == 0) {
        unsigned long long* bs = reinterpret_cast<unsigned long long*>(bst);
        atomicAdd(bs + kStChanged, (unsigned long long)v0);
        atomicAdd(bs + kStComputed, (unsigned long long)v1);
        atomicAdd(bs + kStClause1, (unsigned long long)c1w);
        atomicAdd(bs + kStRecheck, (unsigned long long)v3);
    }
    __syncthreads();
    flush_block(P, acc, cnt, bst, AR, kGenThreads);
}

// ---------------------------------------------------------------------------
// Matrix-core form.  A wave settles 32 survivors at a time: lanes l and l + 32
// serve survivor l % 32, lane half h loading dimensions 16 s + 8 h .. + 7 of
// k-step s straight from the row in X (two 16-byte loads; the next kQS steps'
// loads, of this batch or the next, are in flight while these are
// multiplied).  x.c is formed on v_mfma_f32_32x32x16_f16 from split operands,
// hi = f16(x 2^a), lo = f16(x 2^a - hi), as hi.hi + hi.lo + lo.hi; the
// centroids' split operands of the whole step stay in LDS in lane order.  The
// scale 2^a (IterState::xscale) maps the bound on |x| that the set-up's
// sample gives to 2^13, so that f16 neither overflows nor loses the low part
// of ordinary values; a row or a centroid table past 2^15 takes the direct
// form over all centroids.
//
// Where the data lie far from the origin, rows and centroids are taken relative
// to mu (Dev::mu), x 2^a - mu 2^a in one rounding: x and c below are then these.
//
// Error of dot' = x.c - |c|^2 / 2 (the nearest centroid has the largest; the
// row's own norm does not enter the comparison), in scaled units (|x|, |c| of
// the scaled row and centroid, D = 16 ceil(d / 16)):
//   - the dropped lo.lo and the two residuals (both conversions round to
//     nearest), 3.01 2^-22 |x_m| |c_m| per dimension;
//   - the accumulation, 18 units of 2^-23 relative to |C| + sum |p| per
//     instruction of 16 exact products: two k-steps at a time have an
//     accumulator of their own, hi.lo and lo.hi first (2^-10 of the
//     magnitude), then hi.hi, and are added to the total, so the chain that
//     carries the magnitude is two instructions long (72.6 2^-24
//     sum |x_m| |c_m|, and one unit of 2^-24 per addition).  k > 128, short of
//     registers, runs one chain of 3 D / 16 instructions (6.9 D 2^-24).  With
//     one chain most survivors of a wide case (d = 174, k = 10, some
//     centroids in the same component) had several candidates;
//   - the final additions and the rounded |c|^2: 2 2^-24 |x| |c| and
//     1.5 2^-24 |c|^2;
//   - with mu the roundings of x and c, 2.1 2^-24 |x| |c|;
//   - f16 values below the normal range (flushed at worst): 2^-14 sqrt(D) R,
//     R = |x| + max |c|.
// The bound of a settled survivor, from |x|^2 - 2 dot', adds the norm's
// (D + 8) 2^-24 R^2.
//
// A lone candidate within the bound is the nearest centroid and settles the
// survivor at once (its bound from the expanded value).  The others are
// listed with their candidates and decided together once enough are listed:
// done in place, the few of them in nearly every batch would hold up all 32.
//
// Bound by latency at small sizes (a wave's chain of batches; a batch's rows
// are requested before the batch before it is settled) and by vector
// instructions (splits, selection) otherwise.  Two waves per SIMD with the
// next four k-steps in registers: held to 128 registers (four waves per SIMD)
// it spilled, 97 us a step against 64 us at 300K x 64, k = 50.  The general
// kernel, which it replaces, took 1230 us there (43 us of the 64 are this
// kernel's), 18.9 ms at 700K x 128, k = 56 (now 119 us a step) and 4.1 ms at
// 575K x 174, k = 10 (now 250 us).  For d <= 32 a whole row is held and the
// next batch's rows are the only loads ahead; up to k = 64 that leaves room for
// three waves per SIMD: 20M x 32, k = 64 takes 0.79 ms a step, 1.10 at two
// waves, and 1.21 took a form with bf16 operands, its centroids in registers
// and queues by the blocks of centroids a survivor needs.  Leaving blocks of
// centroids out by Clause 2 costs a tenth where few batches can (0.99 to 1.10
// ms at two waves there): only the four-block form does (k > 64), where well
// separated clusters leave out most of the products.

// k-steps loaded ahead (kQS); ONE: all of a row (d <= 32).
template <int KB, bool ONE>
constexpr int gen_mat_steps() { return ONE || KB >= 4 ? 2 : 4; }

template <int KB, bool VEC, bool ONE>
__global__ __launch_bounds__(64 * gen_mat_waves(KB, ONE)) __attribute__((amdgpu_waves_per_eu(gen_mat_waves(KB, ONE) / 4))) void k_inc_mat(Dev P_, int first, int check, int nsub) {
    const Dev P = with_scales(P_);
    IterState* st = P.st;
    if (step_idle(st, first, check)) return;
    if (blockIdx.x == 0 && threadIdx.x == 0) st->active = 1;
    constexpr int CB = KB == 8 ? 8 : 7;   // cluster bits of a state word
    constexpr int QS = gen_mat_steps<KB, ONE>();
    constexpr bool kSkip = KB == 4;       // Clause 2 per block of centroids
    constexpr int NW = gen_mat_waves(KB, ONE), NT = 64 * NW;
    constexpr bool kTwo = KB <= 4;        // two k-steps at a time in an accumulator of their own
    const int k = P.k, d = P.d, tid = threadIdx.x, lane = tid & 63;
    const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int col = lane & 31, half = lane >> 5;
    const int ns = (d + 15) / 16;
    const float xsc = st->xscale, xinv = st->xinv;
    const bool shift = st->shift != 0;
    const float ecmax = st->ec_max, ecs_max = st->ec_max * xsc, gamma = P.gamma;
    const GenMatLds lay = gen_mat_lds(KB, NW, d, k);
    const int AR = lay.ar;
    uint4* cau = reinterpret_cast<uint4*>(km_smem + lay.off_ca);   // [s][cb][hi, lo][lane]
    float* nb = reinterpret_cast<float*>(km_smem + lay.off_nb);
    float* thr = reinterpret_cast<float*>(km_smem + lay.off_thr);
    float* ecs = reinterpret_cast<float*>(km_smem + lay.off_ec);
    float* ddn = reinterpret_cast<float*>(km_smem + lay.off_ddn);
    float* dup = reinterpret_cast<float*>(km_smem + lay.off_dup);
    float* hm = reinterpret_cast<float*>(km_smem + lay.off_hm);
    uint64_t* acc = reinterpret_cast<uint64_t*>(km_smem + lay.off_acc);
    int* cnt = reinterpret_cast<int*>(km_smem + lay.off_cnt);
    int* tcount = reinterpret_cast<int*>(km_smem + lay.off_misc);
    uint64_t* bst = reinterpret_cast<uint64_t*>(km_smem + lay.off_misc + 16);
    GenMatWave* wl = reinterpret_cast<GenMatWave*>(km_smem + lay.off_w) + w;   // this wave's lists

    // Split operands of the centroids: lane l of (s, cb) feeds centroid row
    // 32 cb + l % 32, dimensions 16 s + 8 (l / 32) .. + 7.
    auto split8 = [](const float (&v)[8], uint4& hi, uint4& lo) __attribute__((always_inline)) {
        uint32_t h[4], o[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const f32x2 ab = {v[2 * p], v[2 * p + 1]};
            const f16x2 hh = __builtin_convertvector(ab, f16x2);
            const f32x2 r = {ab.x - (float)hh.x, ab.y - (float)hh.y};
            h[p] = __builtin_bit_cast(uint32_t, hh);
            o[p] = __builtin_bit_cast(uint32_t, __builtin_convertvector(r, f16x2));
        }
        hi = make_uint4(h[0], h[1], h[2], h[3]);
        lo = make_uint4(o[0], o[1], o[2], o[3]);
    };
    for (int i = tid; i < ns * KB * 64; i += NT) {
        const int l = i & 63, cb = (i >> 6) % KB, s = i / (64 * KB);
        const int j = cb * 32 + (l & 31), m0 = 16 * s + 8 * (l >> 5);
        float v[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) v[e] = j < k && m0 + e < d ? P.C32[(int64_t)j * d + m0 + e] : 0.f;
        if (shift) {   // uniform
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = j < k ? fmaf(v[e], xsc, -(P.mu[m0 + e] * xsc)) : 0.f;
        } else {
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] *= xsc;
        }
        uint4 hi, lo;
        split8(v, hi, lo);
        cau[((s * KB + cb) * 2) * 64 + l] = hi;
        cau[((s * KB + cb) * 2 + 1) * 64 + l] = lo;
    }
    // -|c|^2 / 2 in scaled units (padding centroids: a value no point reaches).
    for (int i = tid; i < 32 * KB; i += NT) nb[i] = i < k ? -0.5f * ((P.cn2[i] * xsc) * xsc) : -0x1p100f;
    for (int i = tid; i < k * AR; i += NT) acc[i] = 0;
    for (int i = tid; i < k; i += NT) {
        thr[i] = first ? 0.f : clause1_thr(P.s[i], P.dhi[i]);
        ecs[i] = P.ec[i];
        ddn[i] = P.ddnf[i];
        if constexpr (kSkip) dup[i] = P.dupf[i];
        cnt[i] = 0;
    }
    if constexpr (kSkip)
        for (int i = tid; i < 4 * k; i += NT) hm[i] = P.hm[i];
    if (tid < kNumStat) bst[tid] = 0;
    if (tid == 0) *tcount = 0;
    __syncthreads();
    float cnmax, cbad = 0.f;
    bool tiny;
    {
        float m2 = 0.f;
        for (int i = lane; i < k; i += 64) {
            const float v = -2.f * nb[i];
            cbad = v <= 0x1p30f ? cbad : 1.f;   // out of range or not finite
            m2 = fmaxf(m2, v);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) {
            m2 = fmaxf(m2, __shfl_xor(m2, off));
            cbad = fmaxf(cbad, __shfl_xor(cbad, off));
        }
        cnmax = sqrtf(m2) * kUp * kUp;
        // Norms this far below 1 have lost bits in cn2 (float32, unscaled) or
        // all of them, and so have the direct form's distances: every survivor
        // is decided in float64.
        tiny = m2 < 0x1p-100f * xsc * xsc;
        if (tiny) cbad = 1.f;
    }
    const float Dp = (float)(16 * ns);
    const float gexp = (Dp + 8.f) * 0x1p-24f;
    const float gacc = kTwo ? 36.3f * (float)min(2, ns) + (float)((ns + 1) / 2) : 6.9f * Dp;
    const float gsp2 = 2.f * (14.1f + (shift ? 2.1f : 0.f) + gacc) * 0x1p-24f * (1.f + 0x1p-10f);
    const float gabs = 0x1p-13f * sqrtf(Dp) * kUp;

    uint32_t my_changed = 0, my_comp = 0, my_rc = 0, c1w = 0;

    // Loads of k-steps [s0, s0 + QS) of the row at rp: this lane's 8
    // dimensions of each, zero past d.
    struct Ahead {
        f32x4 v[2 * QS];
    };
    auto load_steps = [&](const float* rp, int s0, Ahead& A) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < QS; ++i) {
            const int s = s0 + i, m0 = 16 * s + 8 * half;
            if (s >= ns) break;   // uniform
            if (16 * s + 16 <= d) {   // uniform
                if constexpr (VEC) {
                    A.v[2 * i] = *reinterpret_cast<const f32x4*>(rp + m0);
                    A.v[2 * i + 1] = *reinterpret_cast<const f32x4*>(rp + m0 + 4);
                } else {
                    A.v[2 * i] = *reinterpret_cast<const f32x4u*>(rp + m0);
                    A.v[2 * i + 1] = *reinterpret_cast<const f32x4u*>(rp + m0 + 4);
                }
            } else {
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    f32x4 t = {0.f, 0.f, 0.f, 0.f};
                    const int m = m0 + 4 * c;
                    if constexpr (VEC) {
                        if (m < d) t = *reinterpret_cast<const f32x4*>(rp + m);
                    } else {
                        if (m < d) t.x = rp[m];
                        if (m + 1 < d) t.y = rp[m + 1];
                        if (m + 2 < d) t.z = rp[m + 2];
                        if (m + 3 < d) t.w = rp[m + 3];
                    }
                    A.v[2 * i + c] = t;
                }
            }
        }
    };

    // Two direct-form squared distances, of points p to centroids j, by a
    // group of lp lanes (lane gl of it): every lane of the group gets them.
    const int lp = d <= 8 ? 1 : d <= 16 ? 2 : d <= 32 ? 4 : d <= 64 ? 8 : 16;
    const int gl = lane & (lp - 1), grp = lane / lp, ngrp = 64 / lp;
    auto direct = [&](const int (&p)[2], const int (&j)[2], float (&a)[2]) __attribute__((always_inline)) {
        const float *x0 = P.X + (int64_t)p[0] * d, *c0 = P.C32 + (int64_t)j[0] * d;
        const float *x1 = P.X + (int64_t)p[1] * d, *c1 = P.C32 + (int64_t)j[1] * d;
        a[0] = a[1] = 0.f;
        auto sq = [](const f32x4& x, const f32x4& c, float s) __attribute__((always_inline)) {
            const float t0 = x.x - c.x, t1 = x.y - c.y, t2 = x.z - c.z, t3 = x.w - c.w;
            return fmaf(t3, t3, fmaf(t2, t2, fmaf(t1, t1, fmaf(t0, t0, s))));
        };
        int m = 4 * gl;
#pragma unroll 2
        for (; m + 4 <= d; m += 4 * lp) {
            const f32x4 u0 = *reinterpret_cast<const f32x4u*>(x0 + m), v0 = *reinterpret_cast<const f32x4u*>(c0 + m);
            const f32x4 u1 = *reinterpret_cast<const f32x4u*>(x1 + m), v1 = *reinterpret_cast<const f32x4u*>(c1 + m);
            a[0] = sq(u0, v0, a[0]);
            a[1] = sq(u1, v1, a[1]);
        }
        for (int e = m; e < min(m + 4, d); ++e) {   // the row's last 1 .. 3 dimensions (one lane of the group)
            const float t0 = x0[e] - c0[e], t1 = x1[e] - c1[e];
            a[0] = fmaf(t0, t0, a[0]);
            a[1] = fmaf(t1, t1, a[1]);
        }
        for (int o = 1; o < lp; o <<= 1) {
            a[0] += __shfl_xor(a[0], o);
            a[1] += __shfl_xor(a[1], o);
        }
    };
    // The listed survivors (ln of them, pn candidate pairs): the pairs'
    // direct-form distances, a group of lanes per pair (coalesced rows, all
    // of a round's loads in flight together); then a lane per survivor takes
    // the nearest (the incumbent wins a tie, then the lowest index); near
    // ties are decided in float64 by the whole wave.
    auto settle_listed = [&](int ln, int pn) __attribute__((always_inline)) {
        for (int r = 0; r < pn; r += 2 * ngrp) {
            const int i0 = r + grp, i1 = i0 + ngrp;
            const uint32_t p0 = wl->pl[i0 < pn ? i0 : 0], p1 = wl->pl[i1 < pn ? i1 : 0];
            const int pp[2] = {(int)wl->lq[p0 >> 8].x, (int)wl->lq[p1 >> 8].x};
            const int jj[2] = {(int)(p0 & 255u), (int)(p1 & 255u)};
            float a[2];
            direct(pp, jj, a);
            if (gl == 0 && i0 < pn) wl->pd[i0] = a[0];
            if (gl == 0 && i1 < pn) wl->pd[i1] = a[1];
        }
        wave_sync();
        const bool live = lane < ln;
        const int e = live ? lane : 0;
        const uint2 pw = wl->lq[e];
        const uint32_t lo = wl->lo[e];   // first pair, number of pairs << 16 (0: all centroids)
        const int p = (int)pw.x, inc = first ? -1 : state_cluster<CB>(pw.y);
        const int o0 = (int)(lo & 0xffffu), tot = (int)(lo >> 16);
        float d1 = INFINITY, d2 = INFINITY;
        int rk1 = INT_MAX, j1 = 0;
        auto take = [&](float a, int rk, int j) __attribute__((always_inline)) {
            if (a < d1 || (a == d1 && rk < rk1)) {
                d2 = d1;
                d1 = a;
                rk1 = rk;
                j1 = j;
            } else if (a < d2) {
                d2 = a;
            }
        };
        for (int i = 0; i < (live ? tot : 0); ++i) {
            const int j = (int)(wl->pl[o0 + i] & 255u);
            take(wl->pd[o0 + i], j == inc ? -1 : j, j);
        }
        uint64_t am = __ballot(live && tot == 0);   // all centroids
        if constexpr (ONE) {
            // Many narrow rows: a lane each, four centroids at a time, as the
            // general kernel scans.  With duplicate centroids these are most
            // survivors, and one after another they took 10 times its step:
            // 500K x 1 whole numbers, k = 128 1130 us a step, now 78 (84 there).
            // The scan takes as long for one row as for all, a row by groups
            // of lanes its own time: they meet near this many rows (1 to 10
            // dimensions, 65 to 256 centroids; with a quarter of them 5000 x 1,
            // k = 200 took 1.33 times as long, 20K x 6, k = 200 1.41 times).
            if (__builtin_expect(d <= kGenLaneD && __popcll(am) > 4 + k * (d + 10) / 100, 0)) {
                const float* xr = P.X + (int64_t)p * d;
                float x[kGenLaneD];
#pragma unroll
                for (int m = 0; m < kGenLaneD; ++m) x[m] = m < d ? xr[m] : 0.f;   // uniform
                for (int j0 = 0; j0 < k; j0 += 4) {
                    float a[4];
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const float* c = P.C32 + (int64_t)min(j0 + q, k - 1) * d;
                        a[q] = 0.f;
#pragma unroll
                        for (int m = 0; m < kGenLaneD; ++m) {
                            if (m >= d) break;   // uniform
                            const float t = x[m] - c[m];
                            a[q] = fmaf(t, t, a[q]);
                        }
                    }
                    if (live && tot == 0) {
#pragma unroll
                        for (int q = 0; q < 4; ++q)
                            if (j0 + q < k) take(a[q], j0 + q == inc ? -1 : j0 + q, j0 + q);
                    }
                }
                am = 0;
            }
        }
        for (; am; am &= am - 1) {   // a group of lanes per centroid
            const int l = __builtin_ctzll(am);
            const int pa = __shfl(p, l), ia = __shfl(inc, l);
            float a1 = INFINITY, a2 = INFINITY;
            int ar = INT_MAX, aj = 0;
            for (int j0 = 0; j0 < k; j0 += 2 * ngrp) {
                const int pp[2] = {pa, pa}, jj[2] = {min(j0 + grp, k - 1), min(j0 + ngrp + grp, k - 1)};
                float a[2];
                direct(pp, jj, a);
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int j = j0 + q * ngrp + grp, rk = j == ia ? -1 : j;
                    if (j >= k) continue;
                    if (a[q] < a1 || (a[q] == a1 && rk < ar)) {
                        a2 = a1;
                        a1 = a[q];
                        ar = rk;
                        aj = j;
                    } else if (a[q] < a2) {
                        a2 = a[q];
                    }
                }
            }
            for (int o = lp; o < 64; o <<= 1) {
                const float b1 = __shfl_xor(a1, o), b2 = __shfl_xor(a2, o);
                const int br = __shfl_xor(ar, o), bj = __shfl_xor(aj, o);
                if (b1 < a1 || (b1 == a1 && br < ar)) {
                    a2 = fminf(a1, b2);
                    a1 = b1;
                    ar = br;
                    aj = bj;
                } else {
                    a2 = fminf(a2, b1);
                }
            }
            if (lane == l) {
                d1 = a1;
                d2 = a2;
                j1 = aj;
            }
        }
        int b = j1;
        float ub = upper_bound(d1, ecs[b], gamma);
        bool re = false;
        if (live && d2 != INFINITY) {
            const float band = 2.f * gamma * (d1 + d2) + 4.f * (sqrtf(d1) + sqrtf(d2)) * ecmax + 8.f * ecmax * ecmax;
            re = d2 - d1 <= band;
        }
        re |= live && tiny;
        // Float64 against the master centroids, every distance summed over the
        // dimensions in order by one lane as on the other paths: rows at equal
        // distances from two centroids then fall alike on all of them.
        if (d <= kGenLaneD) {   // a lane per row
            if (__builtin_expect(re, 0)) {
                const float* xr = P.X + (int64_t)p * d;
                double Dbb = INFINITY;
                int kb = INT_MAX, bb = -1;
                for (int i = 0; i < (tot ? tot : k); ++i) {
                    const int j = tot ? (int)(wl->pl[o0 + i] & 255u) : i;
                    const double Dj = sqd64(xr, P.C64 + (int64_t)j * d, d);
                    const int rk = j == inc ? -1 : j;
                    if (Dj < Dbb || (Dj == Dbb && rk < kb)) {
                        Dbb = Dj;
                        kb = rk;
                        bb = j;
                    }
                }
                b = bb < 0 ? 0 : bb;
                ub = f32_up(sqrt(Dbb) * (1.0 + 0x1p-40));
                my_rc += 1;
            }
        } else {
            for (uint64_t rm = __ballot(re); rm; rm &= rm - 1) {
                const int l = __builtin_ctzll(rm);
                const int pa = __shfl(p, l), ia = __shfl(inc, l), oa = __shfl(o0, l), ta = __shfl(tot, l);
                const float* xr = P.X + (int64_t)pa * d;
                double Dbb = INFINITY;
                int kb = INT_MAX, bb = -1;
                auto take64 = [&](double D, int rk, int j) __attribute__((always_inline)) {
                    if (D < Dbb || (D == Dbb && rk < kb)) {
                        Dbb = D;
                        kb = rk;
                        bb = j;
                    }
                };
                // Few candidates: the whole wave forms one distance after
                // another, which decides unless the two smallest lie within
                // the rounding of the sums.
                bool order = ta == 0;
                if (ta) {
                    double D2 = INFINITY;
                    for (int i = 0; i < ta; ++i) {
                        const int j = (int)(wl->pl[oa + i] & 255u);
                        const double* cr = P.C64 + (int64_t)j * d;
                        double Dj = 0.0;
                        for (int m = lane; m < d; m += 64) {
                            const double t = (double)xr[m] - cr[m];
                            Dj = fma(t, t, Dj);
                        }
#pragma unroll
                        for (int o = 32; o > 0; o >>= 1) Dj += __shfl_xor(Dj, o);
                        D2 = fmin(D2, fmax(Dj, Dbb));
                        take64(Dj, j == ia ? -1 : j, j);
                    }
                    order = !(D2 - Dbb > 0x1p-40 * D2);   // (two orders differ by 2 (d + 6) 2^-53 of it, d <= 1024)
                }
                if (order) {   // a lane per centroid
                    Dbb = INFINITY;
                    kb = INT_MAX;
                    bb = -1;
                    for (int i = lane; i < (ta ? ta : k); i += 64) {
                        const int j = ta ? (int)(wl->pl[oa + i] & 255u) : i;
                        take64(sqd64(xr, P.C64 + (int64_t)j * d, d), j == ia ? -1 : j, j);
                    }
#pragma unroll
                    for (int o = 32; o > 0; o >>= 1) take64(__shfl_xor(Dbb, o), __shfl_xor(kb, o), __shfl_xor(bb, o));
                }
                if (lane == l) {
                    b = bb < 0 ? 0 : bb;
                    ub = f32_up(sqrt(Dbb) * (1.0 + 0x1p-40));
                    my_rc += 1;
                }
            }
        }
        const bool moved = live && b != inc;
        if (live) {
            P.w[p] = state_of<CB>(ub, ddn[b], b);
            my_changed += moved ? 1u : 0u;
        }
        const uint64_t mm = __ballot(moved);
        if (mm) {
            if (moved) wl->ml[lanes_below(mm)] = make_uint2((uint32_t)p, (uint32_t)b | ((uint32_t)(inc + 1) << 16));
            wave_sync();
            apply_moves(wl->ml, __popcll(mm), P.X, d, AR, P.qscale, acc, cnt);
        }
        wave_sync();
    };

    Ahead A;
    int bcnt = 0, ln = 0, pn = 0;     // survivors of the batch in flight; listed survivors and their candidate pairs
    int bp = 0;                       // the batch's point of this lane
    uint32_t bw = 0;                  // and its state
    auto take_batch = [&](int e0, int c) __attribute__((always_inline)) {
        const uint2 e = wl->q[e0 + (col < c ? col : 0)];
        bp = (int)e.x;
        bw = e.y;
        bcnt = c;
        load_steps(P.X + (int64_t)bp * d, 0, A);
    };
    auto bf = [](uint4 u) { return __builtin_bit_cast(f16x8, u); };
    auto scan_batch = [&]() __attribute__((always_inline)) {
        const bool live = col < bcnt;
        const int inc = first ? -1 : state_cluster<CB>(bw);
        const float* rp = P.X + (int64_t)bp * d;
        // Clause 2 per block of centroids over the whole batch: a block is
        // left out when every survivor's bound is at most half the distance
        // from its centroid to each of the block's (its own block never is).
        bool eval[KB];
        int nreal = k;   // centroids of the blocks taken
#pragma unroll
        for (int cb = 0; cb < KB; ++cb) eval[cb] = true;
        if constexpr (kSkip) {
            if (!first) {
                const float u = (state_value<CB>(bw) + dup[inc]) * kUp;
#pragma unroll
                for (int cb = 0; cb < KB; ++cb) {
                    eval[cb] = __ballot(live && !(u <= hm[4 * inc + cb])) != 0;
                    if (!eval[cb]) nreal -= min(32, max(k - 32 * cb, 0));
                }
            }
        }
        f32x16 dot[KB];
#pragma unroll
        for (int cb = 0; cb < KB; ++cb)
#pragma unroll
            for (int e = 0; e < 16; ++e) dot[cb][e] = eval[cb] ? 0.f : -INFINITY;
        float x2 = 0.f;
        for (int s0 = 0; s0 < (ONE ? 1 : ns); s0 += QS) {
            Ahead N;
            const bool more = !ONE && s0 + QS < ns;
            if (more) load_steps(rp, s0 + QS, N);
#pragma unroll
            for (int i = 0; i < QS; i += 2) {
                if (s0 + i >= ns) break;   // uniform
                const bool both = s0 + i + 1 < ns;
                uint4 bhi[2], blo[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    float v[8];
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        const f32x4 t = A.v[2 * (i + q) + c];
                        v[4 * c] = t.x * xsc;
                        v[4 * c + 1] = t.y * xsc;
                        v[4 * c + 2] = t.z * xsc;
                        v[4 * c + 3] = t.w * xsc;
                    }
                    if (__builtin_expect(shift && (q == 0 || both), 0)) {   // uniform
                        const float* mp = P.mu + 16 * (s0 + i + q) + 8 * half;
#pragma unroll
                        for (int e = 0; e < 8; ++e) v[e] = fmaf(A.v[2 * (i + q) + e / 4][e % 4], xsc, -(mp[e] * xsc));
                    }
                    if (q == 0 || both) {
#pragma unroll
                        for (int e = 0; e < 8; ++e) x2 = fmaf(v[e], v[e], x2);
                        split8(v, bhi[q], blo[q]);
                    }
                }
                const uint4* ca = cau + (s0 + i) * KB * 128 + lane;
#pragma unroll
                for (int cb = 0; cb < KB; ++cb) {
                    if (!eval[cb]) continue;   // uniform
                    f32x16 pr = kTwo ? f32x16{} : dot[cb];
                    const uint4 ah = ca[cb * 128], al = ca[cb * 128 + 64];
                    pr = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf(ah), bf(blo[0]), pr, 0, 0, 0);
                    pr = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf(al), bf(bhi[0]), pr, 0, 0, 0);
                    if (both) {
                        const uint4 ah1 = ca[(KB + cb) * 128], al1 = ca[(KB + cb) * 128 + 64];
                        pr = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf(ah1), bf(blo[1]), pr, 0, 0, 0);
                        pr = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf(al1), bf(bhi[1]), pr, 0, 0, 0);
                        pr = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf(ah1), bf(bhi[1]), pr, 0, 0, 0);
                    }
                    pr = __builtin_amdgcn_mfma_f32_32x32x16_f16(bf(ah), bf(bhi[0]), pr, 0, 0, 0);
                    if constexpr (kTwo) {
#pragma unroll
                        for (int e = 0; e < 16; ++e) dot[cb][e] += pr[e];
                    } else {
                        dot[cb] = pr;
                    }
                }
            }
            if (more) A = N;
        }
        x2 += __shfl_xor(x2, 32);
        // dot' = x.c - |c|^2 / 2: the nearest centroid has the largest.
        float dmax = -INFINITY;
#pragma unroll
        for (int cb = 0; cb < KB; ++cb)
#pragma unroll
            for (int a4 = 0; a4 < 4; ++a4) {
                const f32x4 nv = *reinterpret_cast<const f32x4*>(nb + cb * 32 + 8 * a4 + 4 * half);
                dot[cb][4 * a4] += nv.x;
                dot[cb][4 * a4 + 1] += nv.y;
                dot[cb][4 * a4 + 2] += nv.z;
                dot[cb][4 * a4 + 3] += nv.w;
                dmax = fmaxf(fmaxf(dmax, dot[cb][4 * a4]), dot[cb][4 * a4 + 1]);
                dmax = fmaxf(fmaxf(dmax, dot[cb][4 * a4 + 2]), dot[cb][4 * a4 + 3]);
            }
        dmax = fmaxf(dmax, __shfl_xor(dmax, 32));
        const float e1 = fmaf(-2.f, dmax, x2);
        const float xn = sqrtf(fmaxf(x2, 0.f)) * (1.0f + 0x1p-20f);
        const float R = xn + cnmax;
        const float E = (gsp2 * xn * cnmax + 0x1.8p-23f * cnmax * cnmax + gabs * R + 4.f * R * ecs_max +
                         2.f * ecs_max * ecs_max) * kUp;
        const float lim = dmax - E;
        // Register e of block cb holds centroid 32 cb + 8 (e / 4) + 4 half + e % 4.
        bool one = false, two = false;
        int jown = -1;
#pragma unroll
        for (int cb = 0; cb < KB; ++cb)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const bool c = dot[cb][e] >= lim;
                two |= one & c;
                one |= c;
                jown = c ? cb * 32 + 8 * (e >> 2) + (e & 3) : jown;
            }
        jown = jown >= 0 ? jown + 4 * half : -1;
        const int joth = __shfl_xor(jown, 32);
        const bool wild = !(x2 <= 0x1p30f) || cbad != 0.f || !(lim > -0x1p99f);
        const bool dbl = two || (jown >= 0 && joth >= 0) || (jown < 0 && joth < 0) || wild;
        const bool several = __shfl_xor((int)dbl, 32) | (int)dbl;
        const int b = max(jown, joth);
        const bool settled = live && !several;
        bool moved = false;
        if (settled && half == 0) {
            const float ub = __builtin_amdgcn_sqrtf(fmaxf(e1 + E + gexp * R * R, 0.f)) * (1.0f + 0x1p-20f) * kUp * xinv;
            P.w[bp] = state_of<CB>(ub * kUp, ddn[b], b);
            moved = b != inc;
            my_changed += moved ? 1u : 0u;
        }
        if (live && half == 0) my_comp += (uint32_t)nreal;
        const uint64_t lm = __ballot(live && several && half == 0);
        if (lm) {   // list them with their candidates
            const int e = ln + __popcll(lm & ((1ull << col) - 1ull));
            const bool mine = live && several;
            int own = 0;
            uint32_t cm[(KB + 1) / 2];   // candidate bits: 16 per block of centroids
#pragma unroll
            for (int c2 = 0; c2 < (KB + 1) / 2; ++c2) {
                uint32_t m = 0;
#pragma unroll
                for (int i = 0; i < 32; ++i) {
                    constexpr int kLast = KB - 1;
                    const int cb = 2 * c2 + (i >> 4) <= kLast ? 2 * c2 + (i >> 4) : kLast;
                    if (2 * c2 + (i >> 4) <= kLast) m |= dot[cb][i & 15] >= lim ? 1u << i : 0u;
                }
                cm[c2] = mine && !wild ? m : 0u;
                own += __popc(cm[c2]);
            }
            const int oth = __shfl_xor(own, 32);
            int tot = own + oth;
            if (!mine || wild || tot > kGenCand) tot = 0;   // 0: all centroids
            // Pair offsets: the total of the listed survivors of lower lanes.
            int pre = half == 0 ? tot : 0;
#pragma unroll
            for (int o = 1; o < 32; o <<= 1) {
                const int t = __shfl_up(pre, o);
                if (col >= o) pre += t;
            }
            const int all = __builtin_amdgcn_readlane(pre, 31);
            pre = __shfl(pre, col) - tot;   // exclusive; both halves
            if (mine) {
                if (half == 0) {
                    wl->lq[e] = make_uint2((uint32_t)bp, bw);
                    wl->lo[e] = (uint32_t)(pn + pre) | ((uint32_t)tot << 16);
                }
                if (tot) {
                    int at = pn + pre + (half == 0 ? 0 : oth);
#pragma unroll
                    for (int c2 = 0; c2 < (KB + 1) / 2; ++c2)
                        for (uint32_t m = cm[c2]; m; m &= m - 1) {
                            const int i = __builtin_ctz(m);
                            const int j = 64 * c2 + 32 * (i >> 4) + 8 * ((i >> 2) & 3) + 4 * half + (i & 3);
                            wl->pl[at++] = (uint16_t)((e << 8) | j);
                        }
                }
            }
            ln += __popcll(lm);
            pn += all;
        }
        const uint64_t mm = __ballot(moved);
        if (mm) {
            if (moved) wl->ml[lanes_below(mm)] = make_uint2((uint32_t)bp, (uint32_t)b | ((uint32_t)(inc + 1) << 16));
            wave_sync();
            apply_moves(wl->ml, __popcll(mm), P.X, d, AR, P.qscale, acc, cnt);
        }
        wave_sync();
        bcnt = 0;
    };

    const int64_t n = P.n;
    const int tile = 64 * nsub;   // points a wave takes at once
    const int nwt = (int)((n + tile - 1) / tile);
    const int wt_lo = (int)((int64_t)blockIdx.x * nwt / gridDim.x);
    const int wt_hi = (int)((int64_t)(blockIdx.x + 1) * nwt / gridDim.x);
    int qn = 0;
    int wt = wt_lo + w, sub = 0, base = 0;
    uint32_t sv[kGenTile / 64] = {};
    // One loop: Clause 1 on the next 64 points while the queue is short of a
    // batch; then the batch in flight is settled and the next one's loads
    // issued.  At the end the queue and the list drain.
    for (;;) {
        if (qn < 32 && wt < wt_hi) {
            if (sub == 0) {
                base = wt * tile;
#pragma unroll
                for (int c = 0; c < kGenTile / 64; ++c)
                    if (c < nsub) sv[c] = P.w[base + 64 * c + lane];   // padded
            }
            const int p = base + 64 * sub + lane;
            const bool valid = p < n;
            const uint32_t ws = sv[0];
#pragma unroll
            for (int i = 0; i + 1 < kGenTile / 64; ++i) sv[i] = sv[i + 1];
            const bool surv = valid && (first || !(state_value<CB>(ws) <= thr[state_cluster<CB>(ws)]));
            const uint64_t bm = __ballot(surv);
            c1w += (uint32_t)__popcll(__ballot(valid && !surv));
            if (surv) wl->q[qn + lanes_below(bm)] = make_uint2((uint32_t)p, ws);
            qn += __popcll(bm);
            wave_sync();
            if (++sub == nsub) {
                sub = 0;
                int nxt = 0;
                if (lane == 0) nxt = wt_lo + NW + atomicAdd(tcount, 1);
                wt = __builtin_amdgcn_readfirstlane(nxt);
            }
            continue;
        }
        if (bcnt > 0) scan_batch();
        const bool last = qn == 0;   // no survivor left to take (then no tile is left either)
        if (ln >= (last ? 1 : kGenList) || pn >= kGenPairs) {
            settle_listed(ln, pn);
            ln = pn = 0;
        }
        if (last) break;
        const int c = min(qn, 32);
        qn -= c;
        take_batch(qn, c);
    }

    const uint64_t v0 = wave_sum_u64(my_changed), v1 = wave_sum_u64(my_comp), v3 = wave_sum_u64(my_rc);
    if (lane == 0) {
        unsigned long long* bs = reinterpret_cast<unsigned long long*>(bst);
        atomicAdd(bs + kStChanged, (unsigned long long)v0);
        atomicAdd(bs + kStComputed, (unsigned long long)v1);
        atomicAdd(bs + kStClause1, (unsigned long long)c1w);
        atomicAdd(bs + kStRecheck, (unsigned long long)v3);
    }
    __syncthreads();
    flush_block(P, acc, cnt, bst, AR, NT);
}

// ---------------------------------------------------------------------------
// The end of a step in one block: new centroids, drift, bookkeeping and the
// half-distance table, as k_update and k_centroid_table form them, from the
// accumulation rows.  Those two are launches of k blocks, latency each (8.2
// and 4.2 us at k = 8, d = 5, with the gaps 13 to 17 us between two steps of
// k_inc_vec); here the new centroids stay in LDS between the phases (6.2 us; a run of 15 steps
// of 10K x 5, k = 8 takes 311 us, 420 before; 1M x 32, k = 20 1238 us, 1264).
// One block does all the work, so only while that is little (gen_finish_applies).

constexpr int kFinThreads = 512;

__global__ __launch_bounds__(kFinThreads) void k_gen_finish(Dev P_) {
    const Dev P = with_scales(P_);
    IterState* st = P.st;
    const int k = P.k, d = P.d, kd = k * d, tid = threadIdx.x, lane = tid & 63;
    double* cn = reinterpret_cast<double*>(km_smem);        // [k][DS] new centroids
    const int DS = d | 1;
    double* co = cn + k * DS;                               // [k][DS] the step's centroids
    int64_t* qs = reinterpret_cast<int64_t*>(co + k * DS);  // [k][DS] exact sums (the magic offset removed)
    uint64_t* nc = reinterpret_cast<uint64_t*>(qs + k * DS);   // [k] member counts
    uint64_t* sc = nc + k;                                  // [8] the step's counters
    float* ecs = reinterpret_cast<float*>(sc + 8);          // [k]
    auto row_sum = [&](int64_t o) __attribute__((always_inline)) {
        uint64_t v = 0;
#pragma unroll
        for (int r = 0; r < kGenRows; ++r) v += P.rows[(int64_t)r * P.L + o];
        return v;
    };
    auto clear = [&](int64_t o) __attribute__((always_inline)) {
#pragma unroll
        for (int r = 0; r < kGenRows; ++r) P.rows[(int64_t)r * P.L + o] = 0;
    };
    // Requested before the loop state is looked at: one trip to memory.
    const int e0 = min(tid, kd - 1), a0 = min(tid, k + kNumStat - 1);
    uint64_t tv0 = P.sums[e0] + row_sum(e0);
    const double cold0 = P.C64[e0];
    const uint64_t cv0 = row_sum(kd + a0) + (a0 < k ? P.sums[kd + a0] : 0);
    const bool shift = st->shift != 0;
    if (!st->active) return;
    for (int i = tid; i < k + kNumStat; i += kFinThreads) {   // counts, then the counters
        const uint64_t v = i == tid ? cv0 : row_sum(kd + i) + (i < k ? P.sums[kd + i] : 0);
        if (i < k) {
            nc[i] = v;
            P.sums[kd + i] = v;
        } else {
            sc[i - k] = v;
        }
        clear(kd + i);
    }
    __syncthreads();
    for (int e = tid; e < kd; e += kFinThreads) {
        const int j = e / d, m = e - j * d;
        const uint64_t tv = e == tid ? tv0 : P.sums[e] + row_sum(e);
        const double cold = e == tid ? cold0 : P.C64[e];
        const uint64_t n = nc[j];
        const int64_t q = (int64_t)(tv - n * kMagicBits);
        co[j * DS + m] = cold;
        qs[j * DS + m] = q;
        cn[j * DS + m] = n ? ((double)q * P.qinv) / (double)n : cold;
        P.sums[e] = tv;
        clear(e);
    }
    __syncthreads();
    // Per cluster, a group of 8 lanes: projection (spherical), drift, float32
    // copy, its rounding error and norm, the inertia term.
    const int g8 = tid & 7;
    for (int j0 = 0; j0 < k; j0 += kFinThreads / 8) {   // whole groups take every round
        const int j = min(j0 + tid / 8, k - 1);
        const uint64_t n = nc[j];
        double* c = cn + j * DS;
        const double* o = co + j * DS;
        auto sum8 = [&](double v) __attribute__((always_inline)) {
#pragma unroll
            for (int s = 1; s < 8; s <<= 1) v += __shfl_xor(v, s);
            return v;
        };
        double scale = 1.0;
        bool keep = n == 0;
        if (P.flags & KM_FLAG_SPHERICAL) {
            double s = 0.0;
            for (int m = g8; m < d; m += 8) s = fma(c[m], c[m], s);
            s = sum8(s);
            if (n > 0 && s > 0.0) scale = sqrt(s);
            else keep = true;
        }
        const bool mine = j0 + tid / 8 < k;   // the group's own cluster (not the repeated last)
        double dr = 0.0, de = 0.0, n2 = 0.0;
        DD term{};
        for (int m = g8; m < d; m += 8) {
            const double cold = o[m], cnew = keep ? cold : c[m] / scale;
            if (P.iterm) term = inertia_add(term, cold, n, qs[j * DS + m], P.qinv);
            const float c32 = (float)cnew;
            const double df = cnew - cold, e = (double)c32 - cnew;
            dr = fma(df, df, dr);
            de = fma(e, e, de);
            n2 = fma((double)c32, (double)c32, n2);
            if (mine) {
                c[m] = cnew;
                P.C64[j * d + m] = cnew;
                P.C32[j * d + m] = c32;
            }
        }
        if (shift) {
            n2 = 0.0;
            for (int m = g8; m < d; m += 8) {
                const double v = (double)(float)(keep ? o[m] : c[m]) - (double)P.mu[m];
                n2 = fma(v, v, n2);
            }
        }
        dr = sum8(dr);
        de = sum8(de);
        n2 = sum8(n2);
        if (P.iterm) {
#pragma unroll
            for (int s = 1; s < 8; s <<= 1) term = dd_add(term, DD{__shfl_xor(term.h, s), __shfl_xor(term.l, s)});
        }
        if (mine && g8 == 0) {
            const double fd = sqrt(dr);
            const float ec = f32_up(sqrt(de) * (1.0 + 0x1p-40));
            const double hi = (P.dhi[j] + fd * (1.0 + 0x1p-40)) * (1.0 + 0x1p-50);
            const double lo = (P.dlo[j] + fd * (1.0 - 0x1p-40)) * (1.0 - 0x1p-50);
            P.f[j] = f32_up(fd * (1.0 + 0x1p-40));
            P.ec[j] = ec;
            ecs[j] = ec;
            P.cn2[j] = (float)n2;
            P.dhi[j] = hi;
            P.dlo[j] = lo;
            P.dupf[j] = f32_up(hi);
            P.ddnf[j] = f32_down(lo);
            if (P.iterm) inertia_fixed(term, P.iscale, P.iterm + 2 * j);
        }
    }
    __syncthreads();
    // The table, 16 lanes per row: h (k_inc_vec reads it), s, and the minima
    // over each 32 centroids.
    const int g16 = tid & 15;
    for (int i0 = 0; i0 < k; i0 += kFinThreads / 16) {
        const int i = min(i0 + tid / 16, k - 1);
        const double* ci = cn + i * DS;
        float mn = INFINITY, bm[4] = {INFINITY, INFINITY, INFINITY, INFINITY};
        for (int j = g16; j < k; j += 16) {
            const double* cj = cn + j * DS;
            double a = 0.0;
            for (int m = 0; m < d; ++m) {
                const double t = ci[m] - cj[m];
                a = fma(t, t, a);
            }
            const float hv = j == i ? 0.f : f32_down(0.5 * sqrt(a) * (1.0 - 0x1p-40));
            if (j != i) mn = fminf(mn, hv);
            if (P.hm) {
#pragma unroll
                for (int b = 0; b < 4; ++b)
                    if (j >> 5 == b) bm[b] = fminf(bm[b], hv);
            }
            P.h[i * k + j] = hv;
        }
#pragma unroll
        for (int s = 1; s < 16; s <<= 1) {
            mn = fminf(mn, __shfl_xor(mn, s));
            if (P.hm) {
#pragma unroll
                for (int b = 0; b < 4; ++b) bm[b] = fminf(bm[b], __shfl_xor(bm[b], s));
            }
        }
        if (g16 == 0) {
            P.s[i] = mn;
            if (P.hm) {
#pragma unroll
                for (int b = 0; b < 4; ++b) P.hm[4 * i + b] = bm[b];
            }
        }
    }
    if (tid < 64) {   // the bookkeeping
        float em = 0.f;
        for (int j = lane; j < k; j += 64) em = fmaxf(em, ecs[j]);
#pragma unroll
        for (int s = 32; s > 0; s >>= 1) em = fmaxf(em, __shfl_xor(em, s));
        if (lane == 0) {
            st->ec_max = em;
            close_step(P, sc, NAN);
        }
        if (P.iterm) {
            __threadfence_block();
            close_inertia(P);
        }
    }
}

static int gen_finish_lds(int d, int k) { return k * (d | 1) * 24 + k * 12 + 64 + 16; }

// One block against two launches of k blocks, whole runs, two launches and one
// block: 12 steps of 3000 x 20, k = 20 (k k d = 8000) 373 and 315 us, of 395 x 27, k =
// 31 (25947) 371 and 335, of 3000 x 8, k = 64 (32768) 395 and 372; 6 steps of 3000
// x 20, k = 40 (32000) 235 and 250, x 14, k = 50 (35000) 229 and 245, x 2, k = 90
// (16200) 239 and 268, x 2, k = 181 (65522) 284 and 413.  The table's k^2 d
// differences and the k d coordinates' 18 words each are what one block has to
// do; past 64 rows its 32 groups of lanes take a third round of them.
bool gen_finish_applies(int d, int k) { return k <= 64 && k * d <= 1024 && k * k * d <= (k * d <= 512 ? 32768 : 28000); }

hipError_t launch_gen_finish(const Dev& dv, hipStream_t s) {
    hipLaunchKernelGGL(k_gen_finish, dim3(1), dim3(kFinThreads), gen_finish_lds(dv.d, dv.k), s, dv);
    return hipGetLastError();
}

template <int CB>
__global__ __launch_bounds__(256) void k_gen_unpack(const uint32_t* __restrict__ w, int64_t n, int32_t* __restrict__ a) {
    const int64_t stride = (int64_t)gridDim.x * blockDim.x;
    for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
        a[i] = state_cluster<CB>(w[i]);
}

// ---------------------------------------------------------------------------
// Dispatch

// The one-lane form costs about k (2 d + 8) vector instructions per 64
// survivors, the matrix-core form about 440 + 110 per block of 32 centroids
// plus 70 per 16 dimensions: they meet near k d = 256 (d rounded up to 4).  1M
// x 10, k = 25 took 71 us a step in the one-lane form and 56 us in the other;
// 6.6M x 8, k = 10 takes 85 us in the one-lane form.  The one-lane form also
// counts distances exactly as the MTI scan does, one centroid after another.
static int gen_mat_kb(int k) { return k <= 32 ? 1 : k <= 64 ? 2 : k <= 128 ? 4 : 8; }

int gen_waves(GenKind kind, int d, int k) { return kind == kGenMat ? gen_mat_waves(gen_mat_kb(k), d <= 32) : kGenWaves; }

GenKind gen_kind(int64_t n, int d, int k, int max_lds) {
    if (n > (int64_t)INT_MAX - kGenTile) return kGenNone;   // int32 point indices, also over the padding
    if (d <= kGenVecMaxD && k <= kGenVecMaxK && k * ((d + 3) / 4 * 4) <= kGenVecMaxKD &&
        gen_vec_lds((d + 3) / 4 * 4, d, k).bytes <= max_lds)
        return kGenVec;
    if (k <= kGenMatMaxK && d <= kGenMatMaxD && gen_mat_lds(gen_mat_kb(k), gen_waves(kGenMat, d, k), d, k).bytes <= max_lds) return kGenMat;
    return kGenNone;
}

int gen_lds_bytes(GenKind kind, int d, int k) {
    return kind == kGenVec ? gen_vec_lds((d + 3) / 4 * 4, d, k).bytes : gen_mat_lds(gen_mat_kb(k), gen_waves(kGenMat, d, k), d, k).bytes;
}

#define KM_GEN_KB(MATX, V_, O_)                                             \
    {                                                                       \
        if (kb == 1) MATX(1, V_, O_) else if (kb == 2) MATX(2, V_, O_)      \
        else if (kb == 4) MATX(4, V_, O_) else MATX(8, V_, O_)              \
    }
#define KM_GEN_CASES(VECX, MATX)                                            \
    if (kind == kGenVec) {                                                  \
        const int dp = (dv.d + 3) / 4 * 4;                                  \
        if (dp == 4) VECX(4) else if (dp == 8) VECX(8) else if (dp == 12) VECX(12) else VECX(16) \
    } else {                                                                \
        const int kb = gen_mat_kb(dv.k);                                    \
        const bool vec = dv.d % 4 == 0 && reinterpret_cast<uintptr_t>(dv.X) % 16 == 0; \
        if (vec) {                                                          \
            if (dv.d <= 32) KM_GEN_KB(MATX, true, true) else KM_GEN_KB(MATX, true, false)    \
        } else {                                                            \
            if (dv.d <= 32) KM_GEN_KB(MATX, false, true) else KM_GEN_KB(MATX, false, false)  \
        }                                                                   \
    }

const void* gen_symbol(GenKind kind, const Dev& dv) {
#define KM_V(DP_) return reinterpret_cast<const void*>(&k_inc_vec<DP_>);
#define KM_M(KB_, V_, O_) return reinterpret_cast<const void*>(&k_inc_mat<KB_, V_, O_>);
    KM_GEN_CASES(KM_V, KM_M)
#undef KM_V
#undef KM_M
}

hipError_t launch_gen(GenKind kind, const Dev& dv, int grid, int nsub, int lds_bytes, int first, int check, hipStream_t s) {
#define KM_V(DP_) { hipLaunchKernelGGL(k_inc_vec<DP_>, dim3(grid), dim3(kGenThreads), lds_bytes, s, dv, first, check, nsub); }
#define KM_M(KB_, V_, O_) { hipLaunchKernelGGL((k_inc_mat<KB_, V_, O_>), dim3(grid), dim3(64 * gen_mat_waves(KB_, O_)), lds_bytes, s, dv, first, check, nsub); }
    KM_GEN_CASES(KM_V, KM_M)
#undef KM_V
#undef KM_M
    return hipGetLastError();
}

hipError_t launch_gen_unpack(GenKind kind, const Dev& dv, int32_t* assign_out, hipStream_t s) {
    int64_t blocks = (dv.n + 255) / 256;
    if (blocks > 8192) blocks = 8192;
    if (kind == kGenMat && dv.k > 128)
        hipLaunchKernelGGL(k_gen_unpack<8>, dim3((unsigned)blocks), dim3(256), 0, s, dv.w, dv.n, assign_out);
    else
        hipLaunchKernelGGL(k_gen_unpack<7>, dim3((unsigned)blocks), dim3(256), 0, s, dv.w, dv.n, assign_out);
    return hipGetLastError();
}

}  // namespace km
