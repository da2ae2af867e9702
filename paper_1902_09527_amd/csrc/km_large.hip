// Global-memory path of the MTI k-means hot path for gfx950 (MI355X), used
// when the centroids or the per-cluster sums do not fit in LDS (large k*d,
// e.g. k = 1000, d = 256).  One iteration (one ||Lloyd's MM step, paper
// section III-B) is:
//   k_bound_large       drift-updated bound and Clause 1 (section III-C) for
//                       every point; survivors compacted into a global list;
//   k_mfma_large        distances of the survivors to all centroids on the
//                       matrix cores (128-survivor x 128-centroid work items,
//                       split-bf16 products over 16-dimension chunks streamed
//                       into LDS by direct loads, expanded form): the four
//                       smallest per survivor and centroid tile;
//   k_refine_large      per survivor, the candidates within the expanded
//                       form's error bound; a lone candidate settles it;
//   k_multi_large,
//   k_full_large        two to kMultiCand candidates: direct form and the
//                       float64 near-tie rule; more: float64 over all
//                       centroids;
//   k_hist_large        per-block cluster counts of the new assignment;
//   k_scan_large_cols,
//   k_scan_large_clusters  cluster starts and per-block write offsets;
//   k_scatter_large     point indices grouped by cluster (counting sort);
//   k_segsum_large      exact fixed-point sums over chunks of each cluster;
//   k_chunk_reduce_large  per-cluster sums and counts into the reduced row
//                       read by k_update;
//   k_centroid_table_tiled  half centroid distances for the next step;
//   k_split_rows        split operand rows of the new centroids with their
//                       squared norms and the per-centroid minimum s of the
//                       table (and, once at set-up, split rows of X).
// The order of points inside a cluster segment is not fixed, but every sum
// is an exact integer sum, so results are bitwise reproducible.
#include <float.h>
#include <limits.h>
#include <math.h>

#include "kmeans_mti.h"
#include "km_device.h"
#include "km_internal.h"

namespace km {

namespace {

constexpr int kTiTile = 16;          // centroid rows per block of the tiled centroid table
constexpr int kTiCols = kLgTableCols; // centroids per block column
constexpr int kTiK = 16;             // dimensions staged at a time
constexpr int kRefineFlush = 128;   // LDS entries of the refinement pass that trigger a flush

// Adds each of n counters (summed over the block) to its slot of the step's
// statistics, one atomic per counter and block (per-wave atomics on the same
// words serialize).  Every thread of the block calls it.
template <int N>
__device__ __forceinline__ void add_stats_block(uint64_t* total, const int (&slot)[N], uint64_t (&v)[N]) {
    __shared__ uint64_t part[N][16];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
#pragma unroll
    for (int c = 0; c < N; ++c) {
        v[c] = wave_sum_u64(v[c]);
        if (lane == 0) part[c][wave] = v[c];
    }
    __syncthreads();
    if (threadIdx.x < N) {
        uint64_t s = 0;
        for (int w = 0; w < nw; ++w) s += part[threadIdx.x][w];
        if (s) atomicAdd(reinterpret_cast<unsigned long long*>(total + slot[threadIdx.x]), (unsigned long long)s);
    }
}

// The step's per-cluster sums come from its moves (added to the running
// sums kept by k_update) when few points moved; otherwise from the counting
// sort and exact segment sums.  The first step always takes the full sums.
__device__ __forceinline__ bool large_incremental(const Dev& P, const Large& Lg) {
    return P.st->t > 0 && *Lg.nmv <= (uint32_t)Lg.mvcap;
}

}  // namespace

// ---------------------------------------------------------------------------
// Bound update and Clause 1 for every point; survivors to the global list.

__global__ __launch_bounds__(kLgBoundThreads) void k_bound_large(Dev P, Large Lg) {
    IterState* st = P.st;
    if (st->done) {
        if (blockIdx.x == 0 && threadIdx.x == 0) st->active = 0;
        return;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) st->active = 1;
    const bool first = st->t == 0;
    const bool prune = !(P.flags & KM_FLAG_NO_PRUNE);
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __shared__ uint32_t cnt[kLgBoundRounds * kLgBoundWaves], base[kLgBoundRounds * kLgBoundWaves];
    // Block b owns points [b kLgBoundSpan, (b + 1) kLgBoundSpan): the flags
    // of its rounds stay in a bit mask, the block's survivors take one atomic
    // on the list counter (few, large blocks: atomics on one counter are
    // serialized), then every survivor its place (block order, then point
    // order).
    const int64_t lo = (int64_t)blockIdx.x * kLgBoundSpan, hi = min(P.n, lo + kLgBoundSpan);
    uint64_t c1 = 0;
    uint32_t mask = 0;
#pragma unroll
    for (int r = 0; r < kLgBoundRounds; ++r) {
        const int64_t i = lo + kLgBoundThreads * r + tid;
        bool surv = false;
        if (i < hi) {
            if (first) {
                surv = true;
            } else {
                const int a = P.a[i];
                const float u = (P.u[i] + P.f[a]) * kUp;
                if (!prune || u > P.s[a]) {
                    surv = true;
                } else {
                    c1 += 1;
                    P.u[i] = u;
                }
            }
        }
        mask |= (surv ? 1u : 0u) << r;
        const uint64_t m = __ballot(surv);
        if (lane == 0) cnt[kLgBoundWaves * r + wave] = (uint32_t)__popcll(m);
    }
    __syncthreads();
    if (tid == 0) {
        uint32_t tot = 0;
        for (int q = 0; q < kLgBoundRounds * kLgBoundWaves; ++q) {
            base[q] = tot;
            tot += cnt[q];
        }
        const uint32_t b0 = tot ? atomicAdd(Lg.nsurv, tot) : 0u;
        for (int q = 0; q < kLgBoundRounds * kLgBoundWaves; ++q) base[q] += b0;
    }
    __syncthreads();
#pragma unroll
    for (int r = 0; r < kLgBoundRounds; ++r) {
        const bool surv = (mask >> r) & 1u;
        const uint64_t m = __ballot(surv);
        if (surv) {
            const int64_t i = lo + kLgBoundThreads * r + tid;
            const uint32_t pos = base[kLgBoundWaves * r + wave] + (uint32_t)__popcll(m & ((1ull << lane) - 1ull));
            Lg.surv[pos] = (int32_t)i;
            Lg.sx2[pos] = Lg.x2[i];
        }
    }
    {
        const int slot[1] = {P.k * P.d + P.k + kStClause1};
        uint64_t v[1] = {c1};
        add_stats_block<1>(P.total, slot, v);
    }
}

// ---------------------------------------------------------------------------
// Split rows of x = row - mu (rounded to float32; mu is zero unless the data lie
// far from the origin): hi = bf16(x), lo = bf16(x - hi) (both rounded to
// nearest; x - hi is exact in float32), in the chunk layout of the matrix-core operands, and
// the float32 squared norm of every row (each lane sums its dimensions in
// order, then a fixed butterfly over the wave: deterministic).  Rows from
// valid to rows are padding: zero operands, norm +inf.  One wave per row.

__global__ __launch_bounds__(256) void k_split_rows(const float* __restrict__ src, int64_t rows, int64_t valid, int d,
                                                    int nch, uint32_t* __restrict__ dst, float* __restrict__ norms,
                                                    const IterState* st, int force, const float* __restrict__ smin,
                                                    float* __restrict__ s_out, const float* __restrict__ mu) {
    if (!force && !st->active) return;
    const bool shift = st->shift != 0;
    const int lane = threadIdx.x & 63;
    const int64_t wstride = (int64_t)gridDim.x * (blockDim.x >> 6);
    for (int64_t r = (int64_t)blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); r < rows; r += wstride) {
        const bool pad = r >= valid;
        const float* x = src + (pad ? 0 : r) * d;
        uint32_t* o = dst + r * nch * 16;
        float sq = 0.f;
        for (int g = lane; g < 2 * nch; g += 64) {   // 8-dimension group g: chunk g / 2, half g % 2
            const int m0 = 8 * g;
            float v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = !pad && m0 + e < d ? x[m0 + e] : 0.f;
            if (shift) {   // uniform
#pragma unroll
                for (int e = 0; e < 8; ++e) v[e] = !pad ? v[e] - mu[m0 + e] : 0.f;   // (mu is zero past d)
            }
            uint32_t hw[4], lw[4];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                float ra, rb;
                hw[p] = split_hi(v[2 * p], v[2 * p + 1], ra, rb);
                lw[p] = split_lo(ra, rb);
                sq = fmaf(v[2 * p], v[2 * p], sq);
                sq = fmaf(v[2 * p + 1], v[2 * p + 1], sq);
            }
            uint32_t* oc = o + (g >> 1) * 16 + 4 * (g & 1);
            *reinterpret_cast<uint4*>(oc) = make_uint4(hw[0], hw[1], hw[2], hw[3]);
            *reinterpret_cast<uint4*>(oc + 8) = make_uint4(lw[0], lw[1], lw[2], lw[3]);
        }
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) sq += __shfl_xor(sq, off);
        if (lane == 0) {
            norms[r] = pad ? INFINITY : sq;
        }
        if (smin && !pad) {   // min over j != r of the half distances: the table's column minima
            float m = INFINITY;
            for (int y = lane; y < (int)((valid + kTiCols - 1) / kTiCols); y += 64)
                m = fminf(m, smin[(int64_t)y * valid + r]);
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) m = fminf(m, __shfl_xor(m, off));
            if (lane == 0) s_out[r] = m;
        }
    }
}

// ---------------------------------------------------------------------------
// Dense survivor distances on the matrix cores.  A work item is one tile of
// kLgM = 128 survivors against one tile of kLgN = 256 centroids; wave
// (wr, wc) of the block owns centroid rows 128 wr .. +127 and survivor
// columns 64 wc .. +63, eight 32x32 float32 accumulators.  Each product x.c
// is formed from the split operands as hi.hi + hi.lo + lo.hi: three bf16
// products on v_mfma_f32_32x32x16_bf16 (16 dimensions each) in place of
// eight float32 ones, with the dropped lo.lo term and the accumulation
// inside the error bound used by the refinement pass.
//
// The 16-dimension chunks of a block's items form one stream that runs
// kLgStages - 1 chunks ahead of the products, across item boundaries (the
// next item's first chunks load during the current item's selection).  They
// go from the split rows straight into a ring of kLgStages LDS stages by
// global_load_lds_dwordx4 (no registers held); a stage is two tiles (256
// and 128 rows x 64 bytes) in 1 KB groups of 16 rows, the four 16-byte
// pieces of each row permuted by lg_swz so that the operand reads of eight
// (and of sixteen) consecutive lanes fall on distinct banks.  Loads return
// in order, so chunk g has landed once at most the loads issued after it
// are outstanding.  Loads in flight per CU are bounded by LDS, so the tile
// is wide: 24 products per wave and chunk for 24 KB.
//
// Work items are ordered so that the nct items of a survivor tile carry
// indices congruent modulo 8: with a resident grid whose size is a multiple
// of 8, they run at the same time on one XCD and its L2 serves the survivor
// rows to all of them (each row leaves HBM about once per step).
//
// Selection: each expanded distance |x|^2 + |c|^2 - 2 x.c is clamped at 0
// (the true distance is >= 0, so the error bound still holds) and packed
// with its centroid into one ordered 32-bit key: the float's bits with the
// low 8 bits (6 within a lane's list) replaced by the centroid's place in
// the item, which lowers the value by less than 2^-15 of itself.  A lane
// keeps, per survivor column, the four smallest keys by min and med3
// (branch-free), and writes the four, with the centroid's place in the item,
// to the candidate buffer.

__device__ __forceinline__ int lg_swz(int rho) { return ((rho >> 2) & 3) ^ (((rho >> 1) & 1) << 1); }

__device__ __forceinline__ uint32_t med3u(uint32_t a, uint32_t b, uint32_t c) {
    uint32_t r;
    asm("v_med3_u32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// Insert key v into the ascending 4-list L.
__device__ __forceinline__ void key4_insert(uint32_t (&L)[4], uint32_t v) {
    const uint32_t l0 = min(L[0], v), l1 = med3u(L[0], L[1], v), l2 = med3u(L[1], L[2], v),
                   l3 = med3u(L[2], L[3], v);
    L[0] = l0;
    L[1] = l1;
    L[2] = l2;
    L[3] = l3;
}

// Sort 4 keys ascending (five compare-exchanges).
__device__ __forceinline__ void sort4(uint32_t (&L)[4]) {
    auto cx = [&](int i, int j) __attribute__((always_inline)) {
        const uint32_t a = L[i], b = L[j];
        L[i] = min(a, b);
        L[j] = max(a, b);
    };
    cx(0, 1);
    cx(2, 3);
    cx(0, 2);
    cx(1, 3);
    cx(1, 2);
}

typedef __attribute__((address_space(3))) void* lds_ptr;

__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void k_mfma_large(Dev P, Large Lg) {
    IterState* st = P.st;
    if (!st->active) return;
    const int ns = (int)*Lg.nsurv;
    const int nch = Lg.nch, nct = Lg.nct;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, col = lane & 31, half = lane >> 5;
    const int wr = wave >> 1, wc = wave & 1;
    extern __shared__ __align__(16) unsigned char smem[];
    // [2][kLgN + kLgM] by item parity: |c|^2 of the centroid tile, then |x|^2 of the survivors.
    float* nrm = reinterpret_cast<float*>(smem + kLgStages * kLgStageBytes);
    int32_t* meta = reinterpret_cast<int32_t*>(nrm + 2 * (kLgN + kLgM));   // [2][4 waves][64]: survivor rows

    const int nst = (ns + kLgM - 1) / kLgM;
    const int per_round = 8 * nct;
    const int64_t nitems = (int64_t)((nst + 7) / 8) * per_round;
    const int G = gridDim.x;
    auto tile_of = [&](int64_t w, int& s0, int& n0) __attribute__((always_inline)) {
        const int64_t r = w / per_round;
        const int rem = (int)(w - r * per_round);
        s0 = (int)(r * 8 + (rem & 7)) * kLgM;
        n0 = (rem >> 3) * kLgN;
    };
    auto next_valid = [&](int64_t w) __attribute__((always_inline)) {
        for (; w < nitems; w += G) {
            int s0, n0;
            tile_of(w, s0, n0);
            if (s0 < ns) break;
        }
        return w;
    };

    // DMA role of this lane in a 16-row group: row rho, LDS slot lane, piece
    // (lane % 4) ^ lg_swz(rho) of the row's chunk.  This wave streams
    // centroid rows 64 wave .. +63 (groups 4 wave .. 4 wave + 3) and
    // survivor rows 32 wave .. +31 (groups 2 wave, 2 wave + 1).
    const int rho = lane >> 2, piece = (lane & 3) ^ lg_swz(rho);
    const int sr0 = 32 * wave + rho;
    // Operand reads of lane (col, half): row col of a 32-row block, pieces
    // half (hi) and 2 + half (lo), at these offsets in its 1 KB group.
    const int rr = col & 15;
    const int offh = 16 * (4 * rr + (half ^ lg_swz(rr))), offl = 16 * (4 * rr + ((2 + half) ^ lg_swz(rr)));
    const int ga = (8 * wr + (col >> 4)) * 1024, gb = kLgN * 64 + (4 * wc + (col >> 4)) * 1024;
    const int64_t rowb = (int64_t)nch * 64;   // bytes per split row
    const unsigned char* csb = reinterpret_cast<const unsigned char*>(Lg.cs) + 16 * piece;
    const unsigned char* xsb = reinterpret_cast<const unsigned char*>(Lg.xs) + 16 * piece;
    const float* __restrict__ cn2p = Lg.cn2p;
    const float* __restrict__ sx2 = Lg.sx2;
    const int32_t* __restrict__ surv = Lg.surv;
    // Item metadata goes to LDS by direct loads too (nothing loaded is held
    // in registers across the loop): the survivor rows of this wave's two
    // row groups (lane l: row 32 wave + l % 32; rows past the list repeat
    // the first), the 256 centroid squared norms (64 per wave) and the 128
    // survivor squared norms (waves 0-1; survivors past the list read the
    // first).
    auto load_meta = [&](int s0, int par) __attribute__((always_inline)) {
        const int r = 32 * wave + (lane & 31);
        __builtin_amdgcn_global_load_lds(surv + s0 + (s0 + r < ns ? r : 0), (lds_ptr)(meta + par * 256 + wave * 64),
                                         4, 0, 0);
    };
    auto load_norms = [&](int s0, int n0, int par) __attribute__((always_inline)) {
        float* dst = nrm + par * (kLgN + kLgM) + 64 * wave;
        __builtin_amdgcn_global_load_lds(cn2p + n0 + tid, (lds_ptr)(dst), 4, 0, 0);
        if (wave < 2) {
            const int sl = tid;
            __builtin_amdgcn_global_load_lds(sx2 + s0 + (s0 + sl < ns ? sl : 0), (lds_ptr)(dst + kLgN), 4, 0, 0);
        }
    };

    // Issue cursor: item wi, its next chunk ci, its parity ipar; wn the item
    // after it.
    int64_t wi = next_valid(blockIdx.x);
    if (wi >= nitems) return;
    int is0, in0;
    tile_of(wi, is0, in0);
    int64_t wn = next_valid(wi + G);
    const unsigned char *pa, *pb0, *pb1;
    {
        const int rows = min(kLgM, ns - is0);
        const int q0 = surv[is0 + (sr0 < rows ? sr0 : 0)], q1 = surv[is0 + (sr0 + 16 < rows ? sr0 + 16 : 0)];
        pa = csb + (int64_t)(in0 + 64 * wave + rho) * rowb;
        pb0 = xsb + (int64_t)q0 * rowb;
        pb1 = xsb + (int64_t)q1 * rowb;
    }
    int ipar = 0;
    load_norms(is0, in0, 0);
    if (wn < nitems) {
        int s1, n1;
        tile_of(wn, s1, n1);
        load_meta(s1, 1);
    }
    int ci = 0;
    bool more = true;
    int64_t issued = 0;
    auto issue_one = [&]() __attribute__((always_inline)) {
        if (ci == nch) {   // the issue cursor enters the next item (its survivor rows landed long ago)
            ci = 0;
            wi = wn;
            ipar ^= 1;
            tile_of(wi, is0, in0);
            const int* mrow = meta + ipar * 256 + wave * 64;
            const int q0 = mrow[rho], q1 = mrow[16 + rho];
            pa = csb + (int64_t)(in0 + 64 * wave + rho) * rowb;
            pb0 = xsb + (int64_t)q0 * rowb;
            pb1 = xsb + (int64_t)q1 * rowb;
            load_norms(is0, in0, ipar);
            wn = next_valid(wn + G);
            if (wn < nitems) {
                int s1, n1;
                tile_of(wn, s1, n1);
                load_meta(s1, ipar ^ 1);
            }
        }
        unsigned char* base = smem + (int)(issued % kLgStages) * kLgStageBytes;
        const int64_t o = (int64_t)ci * 64;
#pragma unroll
        for (int t = 0; t < 4; ++t)
            __builtin_amdgcn_global_load_lds(pa + 16 * t * rowb + o, (lds_ptr)(base + (4 * wave + t) * 1024), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(pb0 + o, (lds_ptr)(base + kLgN * 64 + 2 * wave * 1024), 16, 0, 0);
        __builtin_amdgcn_global_load_lds(pb1 + o, (lds_ptr)(base + kLgN * 64 + (2 * wave + 1) * 1024), 16, 0, 0);
        ++issued;
        if (++ci == nch && wn >= nitems) more = false;
    };
    // Compute cursor: item wcur (tile cs0, cn0), chunk cc, parity par.
    int64_t wcur = wi;
    int cs0 = is0, cn0 = in0, cc = 0, par = 0;
    const int ahead = min(kLgStages - 1, nch);
    for (int e = 0; e < ahead && more; ++e) issue_one();

    f32x16 acc[4][2];
#pragma unroll
    for (int a = 0; a < 4; ++a)
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.f;
    for (int64_t g = 0; g < issued; ++g) {
        // Chunk g has landed once at most the chunks issued after it (six
        // loads each per wave) are outstanding (with it every older load:
        // the item's norms and the next item's survivor rows); the barrier
        // then makes every wave's part visible and frees the stage of chunk
        // g - 1 for the load issued next.
        if (issued - 1 - g >= 1)
            asm volatile("s_waitcnt vmcnt(6) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        else
            asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (more) issue_one();
        const unsigned char* S = smem + (int)(g % kLgStages) * kLgStageBytes;
        bf16x8 ah[4], al[4], bh[2], bl[2];
#pragma unroll
        for (int a = 0; a < 4; ++a) {
            ah[a] = *reinterpret_cast<const bf16x8*>(S + ga + 2048 * a + offh);
            al[a] = *reinterpret_cast<const bf16x8*>(S + ga + 2048 * a + offl);
        }
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            bh[b] = *reinterpret_cast<const bf16x8*>(S + gb + 2048 * b + offh);
            bl[b] = *reinterpret_cast<const bf16x8*>(S + gb + 2048 * b + offl);
        }
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[a], bh[b], acc[a][b], 0, 0, 0);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ah[a], bl[b], acc[a][b], 0, 0, 0);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
                acc[a][b] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(al[a], bh[b], acc[a][b], 0, 0, 0);
        if (++cc < nch) continue;

        // Item done.  Register e of accumulator [a][cb]: centroid cn0 + 128 wr
        // + 32 a + 8 (e / 4) + 4 half + e % 4, survivor column 64 wc + 32 cb +
        // col; its place in the lane's list: 16 a + 4 (e / 4) + e % 4.
        const float* nr = nrm + par * (kLgN + kLgM);
        uint32_t KP[2][4];
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            uint32_t K[4] = {0xffffffffu, 0xffffffffu, 0xffffffffu, 0xffffffffu};
            const float xa = nr[kLgN + 64 * wc + 32 * cb + col];
#pragma unroll
            for (int a = 0; a < 4; ++a)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 cn = *reinterpret_cast<const f32x4*>(nr + 128 * wr + 32 * a + 8 * q + 4 * half);
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const float v = fmaxf(fmaf(-2.f, acc[a][cb][4 * q + e], xa + cn[e]), 0.f);
                        key4_insert(K, (__float_as_uint(v) & ~63u) | (uint32_t)(16 * a + 4 * q + e));
                    }
                }
            // Place in the item: 128 wr + 32 a + 8 q + 4 half + e.  Clearing
            // two more value bits can reorder the list: sort it again.
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint32_t lo = K[q] & 63u;
                const uint32_t place = 128 * wr + 4 * half + (lo & 3u) + 8 * ((lo >> 2) & 3u) + 32 * (lo >> 4);
                KP[cb][q] = (K[q] & ~255u) | place;
            }
            sort4(KP[cb]);
        }
        // Both half-waves' lists of a column go out: four keys for each 64
        // centroids (merged to four for 128 they overflowed where several
        // centroids share a component; the keys alone are half the words of
        // (value, centroid) pairs).
        const int rows = min(kLgM, ns - cs0);
#pragma unroll
        for (int cb = 0; cb < 2; ++cb) {
            const int sc = 64 * wc + 32 * cb + col;
            if (sc < rows)
                reinterpret_cast<uint4*>(Lg.cand)[(((int64_t)(cs0 + sc) * nct + cn0 / kLgN) * 2 + wr) * 2 + half] =
                    make_uint4(KP[cb][0], KP[cb][1], KP[cb][2], KP[cb][3]);
        }
        // Next item of the compute cursor.
        cc = 0;
        par ^= 1;
        wcur = next_valid(wcur + G);
        if (wcur < nitems) tile_of(wcur, cs0, cn0);
#pragma unroll
        for (int a = 0; a < 4; ++a)
#pragma unroll
            for (int b = 0; b < 2; ++b)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[a][b][e] = 0.f;
    }
}

// ---------------------------------------------------------------------------
// Refinement of every survivor by a thread pair (each reading half of its
// candidate lists: the four smallest keys of each 64 centroids): only
// centroids within twice the expanded form's error bound of the smallest can be the
// nearest.  A lone candidate is the assignment, its bound taken from the
// expanded value; two to kMultiCand go to k_multi_large (direct form, float64
// near-tie rule); a survivor with more, or with four from one list (more
// of its 64 centroids may lie outside it), goes to k_full_large, which decides it in
// float64 over all centroids: 2 MB of centroids read per survivor at k = 1000,
// d = 256, so that it has to stay rare.  Where several centroids share a
// component (uneven weights, start rows drawn from the data) four to six
// candidates are common; sent to the full decision they made a step of 700K x
// 128, k = 56 take 1.5 ms and one of 2M x 256, k = 1000 with Dirichlet weights
// 154 ms (now 24 ms), one of 400K x 128, k = 200 3.5 ms (now 0.35 ms).
//
// Error bounds (x and c the float32 row and centroid, less mu).  What decides between
// centroids is |c|^2 - 2 x.c (a row's own norm shifts all of them alike):
//   - the split product: dropping lo.lo and the residuals of the two
//     roundings costs at most 3.04 2^-16 |x_m| |c_m| per dimension;
//   - the bf16 products are exact in float32 and each instruction adds 16
//     of them to its accumulator; assuming an error of at most 18 units of
//     2^-23 relative to |C| + sum |p| per instruction (true of sequential
//     float32 additions, rounded or truncated, and of one alignment of all
//     17 addends to the largest), the 3 ceil(d/16) instructions of a
//     product contribute at most 6.9 d' 2^-24 sum_m |x_m| |c_m|, d' = 16
//     ceil(d / 16);
//   - |c|^2 summed in float32: (d / 64 + 16) 2^-24 |c|^2 (lanes share the
//     dimensions), at most (d + 8) 2^-24 |c|^2; two additions and the norm's
//     rounding at the magnitude of the values: 4 2^-24 R^2, R = |x| + max |c|;
//     the roundings of row - mu and centroid - mu, 2^-24 of each, move the
//     squared distance by 2 2^-24 R^2;
//   so a value is within e = (d + 8) 2^-24 max |c|^2 + 6 2^-24 R^2 +
//   2 (778 + 6.9 d') 2^-24 |x| max |c| of the row's common offset, plus an
//   absolute 2^-100 (1 + R) for bf16 values below the normal range.
// The packed key lowers a value v by less than 2^-15 of itself: the key of
// every centroid that can be nearest is at most (T0 (1 + 2^-15) + 2 e), T0 the
// smallest key, itself lowered (T0 is a squared distance, far below R^2 where
// rows are near their centroid; with 2^-15 R^2 instead, 700K x 128, k = 56 sent
// so many survivors to the full decision that it took 1 ms a step).  The
// bound of a lone candidate adds the row's norm, (d + 8) 2^-24 |x|^2.  Rows with
// |x|^2 or R out of range (non-finite data) are decided in float64 over all
// centroids.

__global__ __launch_bounds__(256) void k_refine_large(Dev P, Large Lg) {
    IterState* st = P.st;
    if (!st->active) return;
    const int k = P.k, d = P.d, nct = Lg.nct;
    const bool first = st->t == 0;
    const uint32_t ns = *Lg.nsurv;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __shared__ float red[4];
    float m2 = 0.f;
    for (int j = tid; j < k; j += blockDim.x) {
        const float v = P.cn2[j];
        m2 = fmaxf(m2, v <= FLT_MAX ? v : INFINITY);   // a non-finite centroid: every row in float64
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) m2 = fmaxf(m2, __shfl_xor(m2, off));
    if (lane == 0) red[wave] = m2;
    __syncthreads();
    const float cnmax = sqrtf(fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]))) * kUp;
    const float ecm = st->ec_max;
    const float gexp = (float)(d + 8) * 0x1p-24f;
    const float gsp2 = 2.f * (778.f + 6.9f * (float)(16 * Lg.nch)) * 0x1p-24f * (1.f + 0x1p-10f);
    uint64_t my_changed = 0, my_comp = 0;
    // A group of lps lanes (a power of two, 2 nct or more up to 64) shares a
    // survivor, a lane per two candidate lists: one coalesced read of its
    // keys.
    int lps = 4;
    while (lps < 2 * nct && lps < 64) lps *= 2;
    const int np = 2 * nct;   // pairs of lists
    const int gl = tid & (lps - 1), per = 256 / lps;
    const uint64_t gmask = (lps == 64 ? ~0ull : (1ull << lps) - 1ull) << (lane & ~(lps - 1));
    const uint64_t below = gmask & ((1ull << lane) - 1ull);
    // Queued survivors and moves gather in LDS and go to the global lists
    // with one atomic per flush of up to 2 kRefineFlush entries (a global
    // counter per wave would take one atomic per 64 survivors).
    // A queued survivor: its list entry, and the ids of its candidates (0xffff
    // past them).  The lanes of its group write disjoint words, so nothing
    // orders their stores before the barrier of the flush.
    __shared__ int qc[2 * kRefineFlush];
    __shared__ uint16_t qid[2 * kRefineFlush][kMultiCand];
    __shared__ int4 mb[2 * kRefineFlush];
    __shared__ uint32_t nqb, nmb, gq, gm;
    if (tid == 0) {
        nqb = 0;
        nmb = 0;
    }
    __syncthreads();
    auto flush = [&](bool all) __attribute__((always_inline)) {
        __syncthreads();
        const uint32_t cq = nqb, cm = nmb;
        const bool fq = cq >= (all ? 1u : (uint32_t)kRefineFlush), fm = cm >= (all ? 1u : (uint32_t)kRefineFlush);
        if (tid == 0) {
            if (fq) gq = atomicAdd(Lg.nmq, cq);
            if (fm) gm = atomicAdd(Lg.nmv, cm);
        }
        __syncthreads();
        if (fq)
            for (uint32_t e = tid; e < cq; e += blockDim.x) {
                auto two = [&](int t) { return (int)((uint32_t)qid[e][t] | (uint32_t)qid[e][t + 1] << 16); };
                Lg.mq[gq + e] = make_int4(qc[e], two(0), two(2), two(4));
            }
        if (fm)
            for (uint32_t e = tid; e < cm; e += blockDim.x)
                if (gm + e < (uint32_t)Lg.mvcap) Lg.mv[gm + e] = mb[e];
        __syncthreads();
        if (tid == 0) {
            if (fq) nqb = 0;
            if (fm) nmb = 0;
        }
        __syncthreads();
    };

    const bool rec_moves = !first;
    // A block takes runs of kRefineFlush list entries (rpf rounds), neighbours
    // in the list being neighbours in the point arrays.  A round's loads are
    // requested a round ahead (two ahead took as long); the buffers are looked
    // at (behind barriers) once per run, which appends at most kRefineFlush
    // entries.
    struct Next {
        uint4 v[2];
        int64_t i;
        float x2;
        int inc;
    } nx;
    // Lists 2 l and 2 l + 1 of a survivor (none past its np pairs).
    auto pair_at = [&](const uint4* cl, int l, uint4 (&v)[2]) __attribute__((always_inline)) {
        const uint4 none = make_uint4(~0u, ~0u, ~0u, ~0u);
        v[0] = l < np ? cl[2 * l] : none;
        v[1] = l < np ? cl[2 * l + 1] : none;
    };
    const int rpf = kRefineFlush / per;
    auto entry = [&](int64_t c0) __attribute__((always_inline)) { return min(c0 + tid / lps, (int64_t)ns - 1); };
    int32_t i2 = 0;   // the point of the round after the next
    auto fetch = [&](int64_t c0) __attribute__((always_inline)) {
        const int64_t cc = entry(c0);
        // the survivor's 4 nct lists (ascending keys; list l covers half
        // (l / 2) % 2 of centroid tile l / 4)
        pair_at(reinterpret_cast<const uint4*>(Lg.cand) + cc * nct * 4, gl, nx.v);
        nx.i = i2;
        nx.x2 = Lg.sx2[cc];
        nx.inc = first ? -1 : P.a[i2];
    };
    // First entry of this block's round r.
    auto start_of = [&](int64_t r) __attribute__((always_inline)) {
        return ((int64_t)blockIdx.x + r / rpf * gridDim.x) * kRefineFlush + r % rpf * per;
    };
    int64_t round = 0;
    if (start_of(0) < (int64_t)ns) {
        i2 = Lg.surv[entry(start_of(0))];
        fetch(start_of(0));
        i2 = Lg.surv[entry(start_of(1))];
    }
    for (int64_t c0 = start_of(0); start_of(round / rpf * rpf) < (int64_t)ns; c0 = start_of(++round)) {
        const int64_t c = c0 + tid / lps;
        const bool live = c < (int64_t)ns, lead = live && gl == 0;
        const uint4* cl = reinterpret_cast<const uint4*>(Lg.cand) + (live ? c : (int64_t)ns - 1) * nct * 4;
        uint4 v[2] = {nx.v[0], nx.v[1]};
        const int64_t i = nx.i;
        const float x2 = nx.x2;
        const int inc = nx.inc;
        fetch(start_of(round + 1));
        i2 = Lg.surv[entry(start_of(round + 2))];
        // The smallest key of all.
        uint32_t k0 = min(v[0].x, v[1].x);
        for (int l = gl + 64; l < np; l += 64) k0 = min(k0, min(cl[2 * l].x, cl[2 * l + 1].x));   // k > 8192
        for (int o = 1; o < lps; o <<= 1) k0 = min(k0, __shfl_xor(k0, o));
        const float T0 = __uint_as_float(k0 & ~255u);
        const float xn = sqrtf(fmaxf(x2, 0.f)) * kUp;
        const float R = xn + cnmax;
        const float e1 = (gexp * cnmax * cnmax + 0x1.8p-22f * R * R + gsp2 * xn * cnmax + 4.f * R * ecm +
                          2.f * ecm * ecm + 0x1p-100f * (1.f + R)) * kUp;
        const float thr = (T0 * (1.f + 0x1.1p-15f) + 2.f * e1) * kUp;
        // Only centroids whose expanded distance lies within thr of the
        // smallest can be the nearest: any other one is certified farther
        // than the smallest's centroid.  A list whose four keys all lie
        // within thr may have left more out.
        const bool wild = !(x2 <= 0x1p120f) || !(R <= 0x1p60f);
        const uint32_t kthr = __float_as_uint(thr);   // thr >= 0: keys order as values
        auto within = [&](uint32_t key) __attribute__((always_inline)) { return (key & ~255u) <= kthr; };
        int nq = 0;
        bool cut = false;
        auto count = [&](const uint4 (&u)[2]) __attribute__((always_inline)) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                const uint64_t last = __ballot(within(u[h].w)) & gmask;
                nq += __popcll(__ballot(within(u[h].x)) & gmask) + __popcll(__ballot(within(u[h].y)) & gmask) +
                      __popcll(__ballot(within(u[h].z)) & gmask) + __popcll(last);
                cut |= last != 0;
            }
        };
        count(v);
        for (int l = gl + 64; l - gl < np; l += 64) {   // k > 8192
            uint4 u[2];
            pair_at(cl, l, u);
            count(u);
        }
        const bool full = wild || cut || nq > kMultiCand || nq == 0;
        // One candidate is the nearest centroid (every other one is certified
        // farther): as on the LDS paths, its bound then comes from its
        // expanded value and the error bound, without the direct form (kept
        // when statistics are gathered: their Clause-1 counts are then those
        // of the direct form's bounds).  Otherwise the survivor and its
        // candidates go to k_multi_large.
        const bool single = !full && nq == 1 && !(P.flags & KM_FLAG_STATS);
        const bool queued = live && !full && !single;
        if (lead) my_comp += (uint64_t)k;
        if (full && lead) {
            Lg.fq[atomicAdd(Lg.nfull, 1u)] = (int32_t)c;
        }
        int b = -1;
        if (live && single) {   // from the lane that holds it
            int at = v[0].x == k0 ? 2 * gl : v[1].x == k0 ? 2 * gl + 1 : -1;
            for (int l = gl + 64; l < np; l += 64)   // k > 8192
                at = cl[2 * l].x == k0 ? 2 * l : cl[2 * l + 1].x == k0 ? 2 * l + 1 : at;
            const uint64_t own = __ballot(at >= 0) & gmask;
            b = (int)__shfl((uint32_t)(at / 4 * kLgN) + (k0 & 255u), __builtin_ctzll(own));
        }
        if (lead && single) {
            const float ub = __builtin_amdgcn_sqrtf(fmaxf(T0 * (1.f + 0x1.1p-15f) + e1 + gexp * x2, 0.f)) *
                             (1.0f + 0x1p-20f) * kUp;
            if (b != inc) {
                P.a[i] = b;
                my_changed += 1;
                if (rec_moves) mb[atomicAdd(&nmb, 1u)] = make_int4((int)i, inc, b, 0);
            }
            P.u[i] = ub;
        }
        if (queued) {   // the group's lanes append the ids they hold, the leader the rest of the entry
            uint32_t e = 0;
            if (lead) {
                e = atomicAdd(&nqb, 1u);
                qc[e] = (int)c;
                for (int t = nq; t < kMultiCand; ++t) qid[e][t] = 0xffffu;
            }
            e = __shfl(e, lane & ~(lps - 1));
            uint16_t* ids = qid[e];
            int done = 0;
            auto put = [&](uint32_t key, int list) __attribute__((always_inline)) {
                const uint64_t hm = __ballot(within(key));
                if (within(key)) ids[done + __popcll(hm & below)] = (uint16_t)(list / 4 * kLgN + (int)(key & 255u));
                done += __popcll(hm & gmask);
            };
            for (int l = gl; l - gl < np; l += 64) {
                uint4 u[2] = {v[0], v[1]};
                if (l != gl) pair_at(cl, l, u);
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    put(u[h].x, 2 * l + h);
                    put(u[h].y, 2 * l + h);
                    put(u[h].z, 2 * l + h);
                    put(u[h].w, 2 * l + h);
                }
            }
        }
        if (round % rpf == rpf - 1) flush(false);
    }
    flush(true);
    {
        const int base = k * d + k;
        const int slot[2] = {base + kStChanged, base + kStComputed};
        uint64_t v[2] = {my_changed, my_comp};
        add_stats_block<2>(P.total, slot, v);
    }
}

// ---------------------------------------------------------------------------
// Survivors with two to kMultiCand candidates inside the bound, one wave each:
// the candidates' direct-form float32 distances (lanes over the dimensions,
// coalesced rows, a fixed butterfly: the float32 error bound holds for any
// summation order), the nearest with the incumbent winning ties, and when
// the two smallest lie within the float32 band the float64 decision with
// the oracle's rule (smaller distance, then the incumbent, then the lower
// index).  With statistics every survivor comes here (direct-form bounds).

__global__ __launch_bounds__(256) void k_multi_large(Dev P, Large Lg) {
    IterState* st = P.st;
    if (!st->active) return;
    const int k = P.k, d = P.d, lane = threadIdx.x & 63;
    const bool first = st->t == 0;
    const bool rec_moves = !first;
    const float gamma = P.gamma, ecm = st->ec_max;
    const uint32_t nq_all = *Lg.nmq;
    const bool vec = (d & 3) == 0;
    uint64_t my_changed = 0, my_rc = 0;
    for (uint32_t q = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); q < nq_all;
         q += gridDim.x * (blockDim.x >> 6)) {
        const int4 e = Lg.mq[q];
        const uint32_t ids[3] = {(uint32_t)e.y, (uint32_t)e.z, (uint32_t)e.w};
        auto js = [&](int t) __attribute__((always_inline)) {
            const uint32_t v = t < 2 ? ids[0] : t < 4 ? ids[1] : ids[2];
            return (int)(t & 1 ? v >> 16 : v & 0xffffu);
        };
        int nq = 0;
        while (nq < kMultiCand && js(nq) != 0xffff) ++nq;   // uniform in the wave
        const int64_t i = Lg.surv[e.x];
        const float* xr = P.X + i * d;
        const int inc = first ? -1 : P.a[i];
        auto dist32 = [&](int j) __attribute__((always_inline)) {
            const float* cr = P.C32 + (int64_t)j * d;
            float acc = 0.f;
            if (vec) {
                for (int m = 4 * lane; m < d; m += 256) {
                    const f32x4 xv = *reinterpret_cast<const f32x4*>(xr + m);
                    const f32x4 cv = *reinterpret_cast<const f32x4*>(cr + m);
                    const float t0 = xv.x - cv.x, t1 = xv.y - cv.y, t2 = xv.z - cv.z, t3 = xv.w - cv.w;
                    acc = fmaf(t0, t0, acc);
                    acc = fmaf(t1, t1, acc);
                    acc = fmaf(t2, t2, acc);
                    acc = fmaf(t3, t3, acc);
                }
            } else {
                for (int m = lane; m < d; m += 64) {
                    const float t = xr[m] - cr[m];
                    acc = fmaf(t, t, acc);
                }
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
            return acc;
        };
        auto dist64 = [&](int j) __attribute__((always_inline)) {
            const double* cr = P.C64 + (int64_t)j * d;
            double acc = 0.0;
            for (int m = lane; m < d; m += 64) {
                const double t = (double)xr[m] - cr[m];
                acc = fma(t, t, acc);
            }
#pragma unroll
            for (int off = 32; off > 0; off >>= 1) acc += __shfl_xor(acc, off);
            return acc;
        };
        float d1 = INFINITY, d2 = INFINITY;
        int rk1 = INT_MAX, j1 = 0;
        for (int t = 0; t < nq; ++t) {
            const int j = js(t);
            const float Dd = dist32(j);
            const int rk = j == inc ? -1 : j;
            if (Dd < d1 || (Dd == d1 && rk < rk1)) {
                d2 = d1;
                d1 = Dd;
                rk1 = rk;
                j1 = j;
            } else if (Dd < d2) {
                d2 = Dd;
            }
        }
        bool re = false;
        if (d2 != INFINITY) {
            const float band = 2.f * gamma * (d1 + d2) + 4.f * (sqrtf(d1) + sqrtf(d2)) * ecm + 8.f * ecm * ecm;
            re = d2 - d1 <= band;
        }
        int b = j1;
        float ub = upper_bound(d1, P.ec[j1], gamma);
        if (re) {
            double Dbb = INFINITY, D2 = INFINITY;
            int bb = -1, kb = INT_MAX;
            auto take64 = [&](double D, int rk, int j) __attribute__((always_inline)) {
                if (D < Dbb || (D == Dbb && rk < kb)) {
                    Dbb = D;
                    bb = j;
                    kb = rk;
                }
            };
            for (int t = 0; t < nq; ++t) {
                const int j = js(t);
                const double Dj = dist64(j);
                D2 = fmin(D2, fmax(Dj, Dbb));
                take64(Dj, j == inc ? -1 : j, j);
            }
            if (!(D2 - Dbb > 0x1p-40 * D2)) {
                // within the rounding of the sums (two orders differ by 2 (d +
                // 6) 2^-53): summed over the dimensions in order, a lane per
                // candidate, as on the other paths, so that rows at equal
                // distances from two centroids fall alike on all of them
                Dbb = INFINITY;
                bb = -1;
                kb = INT_MAX;
                if (lane < nq) {
                    const int j = js(lane);
                    take64(sqd64(xr, P.C64 + (int64_t)j * d, d), j == inc ? -1 : j, j);
                }
#pragma unroll
                for (int o = 4; o > 0; o >>= 1) take64(__shfl_xor(Dbb, o), __shfl_xor(kb, o), __shfl_xor(bb, o));
            }
            b = bb < 0 ? 0 : bb;
            ub = f32_up(sqrt(Dbb) * (1.0 + 0x1p-40));
        }
        if (lane == 0) {
            if (b != inc) {
                P.a[i] = b;
                my_changed += 1;
                if (rec_moves) {
                    const uint32_t qm = atomicAdd(Lg.nmv, 1u);
                    if (qm < (uint32_t)Lg.mvcap) Lg.mv[qm] = make_int4((int)i, inc, b, 0);
                }
            }
            P.u[i] = ub;
            my_rc += re ? 1 : 0;
        }
    }
    {
        const int base = k * d + k;
        const int slot[2] = {base + kStChanged, base + kStRecheck};
        uint64_t v[2] = {my_changed, my_rc};
        add_stats_block<2>(P.total, slot, v);
    }
}

// ---------------------------------------------------------------------------
// Decision over all centroids for the queued survivors, in float64.  The first
// kFullCap of them are split over kFullSplit blocks, each taking a range of
// centroids (the row in LDS as float64, one centroid per thread, its
// distance summed over the dimensions in order) and writing its best under
// the oracle's rule (smaller distance, then the incumbent, then the lower
// index); the block that finishes a survivor last (a counter per survivor
// behind a fence) combines the ranges and writes the decision.  Survivors
// past kFullCap take one block over all centroids.
//
// Many narrow rows (d <= kFullLaneD, more than kFullLaneRows k of them) take a lane
// each: the direct float32 form over all centroids, as the general kernel
// scans, and float64 only for the near ties.  Duplicate centroids and centroids
// closer than the split products tell apart send most survivors here: 50K x 1,
// k = 500 took 813 us a step with a block each, 280 with a lane each (196 on the
// general kernel).  A block per row costs about 2 us of one of 1024 blocks, the
// scan about 0.1 us a centroid however many rows there are: 8 rows per centroid
// is where a split row's 8 blocks and the scan take as long.

__global__ __launch_bounds__(256) void k_full_large(Dev P, Large Lg) {
    IterState* st = P.st;
    if (!st->active) return;
    const int k = P.k, d = P.d;
    const bool first = st->t == 0;
    const bool rec_moves = !first;
    const uint32_t nf = *Lg.nfull;
    const uint32_t nsplit = min(nf, (uint32_t)kFullCap);
    const int kr = (k + kFullSplit - 1) / kFullSplit;
    extern __shared__ __align__(16) unsigned char smem[];
    double* xd = reinterpret_cast<double*>(smem);   // [d]
    __shared__ double rD[256];
    __shared__ int rJ[256], rK[256];
    __shared__ uint32_t last;
    const int tid = threadIdx.x;
    uint64_t my_changed = 0;
    auto decide = [&](int64_t i, int inc, double D, int bj) __attribute__((always_inline)) {
        const int b = bj < 0 ? 0 : bj;
        if (b != inc) {
            P.a[i] = b;
            my_changed += 1;
            if (rec_moves) {
                const uint32_t qm = atomicAdd(Lg.nmv, 1u);
                if (qm < (uint32_t)Lg.mvcap) Lg.mv[qm] = make_int4((int)i, inc, b, 0);
            }
        }
        P.u[i] = f32_up(sqrt(D) * (1.0 + 0x1p-40));
    };
    if (d <= kFullLaneD && nf > (uint32_t)(kFullLaneRows * k)) {
        const float gamma = P.gamma, ecm = st->ec_max;
        uint64_t my_rc = 0;
        for (uint32_t q = blockIdx.x * blockDim.x + tid; q < nf; q += gridDim.x * blockDim.x) {
            const int64_t i = Lg.surv[Lg.fq[q]];
            const int inc = first ? -1 : P.a[i];
            const float* xr = P.X + i * d;
            float x[kFullLaneD];
#pragma unroll
            for (int m = 0; m < kFullLaneD; ++m) x[m] = m < d ? xr[m] : 0.f;   // uniform
            float d1 = INFINITY, d2 = INFINITY;
            int rk1 = INT_MAX, b = 0;
            for (int j0 = 0; j0 < k; j0 += 4) {
                float a[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const float* c = P.C32 + (int64_t)min(j0 + e, k - 1) * d;
                    a[e] = 0.f;
#pragma unroll
                    for (int m = 0; m < kFullLaneD; ++m) {
                        if (m >= d) break;   // uniform
                        const float t = x[m] - c[m];
                        a[e] = fmaf(t, t, a[e]);
                    }
                }
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int j = j0 + e, rk = j == inc ? -1 : j;
                    if (j >= k) continue;
                    if (a[e] < d1 || (a[e] == d1 && rk < rk1)) {
                        d2 = d1;
                        d1 = a[e];
                        rk1 = rk;
                        b = j;
                    } else if (a[e] < d2) {
                        d2 = a[e];
                    }
                }
            }
            // Float64 for near ties, and where float32 squares overflow or lose
            // bits; a distance below 2^-50 alone is bounded by 2^-49.
            float ub = upper_bound(d1, P.ec[b], gamma);
            if (d1 < 0x1p-100f) ub = fmaxf(ub, 0x1p-49f);
            const float band = 2.f * gamma * (d1 + d2) + 4.f * (sqrtf(d1) + sqrtf(d2)) * ecm + 8.f * ecm * ecm;
            if (!(d2 - d1 > band) || !(d2 <= 0x1p120f) || (d1 < 0x1p-100f && d2 < 0x1p-96f)) {
                double Db = INFINITY;
                int kb = INT_MAX, bb = 0;
                for (int j = 0; j < k; ++j) {
                    const double D = sqd64(xr, P.C64 + (int64_t)j * d, d);
                    const int rk = j == inc ? -1 : j;
                    if (D < Db || (D == Db && rk < kb)) {
                        Db = D;
                        kb = rk;
                        bb = j;
                    }
                }
                b = bb;
                ub = f32_up(sqrt(Db) * (1.0 + 0x1p-40));
                my_rc += 1;
            }
            if (b != inc) {
                P.a[i] = b;
                my_changed += 1;
                if (rec_moves) {
                    const uint32_t qm = atomicAdd(Lg.nmv, 1u);
                    if (qm < (uint32_t)Lg.mvcap) Lg.mv[qm] = make_int4((int)i, inc, b, 0);
                }
            }
            P.u[i] = ub;
        }
        const int base = k * d + k;
        const int slot[2] = {base + kStChanged, base + kStRecheck};
        uint64_t v[2] = {my_changed, my_rc};
        add_stats_block<2>(P.total, slot, v);
        return;
    }
    if (blockIdx.x == 0 && tid == 0 && nf) {   // every survivor below is decided in float64
        unsigned long long* sc = reinterpret_cast<unsigned long long*>(P.total + (int64_t)k * d + k);
        atomicAdd(&sc[kStRecheck], (unsigned long long)nf);
    }
    const uint32_t items = nsplit * kFullSplit + (nf - nsplit);
    for (uint32_t it = blockIdx.x; it < items; it += gridDim.x) {
        const bool split = it < nsplit * kFullSplit;
        const uint32_t q = split ? it / kFullSplit : nsplit + (it - nsplit * kFullSplit);
        const int part = split ? (int)(it % kFullSplit) : 0;
        const int j0 = split ? part * kr : 0, j1 = split ? min(k, j0 + kr) : k;
        const int64_t i = Lg.surv[Lg.fq[q]];
        __syncthreads();   // the previous item's row and reduction are consumed
        for (int m = tid; m < d; m += blockDim.x) xd[m] = (double)P.X[i * d + m];
        __syncthreads();
        const int inc = first ? -1 : P.a[i];
        double Db = INFINITY;
        int bb = -1, kb = INT_MAX;
        for (int j = j0 + tid; j < j1; j += blockDim.x) {
            const double* cr = P.C64 + (int64_t)j * d;
            double acc = 0.0;
            for (int m = 0; m < d; ++m) {
                const double t = xd[m] - cr[m];
                acc = fma(t, t, acc);
            }
            const int rk = j == inc ? -1 : j;
            if (acc < Db || (acc == Db && rk < kb)) {
                Db = acc;
                bb = j;
                kb = rk;
            }
        }
        rD[tid] = Db;
        rJ[tid] = bb;
        rK[tid] = kb;
        __syncthreads();
        for (int w = 128; w > 0; w >>= 1) {
            if (tid < w) {
                const double D2 = rD[tid + w];
                const int k2 = rK[tid + w];
                if (D2 < rD[tid] || (D2 == rD[tid] && k2 < rK[tid])) {
                    rD[tid] = D2;
                    rJ[tid] = rJ[tid + w];
                    rK[tid] = k2;
                }
            }
            __syncthreads();
        }
        if (!split) {
            if (tid == 0) decide(i, inc, rD[0], rJ[0]);
            continue;
        }
        if (tid == 0) {
            FullPart* fp = Lg.fpart + (int64_t)q * kFullSplit;
            fp[part] = FullPart{rD[0], rJ[0], rK[0]};
            __threadfence();
            last = atomicAdd(&Lg.fcnt[q], 1u);
        }
        __syncthreads();
        if (tid == 0 && last == kFullSplit - 1) {   // every range is in: combine
            __threadfence();
            const volatile FullPart* fp = Lg.fpart + (int64_t)q * kFullSplit;
            double D = INFINITY;
            int bj = -1, bk = INT_MAX;
            for (int r = 0; r < kFullSplit; ++r) {
                const double D2 = fp[r].D;
                const int k2 = fp[r].rk;
                if (D2 < D || (D2 == D && k2 < bk)) {
                    D = D2;
                    bj = fp[r].j;
                    bk = k2;
                }
            }
            Lg.fcnt[q] = 0;   // ready for the next step
            decide(i, inc, D, bj);
        }
    }
    if (threadIdx.x == 0 && my_changed) {
        unsigned long long* sc = reinterpret_cast<unsigned long long*>(P.total + (int64_t)k * d + k);
        atomicAdd(&sc[kStChanged], (unsigned long long)my_changed);
    }
}

// ---------------------------------------------------------------------------
// Counting sort of the points by their new cluster.

__global__ __launch_bounds__(256) void k_hist_large(Dev P, Large Lg) {
    if (!P.st->active || large_incremental(P, Lg)) return;
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t* h = reinterpret_cast<uint32_t*>(smem);
    const int k = P.k;
    for (int j = threadIdx.x; j < k; j += blockDim.x) h[j] = 0;
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * Lg.span;
    const int64_t hi = min(P.n, lo + Lg.span);
    for (int64_t i = lo + threadIdx.x; i < hi; i += blockDim.x) atomicAdd(&h[P.a[i]], 1u);
    __syncthreads();
    for (int j = threadIdx.x; j < k; j += blockDim.x) Lg.cnt[(int64_t)blockIdx.x * k + j] = h[j];
}

// Per cluster j: exclusive prefix of the block counts (write offsets
// relative to the cluster start) and the cluster size into base[j].
__global__ __launch_bounds__(256) void k_scan_large_cols(Dev P, Large Lg) {
    if (!P.st->active || large_incremental(P, Lg)) return;
    const int j = blockIdx.x * blockDim.x + threadIdx.x;
    if (j >= P.k) return;
    uint32_t run = 0;
    for (int g = 0; g < Lg.Gs; ++g) {
        const int64_t o = (int64_t)g * P.k + j;
        const uint32_t c = Lg.cnt[o];
        Lg.off[o] = run;
        run += c;
    }
    Lg.base[j] = run;
}

// One block: cluster starts (exclusive scan of the sizes) and the first
// segment chunk of every cluster.  base[k] = n, cbase[k] = chunk count.
__global__ __launch_bounds__(1024) void k_scan_large_clusters(Dev P, Large Lg) {
    if (!P.st->active || large_incremental(P, Lg)) return;
    const int k = P.k, t = threadIdx.x, T = blockDim.x;
    __shared__ uint32_t ps[1024], pc[1024];
    const int per = (k + T - 1) / T, j0 = t * per, j1 = min(k, j0 + per);
    uint32_t s = 0, sc = 0;
    for (int j = j0; j < j1; ++j) {
        const uint32_t sz = Lg.base[j];
        s += sz;
        sc += (sz + kLgChunkRows - 1) / kLgChunkRows;
    }
    ps[t] = s;
    pc[t] = sc;
    __syncthreads();
    for (int w = 1; w < T; w <<= 1) {   // inclusive Hillis-Steele scan
        const uint32_t a = t >= w ? ps[t - w] : 0, b = t >= w ? pc[t - w] : 0;
        __syncthreads();
        ps[t] += a;
        pc[t] += b;
        __syncthreads();
    }
    uint32_t run = ps[t] - s, crun = pc[t] - sc;
    for (int j = j0; j < j1; ++j) {
        const uint32_t sz = Lg.base[j];
        Lg.base[j] = run;
        Lg.cbase[j] = crun;
        run += sz;
        crun += (sz + kLgChunkRows - 1) / kLgChunkRows;
    }
    if (t == T - 1) {
        Lg.base[k] = ps[T - 1];
        Lg.cbase[k] = pc[T - 1];
    }
}

__global__ __launch_bounds__(256) void k_scatter_large(Dev P, Large Lg) {
    if (!P.st->active || large_incremental(P, Lg)) return;
    extern __shared__ __align__(16) unsigned char smem[];
    uint32_t* pos = reinterpret_cast<uint32_t*>(smem);
    const int k = P.k;
    for (int j = threadIdx.x; j < k; j += blockDim.x)
        pos[j] = Lg.base[j] + Lg.off[(int64_t)blockIdx.x * k + j];
    __syncthreads();
    const int64_t lo = (int64_t)blockIdx.x * Lg.span;
    const int64_t hi = min(P.n, lo + Lg.span);
    for (int64_t i = lo + threadIdx.x; i < hi; i += blockDim.x)
        Lg.perm[atomicAdd(&pos[P.a[i]], 1u)] = (int32_t)i;
}

// One block per chunk of <= kLgChunkRows points of one cluster: exact
// fixed-point coordinate sums.
__global__ __launch_bounds__(256) void k_segsum_large(Dev P_, Large Lg) {
    const Dev P = with_scales(P_);
    if (!P.st->active || large_incremental(P, Lg)) return;
    const int c = blockIdx.x;
    const int k = P.k, d = P.d;
    if (c >= (int)Lg.cbase[k]) return;
    int lo = 0, hi = k;   // cluster j with cbase[j] <= c < cbase[j + 1]
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if ((int)Lg.cbase[mid] <= c) lo = mid;
        else hi = mid;
    }
    const int j = lo;
    const uint32_t r0 = Lg.base[j] + (uint32_t)(c - (int)Lg.cbase[j]) * kLgChunkRows;
    const uint32_t r1 = min(Lg.base[j + 1], r0 + kLgChunkRows);
    for (int m = threadIdx.x; m < d; m += blockDim.x) {
        uint64_t acc = 0;
        for (uint32_t r = r0; r < r1; ++r) acc += fixed_bits((double)P.X[(int64_t)Lg.perm[r] * d + m], P.qscale);
        Lg.cpart[(int64_t)c * d + m] = acc;
    }
}

// Per-cluster sums (over the cluster's chunks) and counts into the reduced
// row, less the running sums that k_update adds back.
__global__ __launch_bounds__(256) void k_chunk_reduce_large(Dev P, Large Lg) {
    if (!P.st->active || large_incremental(P, Lg)) return;
    const int k = P.k, d = P.d;
    const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (e < (int64_t)k * d) {
        const int j = (int)(e / d), m = (int)(e - (int64_t)j * d);
        uint64_t acc = 0;
        for (uint32_t cc = Lg.cbase[j]; cc < Lg.cbase[j + 1]; ++cc) acc += Lg.cpart[(int64_t)cc * d + m];
        P.total[e] = acc - P.sums[e];
        if (m == 0) {
            const int64_t o = (int64_t)k * d + j;
            P.total[o] = (uint64_t)(Lg.base[j + 1] - Lg.base[j]) - P.sums[o];
        }
    }
}

// Incremental sums: every move takes its row's exact fixed-point image out
// of the old cluster's sum and into the new one's (wrap-around integers, so
// the result equals the full sum bit for bit); one wave per move.
__global__ __launch_bounds__(256) void k_moves_large(Dev P_, Large Lg) {
    const Dev P = with_scales(P_);
    if (!P.st->active || !large_incremental(P, Lg)) return;
    const int k = P.k, d = P.d, lane = threadIdx.x & 63;
    const uint32_t nm = *Lg.nmv;
    unsigned long long* T = reinterpret_cast<unsigned long long*>(P.total);
    for (uint32_t q = blockIdx.x * (blockDim.x >> 6) + (threadIdx.x >> 6); q < nm;
         q += gridDim.x * (blockDim.x >> 6)) {
        const int4 mv = Lg.mv[q];
        const float* xr = P.X + (int64_t)mv.x * d;
        for (int m = lane; m < d; m += 64) {
            const uint64_t img = fixed_bits((double)xr[m], P.qscale);
            atomicAdd(&T[(int64_t)mv.y * d + m], (unsigned long long)(0ull - img));
            atomicAdd(&T[(int64_t)mv.z * d + m], (unsigned long long)img);
        }
        if (lane == 0) {
            atomicAdd(&T[(int64_t)k * d + mv.y], ~0ull);
            atomicAdd(&T[(int64_t)k * d + mv.z], 1ull);
        }
    }
}

// ---------------------------------------------------------------------------
// Centroid table for large k*d: the minima s of the half distances (the
// distances themselves are not kept; this path tests Clause 1 only).  A block
// takes kTiTile rows against kTiCols centroids, kTiK dimensions at a time
// staged in LDS from coalesced loads (the next ones in registers); a lane
// forms four rows' distances to one centroid.  Bound by float64 vector work,
// 2 k^2 d of it, at k = 1000 and by latency at a few hundred centroids.  With
// four block columns whatever k, a lane per centroid reading its own row, and
// each row's norm summed by one lane, 16 rows against 250 centroids took 77 us
// at k = 1000, d = 256 and 37 us at k = 200, d = 128; now 49 and 13 us.

__global__ __launch_bounds__(256) void k_centroid_table_tiled(Dev P, Large Lg, int force) {
    if (!force && !P.st->active) return;
    const int tid = threadIdx.x, lane = tid & 63, rg = tid >> 6;
    if (blockIdx.x == 0 && blockIdx.y == 0 && tid == 0) {   // the next step's lists start empty
        *Lg.nsurv = 0;
        *Lg.nfull = 0;
        *Lg.nmq = 0;
        *Lg.nmv = 0;
    }
    if (P.iterm && !force && blockIdx.x == 0 && blockIdx.y == 0 && tid < 64) close_inertia(P);
    const int k = P.k, d = P.d;
    const int i0 = blockIdx.x * kTiTile, j0 = blockIdx.y * kTiCols;
    __shared__ double A[kTiTile][kTiK + 1], B[kTiCols][kTiK + 1];
    const int sr = tid >> 4, sm = tid & 15;   // this lane's row (of 16) and dimension in a staged piece
    auto at = [&](int r, int m) __attribute__((always_inline)) {
        return r < k && m < d ? P.C64[(int64_t)r * d + m] : 0.0;
    };
    double na, nb[kTiCols / 16];
    auto load = [&](int m0) __attribute__((always_inline)) {
        na = at(i0 + sr, m0 + sm);
#pragma unroll
        for (int q = 0; q < kTiCols / 16; ++q) nb[q] = at(j0 + 16 * q + sr, m0 + sm);
    };
    double acc[4] = {0.0, 0.0, 0.0, 0.0};
    load(0);
    for (int m0 = 0; m0 < d; m0 += kTiK) {
        __syncthreads();
        A[sr][sm] = na;
#pragma unroll
        for (int q = 0; q < kTiCols / 16; ++q) B[16 * q + sr][sm] = nb[q];
        __syncthreads();
        if (m0 + kTiK < d) load(m0 + kTiK);
#pragma unroll
        for (int m = 0; m < kTiK; ++m) {   // zero past d
            const double b = B[lane][m];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const double t = A[4 * rg + r][m] - b;
                acc[r] = fma(t, t, acc[r]);
            }
        }
    }
    const int j = j0 + lane;
#pragma unroll
    for (int r = 0; r < 4; ++r) {   // this column block's minimum; k_split_rows forms s from them
        const int i = i0 + 4 * rg + r;
        float hv = j < k && j != i ? f32_down(0.5 * sqrt(acc[r]) * (1.0 - 0x1p-40)) : INFINITY;
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) hv = fminf(hv, __shfl_xor(hv, off));
        if (lane == 0 && i < k) Lg.smin[(int64_t)blockIdx.y * k + i] = hv;
    }
    if (blockIdx.y == 0) {   // the rows' float32 squared norms, 16 lanes each
        const int i = min(i0 + sr, k - 1);
        const float* c32 = P.C32 + (int64_t)i * d;
        double n2 = 0.0;
        for (int m = sm; m < d; m += 16) {
            const double v = (double)c32[m] - (double)P.mu[m];
            n2 = fma(v, v, n2);
        }
#pragma unroll
        for (int off = 8; off > 0; off >>= 1) n2 += __shfl_xor(n2, off);
        if (sm == 0 && i0 + sr < k) P.cn2[i] = (float)n2;
    }
    if (blockIdx.x == 0 && blockIdx.y == 0) {
        __shared__ float mx[4];
        float em = 0.f;
        for (int q = tid; q < k; q += 256) em = fmaxf(em, P.ec[q]);
#pragma unroll
        for (int off = 32; off > 0; off >>= 1) em = fmaxf(em, __shfl_xor(em, off));
        if (lane == 0) mx[rg] = em;
        __syncthreads();
        if (tid == 0) P.st->ec_max = fmaxf(fmaxf(mx[0], mx[1]), fmaxf(mx[2], mx[3]));
    }
}

// ---------------------------------------------------------------------------
// Launchers

const void* large_mfma_symbol() { return reinterpret_cast<const void*>(&k_mfma_large); }

// Assignment group: Clause 1 and the matrix-core candidates.  The candidates'
// refinement opens the reduction group (its timing slot).
hipError_t launch_large_assign(const Dev& dv, const Large& lg, int gb, hipStream_t s) {
    hipLaunchKernelGGL(k_bound_large, dim3(gb), dim3(kLgBoundThreads), 0, s, dv, lg);
    hipLaunchKernelGGL(k_mfma_large, dim3(lg.Gm), dim3(256), large_mfma_lds(), s, dv, lg);
    return hipGetLastError();
}

hipError_t launch_large_split_x(const Dev& dv, const Large& lg, int cus, hipStream_t s) {
    int64_t g = (dv.n + 3) / 4;
    if (g > (int64_t)cus * 16) g = (int64_t)cus * 16;
    hipLaunchKernelGGL(k_split_rows, dim3((unsigned)g), dim3(256), 0, s, dv.X, dv.n, dv.n, dv.d, lg.nch, lg.xs,
                       lg.x2, static_cast<const IterState*>(dv.st), 1, static_cast<const float*>(nullptr),
                       static_cast<float*>(nullptr), static_cast<const float*>(dv.mu));
    return hipGetLastError();
}

hipError_t launch_large_reduce(const Dev& dv, const Large& lg, hipStream_t s) {
    hipLaunchKernelGGL(k_refine_large, dim3(lg.Gr), dim3(256), 0, s, dv, lg);
    hipLaunchKernelGGL(k_multi_large, dim3(lg.Gr), dim3(256), 0, s, dv, lg);
    hipLaunchKernelGGL(k_full_large, dim3(lg.Gr), dim3(256), 8 * dv.d, s, dv, lg);
    const int hl = 4 * dv.k;
    hipLaunchKernelGGL(k_hist_large, dim3(lg.Gs), dim3(256), hl, s, dv, lg);
    hipLaunchKernelGGL(k_scan_large_cols, dim3((dv.k + 255) / 256), dim3(256), 0, s, dv, lg);
    hipLaunchKernelGGL(k_scan_large_clusters, dim3(1), dim3(1024), 0, s, dv, lg);
    hipLaunchKernelGGL(k_scatter_large, dim3(lg.Gs), dim3(256), hl, s, dv, lg);
    hipLaunchKernelGGL(k_segsum_large, dim3(lg.NCmax), dim3(256), 0, s, dv, lg);
    const int64_t kd = (int64_t)dv.k * dv.d;
    hipLaunchKernelGGL(k_chunk_reduce_large, dim3((unsigned)((kd + 255) / 256)), dim3(256), 0, s, dv, lg);
    hipLaunchKernelGGL(k_moves_large, dim3(lg.Gr), dim3(256), 0, s, dv, lg);
    return hipGetLastError();
}

const void* large_dynamic_symbol(int i) {
    const void* const s[kLgDynamic] = {reinterpret_cast<const void*>(&k_full_large),
                                       reinterpret_cast<const void*>(&k_hist_large),
                                       reinterpret_cast<const void*>(&k_scatter_large)};
    return s[i];
}

hipError_t launch_large_table(const Dev& dv, const Large& lg, int force, hipStream_t s) {
    hipLaunchKernelGGL(k_centroid_table_tiled, dim3((dv.k + kTiTile - 1) / kTiTile, (dv.k + kTiCols - 1) / kTiCols),
                       dim3(256), 0, s, dv, lg, force);
    const int64_t kp = (int64_t)lg.nct * kLgN;   // padded to whole centroid tiles
    hipLaunchKernelGGL(k_split_rows, dim3((unsigned)((kp + 3) / 4)), dim3(256), 0, s, static_cast<const float*>(dv.C32),
                       kp, (int64_t)dv.k, dv.d, lg.nch, lg.cs, lg.cn2p, static_cast<const IterState*>(dv.st), force,
                       static_cast<const float*>(lg.smin), dv.s, static_cast<const float*>(dv.mu));
    return hipGetLastError();
}

}  // namespace km
