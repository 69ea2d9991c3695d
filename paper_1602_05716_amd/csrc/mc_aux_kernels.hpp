// mc_aux_kernels.hpp -- double-precision total-energy re-sum and pair
// correlation (g(r)) kernels for gfx950.
//
// Paper: Liang, Xing, Li, arXiv:1602.05716.  Sec. 3.3: energy sums in double
// precision; Sec. 5.2: the total energy is monitored, and the pair
// correlation functions are measured on ions away from the wall.
#pragma once

#include "mc_sweep_kernel.hpp"

namespace mcdev {

// Small device-side record of the energy bookkeeping.
struct EnergyAux {
    double e_resum;      // last re-summed total energy
    double drift_last;   // running minus re-summed energy at the last re-sum
    double drift_max;    // largest |drift| seen
    unsigned long long n_resum;
};

// Stats slots written by the sweep kernel.
enum { ST_MOVES = 0, ST_ACC, ST_WALL, ST_OVERLAP, ST_METRO, ST_ITERS, ST_EARLY,
       ST_DA_MOVES, ST_DA_CONFLICTS, ST_DA_S1REJ, ST_DA_S1PASS, ST_DA_S2REJ, ST_N };

// What the host reads of a chain between launches, and where it lies.
struct ChainReport {
    int32_t abort, pad;
    double e_state;
    EnergyAux aux;
    DAState da;
    unsigned long long stats[ST_N];
};
constexpr size_t kReportHead = 512;  // positions follow the report from here
static_assert(sizeof(ChainReport) <= kReportHead, "report layout");
struct ReportSource {
    const int* abort;
    const double* e_state;
    const EnergyAux* aux;
    const DAState* da;
    const unsigned long long* stats;
};

// The report to r and count values of the packed positions to xyz, both
// pinned host memory, four values a thread (xyz has room for whole fours).
// Bound: one launch and one wait: 12 us for an energy, 13 for the counters, 16
// with the positions of 2001 ions in double (the kernel itself 2.8); a copy per
// item into pageable memory took 10 us each.
template <typename T, typename T4>
__global__ void __launch_bounds__(256)
report_kernel(ReportSource s, ChainReport* __restrict__ r, const T4* __restrict__ pos, int count, T* __restrict__ xyz)
{
    const int t = blockIdx.x * 256 + threadIdx.x;
    if (blockIdx.x == 0) {
        if (t < ST_N) r->stats[t] = s.stats[t];
        if (t == 64) {
            r->abort = *s.abort;
            r->e_state = *s.e_state;
        }
        if (t == 128) r->aux = *s.aux;
        if (t == 192) r->da = *s.da;
    }
    if (4 * t >= count) return;
    T v[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const int e = min(4 * t + k, count - 1);
        const T* p = reinterpret_cast<const T*>(pos + e / 3);
        v[k] = p[e % 3];
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) xyz[4 * t + k] = v[k];
}

// Work item of a batched auxiliary launch: chain index and the block's index
// inside that chain.
struct BlockItem {
    int32_t chain;
    int32_t part;
};

// Pairs of super-rows of a chain of nb groups, for the re-sum (below).
__host__ __device__ inline int energy_pairs(int nb) { return ((nb + 1) / 2 + 1) / 2; }
// Blocks per pair of super-rows: enough for eight a CU (2048 in all) from the
// chain alone, while every wave keeps at least two tiles.  From the chain
// only, so that the order of its sum, and with it the last bits of its
// energy, is the same whatever other chains its handle holds.
__host__ __device__ inline int energy_split(int nb) {
    const int want = (2048 + energy_pairs(nb) - 1) / energy_pairs(nb);
    const int most = nb / 8;
    return want < most ? want : (most > 1 ? most : 1);
}

// Positions are read as {x, y, z, *} records (the fourth word is the sweep
// version tag of the sweep kernel) from the image of the given parity, and
// charges from their own array.  E = l_B sum_{i<j} q_i q_j / r_ij in double.
//
// Bound: the double-precision ALU.  A super-row is 128 ions, two a lane, so
// that each partner read from LDS (32 bytes, a broadcast) serves two pair
// terms: with one ion a lane the LDS reads of four waves would take as long
// as their arithmetic.  Block (p, c) of a chain takes super-rows p and
// K-1-p (K super-rows; the pair has about the same number of tiles for
// every p), and its wave w the tiles row + 4 c + w, + 4 e_split, ...: the
// split over c fills the chip where a chain has few groups.  The chain's
// e_partial[p e_split + c] receives the block's sum.  N = 65536: 1.0 ms
// (2.1e12 pair terms/s) with the read-out, 3.7 ms with one ion a lane, two
// waves per SIMD and a rounded sqrt and division a term.
template <typename T>
__global__ void __launch_bounds__(256)
energy_partial_kernel(const ChainDesc* __restrict__ chains, const BlockItem* __restrict__ items, int parity)
{
    using T4 = typename Prec<T>::T4;
    __shared__ double4 st[4][kGroup];
    __shared__ double wsum[4];
    const BlockItem it = items[blockIdx.x];
    const ChainDesc& cd = chains[it.chain];
    const int nb = cd.nb, split = cd.e_split;
    const T4* __restrict__ pos = (const T4*)cd.pos + (size_t)parity * nb * kGroup;
    const T* __restrict__ charge = (const T*)cd.charge;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int K = (nb + 1) / 2, p = it.part / split, c = it.part - p * split;
    double acc = 0.0;
    for (int pass = 0; pass < 2; ++pass) {
        const int sr = pass == 0 ? p : K - 1 - p;
        if (pass == 1 && sr == p) break;
        const int row0 = 2 * sr, row1 = 2 * sr + 1 < nb ? 2 * sr + 1 : 2 * sr;
        const T4 a4 = pos[row0 * kGroup + lane], b4 = pos[row1 * kGroup + lane];
        const double ax = (double)a4.x, ay = (double)a4.y, az = (double)a4.z;
        const double bx = (double)b4.x, by = (double)b4.y, bz = (double)b4.z;
        const double qa = (double)charge[row0 * kGroup + lane];
        // no second row past the end: its terms are formed and count nothing
        const double qb = row1 != row0 ? (double)charge[row1 * kGroup + lane] : 0.0;
        double ea = 0.0, eb = 0.0;
        int t = row0 + 4 * c + wave;
        T4 nx{};
        T nq = (T)0;
        if (t < nb) {
            nx = pos[t * kGroup + lane];
            nq = charge[t * kGroup + lane];
        }
        for (; t < nb; t += 4 * split) {
            st[wave][lane] = make_double4((double)nx.x, (double)nx.y, (double)nx.z, (double)nq);
            wave_lds_sync();
            if (t + 4 * split < nb) {  // the next tile travels while this one is summed
                nx = pos[(t + 4 * split) * kGroup + lane];
                nq = charge[(t + 4 * split) * kGroup + lane];
            }
            double sa = 0.0, sb = 0.0;
            // partners m >= m0 of the tile, from row a's and row b's view
            auto terms = [&](auto masked_c, auto inv) {
                constexpr bool MASKED = decltype(masked_c)::value;
#pragma unroll 4
                for (int m = 0; m < kGroup; ++m) {
                    const double4 pj = st[wave][m];
                    const double dx = ax - pj.x, dy = ay - pj.y, dz = az - pj.z;
                    const double fx = bx - pj.x, fy = by - pj.y, fz = bz - pj.z;
                    const double ya = inv(__builtin_fma(dz, dz, __builtin_fma(dy, dy, dx * dx)));
                    const double yb = inv(__builtin_fma(fz, fz, __builtin_fma(fy, fy, fx * fx)));
                    if constexpr (MASKED) {
                        // the tile holds one of the two rows: j > i only
                        if (t > row0 || m > lane) sa = __builtin_fma(pj.w, ya, sa);
                        if (t > row1 || (t == row1 && m > lane)) sb = __builtin_fma(pj.w, yb, sb);
                    } else {
                        sa = __builtin_fma(pj.w, ya, sa);
                        sb = __builtin_fma(pj.w, yb, sb);
                    }
                }
            };
            auto fast = [](double d2) { return rsqrt_step(d2, __builtin_amdgcn_rsq(d2)); };
            auto plain = [](double d2) { return 1.0 / __builtin_sqrt(d2); };
            if (t > row1)
                terms(std::false_type{}, fast);
            else
                terms(std::true_type{}, fast);
            if (__ballot(sa != sa || sb != sb) != 0ull) {
                // a distance whose square is zero or infinite in double
                sa = sb = 0.0;
                terms(std::true_type{}, plain);
            }
            ea += sa;
            eb += sb;
            wave_lds_sync();
        }
        acc += qa * ea + qb * eb;
    }
    const double ws = __shfl(wave_sum(acc), 0, 64);
    if (lane == 0) wsum[wave] = ws;
    __syncthreads();
    if (threadIdx.x == 0) cd.e_partial[it.part] = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
}

// One block per chain: sums the chain's partials in a fixed order, records
// the drift of the running energy and, when `reset` is set, makes the re-sum
// the new running energy.
__global__ void __launch_bounds__(256)
energy_finalize_kernel(const ChainDesc* __restrict__ chains, int reset, int record_drift)
{
    __shared__ double wsum[4];
    const ChainDesc& cd = chains[blockIdx.x];
    const int nparts = energy_pairs(cd.nb) * cd.e_split;
    double v = 0.0;
    for (int k = threadIdx.x; k < nparts; k += 256) v += cd.e_partial[k];
    v = wave_sum(v);
    if ((threadIdx.x & 63) == 0) wsum[threadIdx.x >> 6] = v;
    __syncthreads();
    if (threadIdx.x != 0) return;
    EnergyAux* aux = (EnergyAux*)cd.aux;
    double e = ((wsum[0] + wsum[1]) + wsum[2]) + wsum[3];
    e *= cd.lB;
    aux->e_resum = e;
    if (record_drift) {
        const double d = *cd.e_state - e;
        aux->drift_last = d;
        const double ad = d < 0 ? -d : d;
        if (ad > aux->drift_max) aux->drift_max = ad;
        aux->n_resum += 1;
    }
    if (reset) *cd.e_state = e;
}

// Pair counts for g_ab(r): centre i needs |x_i| <= R - rmax (the wall
// exclusion of Sec. 5.2), neighbours are all j != i; bin k = floor(r / dr)
// for r < rmax.  Distances and bins are formed in double exactly as written
// (no fused multiply-add), so the integer counts do not depend on the
// kernel's tiling.  One block of 4 waves per group of 64 centres of a chain;
// each wave takes every 4th partner tile; counts go to an LDS histogram
// first.
template <typename T>
__global__ void __launch_bounds__(256)
rdf_kernel(const ChainDesc* __restrict__ chains, const BlockItem* __restrict__ items, int parity,
           double rmax, double dr, int bins)
{
    using T4 = typename Prec<T>::T4;
    extern __shared__ unsigned int hist[];   // [ntypes*ntypes*bins]
    __shared__ double st[4][kGroup][3];
    __shared__ int stt[4][kGroup];
    const BlockItem item = items[blockIdx.x];
    const ChainDesc& cd = chains[item.chain];
    const int n = cd.n, nb = cd.nb, ntypes = cd.ntypes;
    const T4* __restrict__ pos = (const T4*)cd.pos + (size_t)parity * nb * kGroup;
    const int32_t* __restrict__ type = cd.type;
    const double rc = cd.rdf_rc;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int nh = ntypes * ntypes * bins;
    for (int k = threadIdx.x; k < nh; k += blockDim.x) hist[k] = 0u;
    __syncthreads();

    const int row = item.part;
    const int i = row * kGroup + lane;
    const T4 xi4 = pos[i];
    const double xi = (double)xi4.x, yi = (double)xi4.y, zi = (double)xi4.z;
    const double r2i = xi * xi + yi * yi + zi * zi;
    const bool centre = i < n && rc >= 0.0 && !(r2i > rc * rc);
    const int ti = i < n ? type[i] : 0;
    const double rmax2 = rmax * rmax * (1.0 + 1e-12);
    if (wave == 0) {
        const unsigned long long cm = __ballot(centre);
        if (cm) {
            // centres of this block by type
            for (int a = 0; a < ntypes; ++a) {
                const unsigned long long ca = __ballot(centre && ti == a);
                if (lane == 0 && ca) atomicAdd(&cd.rdf_centres[a], (unsigned long long)__popcll(ca));
            }
        }
    }
    for (int t = wave; t < nb; t += 4) {
        const int jj = t * kGroup + lane;
        const T4 pj = pos[jj];
        st[wave][lane][0] = (double)pj.x;
        st[wave][lane][1] = (double)pj.y;
        st[wave][lane][2] = (double)pj.z;
        stt[wave][lane] = jj < n ? type[jj] : -1;
        wave_lds_sync();
        if (centre) {
            for (int m = 0; m < kGroup; ++m) {
                const int j = t * kGroup + m;
                const int tj = stt[wave][m];
                if (j == i || tj < 0) continue;
                const double dx = xi - st[wave][m][0];
                const double dy = yi - st[wave][m][1];
                const double dz = zi - st[wave][m][2];
                const double d2 = dx * dx + dy * dy + dz * dz;
                if (d2 < rmax2) {
                    const double r = __builtin_sqrt(d2);
                    if (r < rmax) {
                        const int k = (int)__builtin_floor(r / dr);
                        if (k < bins) atomicAdd(&hist[(ti * ntypes + tj) * bins + k], 1u);
                    }
                }
            }
        }
        wave_lds_sync();
    }
    __syncthreads();
    for (int k = threadIdx.x; k < nh; k += blockDim.x)
        if (hist[k]) atomicAdd(&cd.rdf_counts[k], (unsigned long long)hist[k]);
}

// ---- pair counts on a grid of cells.  rdf_kernel above tests all N^2 pairs;
// of these only the fraction (rmax / R)^3 lies in range (0.4 % in the 3:-1
// production system).  Here the ions are first sorted into cubic cells
// of side h = rmax / 2 (rdf_grid), so that a centre meets the ions of the
// 5 x 5 x 5 cells around its own only.  The counts are integers formed from
// the same exact distances, so the order of the ions in a cell, which the
// atomics leave open, does not show.  Four launches: bin, scan, scatter,
// count.  One sample of the 3:-1 system at N = 131072 (range 0.16 R): 0.5 ms
// with its read-out where the test of all pairs took 9.8; of the 2:1 system
// at N = 98304: 0.6 ms for 8.6.  The bound is the double-precision test and
// the binning of the partners that a cell neighbourhood holds (a quarter of
// them in range).

// Cells per side of a chain's grid, of side rmax / 2, wider where that would
// make more cells than ions or more than 40 across (the scan of empty cells
// then costs more than they save).  The side is a hair above rmax / 2, so
// that rounding in the cell index never puts a pair in range more than two
// cells apart.
// The most cells across, 24 / 32 / 40 / 48 / 64, in one sample: 437 / 348 / 334 /
// 345 / 348 us at N = 131072 (range 0.02 R), 1162 / 743 / 617 / 617 / 617 at 262144
// (0.02 R), 1246 / 826 / 758 / 809 / 805 (0.1 R).
constexpr int kRdfReach = 2;
constexpr int kRdfMaxSide = 40;
inline void rdf_grid(int n, double R, double rmax, int* side, double* h) {
    int most = 4;
    while (most < kRdfMaxSide && (most + 1) * (most + 1) * (most + 1) <= n) ++most;
    double w = rmax / (double)kRdfReach;
    if (w < 2.0 * R / (double)(most - 1)) w = 2.0 * R / (double)(most - 1);
    *h = w * (1.0 + 1e-9);
    *side = (int)(2.0 * R / *h) + 1;
}

// Cell coordinate: positions lie in [-R, R]; rounding at the wall is clamped
// (which keeps the order of the cells).
__device__ __forceinline__ int rdf_cell(double x, const ChainDesc& cd) {
    const int k = (int)__builtin_floor((x + cd.rdf_org) * cd.rdf_inv_h);
    return k < 0 ? 0 : (k >= cd.rdf_side ? cd.rdf_side - 1 : k);
}

// Counts the ions of every cell and gives each its rank there; counts the
// centres by species.  One block of 64 per group of a chain.
template <typename T>
__global__ void __launch_bounds__(64)
rdf_bin_kernel(const ChainDesc* __restrict__ chains, const BlockItem* __restrict__ items, int parity)
{
    using T4 = typename Prec<T>::T4;
    const BlockItem item = items[blockIdx.x];
    const ChainDesc& cd = chains[item.chain];
    const T4* __restrict__ pos = (const T4*)cd.pos + (size_t)parity * cd.nb * kGroup;
    const int i = item.part * kGroup + (int)threadIdx.x;
    const bool valid = i < cd.n;
    const T4 p = pos[i];
    const double x = (double)p.x, y = (double)p.y, z = (double)p.z;
    const double r2 = x * x + y * y + z * z;
    const bool centre = valid && cd.rdf_rc >= 0.0 && !(r2 > cd.rdf_rc * cd.rdf_rc);
    const int t = valid ? cd.type[i] : 0;
    if (__ballot(centre) != 0ull) {
        for (int a = 0; a < cd.ntypes; ++a) {
            const unsigned long long ca = __ballot(centre && t == a);
            if (threadIdx.x == 0 && ca) atomicAdd(&cd.rdf_centres[a], (unsigned long long)__popcll(ca));
        }
    }
    if (valid) {
        const int cell = (rdf_cell(z, cd) * cd.rdf_side + rdf_cell(y, cd)) * cd.rdf_side + rdf_cell(x, cd);
        cd.rdf_rank[i] = atomicAdd(&cd.rdf_cells[cell], 1);
    }
}

// Exclusive scan of the cell counts into rdf_start[cells + 1]; clears the
// counts for the next sample.  One block per chain, a contiguous run of cells
// per wave, read 64 at a time (a run per thread, strided over the lanes, took
// 0.25 ms for 64000 cells).
__global__ void __launch_bounds__(1024)
rdf_scan_kernel(const ChainDesc* __restrict__ chains)
{
    __shared__ int wsum[16];
    const ChainDesc& cd = chains[blockIdx.x];
    const int cells = cd.rdf_side * cd.rdf_side * cd.rdf_side;
    if (cells == 0) return;  // a chain without a grid
    int* __restrict__ count = cd.rdf_cells;
    int* __restrict__ start = cd.rdf_start;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int run = ((cells + 16 * kGroup - 1) / (16 * kGroup)) * kGroup;
    const int c0 = wave * run, c1 = c0 + run < cells ? c0 + run : cells;
    int sum = 0;
#pragma unroll 8
    for (int c = c0 + lane; c < c1; c += kGroup) sum += count[c];
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) sum += __shfl_xor(sum, d, 64);
    if (lane == 0) wsum[wave] = sum;
    __syncthreads();
    int before = 0;
    for (int w = 0; w < wave; ++w) before += wsum[w];
    for (int b = c0; b < c1; b += kGroup) {
        const int c = b + lane;
        const int v = c < c1 ? count[c] : 0;
        int incl = v;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int u = __shfl_up(incl, d, 64);
            if (lane >= d) incl += u;
        }
        if (c < c1) {
            count[c] = 0;
            start[c] = before + incl - v;
        }
        before += __builtin_amdgcn_readlane(incl, 63);
    }
    if (wave == 15 && lane == 0) start[cells] = before;
}

// The ions in cell order, {x, y, z, species}.
template <typename T>
__global__ void __launch_bounds__(64)
rdf_scatter_kernel(const ChainDesc* __restrict__ chains, const BlockItem* __restrict__ items, int parity)
{
    using T4 = typename Prec<T>::T4;
    const BlockItem item = items[blockIdx.x];
    const ChainDesc& cd = chains[item.chain];
    const T4* __restrict__ pos = (const T4*)cd.pos + (size_t)parity * cd.nb * kGroup;
    const int i = item.part * kGroup + (int)threadIdx.x;
    if (i >= cd.n) return;
    const T4 p = pos[i];
    const int cell = (rdf_cell((double)p.z, cd) * cd.rdf_side + rdf_cell((double)p.y, cd)) * cd.rdf_side +
                     rdf_cell((double)p.x, cd);
    ((T4*)cd.rdf_sorted)[cd.rdf_start[cell] + cd.rdf_rank[i]] = mk4<T>(p.x, p.y, p.z, (T)cd.type[i]);
}

// Pair counts.  An item is 64 ions in cell order, the centres, one a lane;
// they lie in one or a few rows of cells (runs of cells along x), and the
// partners of a row's centres are 25 runs of cells, each contiguous in the
// sorted order.  The block's eight waves share the partners, 64 at a time.
// A persistent grid: each block takes items in turn and adds its LDS
// histogram to the chain's once per chain (3200 bins by hundreds of blocks
// are as many atomics as a sample has pairs to bin), or sooner where a
// counter could wrap.
constexpr int kRdfWaves = 8;
// The histogram's counters have 32 bits and an item adds at most 64 n to one,
// so it is also added (and cleared) after this many items of a chain: 3 at
// n = 2^24; up to n = 1.4e6 a block of 512 has fewer items in all.
__host__ __device__ constexpr int rdf_items_per_flush(int n) { return (int)(0xFFFFFFFFull / (64ull * (unsigned)n)); }
template <typename T>
__global__ void __launch_bounds__(64 * kRdfWaves)
rdf_count_kernel(const ChainDesc* __restrict__ chains, const BlockItem* __restrict__ items, int n_items, double rmax,
                 double dr, int bins)
{
    using T4 = typename Prec<T>::T4;
    extern __shared__ unsigned int hist[];   // [ntypes*ntypes*bins]
    __shared__ double4 st[kRdfWaves][kGroup];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const double rmax2 = rmax * rmax * (1.0 + 1e-12);
    const float inv_dr = (float)(1.0 / dr), near = 1e-4f + 1e-6f * (float)bins;
    int chain = -1, nh = 0, room = 0;  // room: items before the next flush
    auto flush = [&]() {
        __syncthreads();
        if (chain >= 0)
            for (int k = threadIdx.x; k < nh; k += blockDim.x)
                if (hist[k]) atomicAdd(&chains[chain].rdf_counts[k], (unsigned long long)hist[k]);
        __syncthreads();
    };
    for (int q = blockIdx.x; q < n_items; q += gridDim.x) {
        const BlockItem item = items[q];
        if (item.chain != chain || room == 0) {
            flush();
            chain = item.chain;
            nh = chains[chain].ntypes * chains[chain].ntypes * bins;
            room = rdf_items_per_flush(chains[chain].n);
            for (int k = threadIdx.x; k < nh; k += blockDim.x) hist[k] = 0u;
            __syncthreads();
        }
        --room;
        const ChainDesc& cd = chains[chain];
        const T4* __restrict__ ions = (const T4*)cd.rdf_sorted;
        const int n = cd.n, side = cd.rdf_side, ntypes = cd.ntypes;
        const int i = item.part * kGroup + lane;
        const T4 pi = ions[i < n ? i : n - 1];
        const double xi = (double)pi.x, yi = (double)pi.y, zi = (double)pi.z;
        const bool centre = i < n && cd.rdf_rc >= 0.0 && !(xi * xi + yi * yi + zi * zi > cd.rdf_rc * cd.rdf_rc);
        unsigned long long left = __ballot(centre);
        if (left == 0ull) continue;
        const int cx = rdf_cell(xi, cd), row = rdf_cell(zi, cd) * side + rdf_cell(yi, cd);
        unsigned int* const mine = hist + (int)pi.w * ntypes * bins;
        int turn = 0;  // chunks of partners so far: the waves take them in turn
        while (left) {
            const int first = __builtin_ctzll(left);
            const int r0 = __builtin_amdgcn_readlane(row, first);
            const unsigned long long here = __ballot(centre && row == r0);
            left &= ~here;
            const int last = 63 - __builtin_clzll(here);
            const bool active = ((here >> lane) & 1ull) != 0;
            int x0 = __builtin_amdgcn_readlane(cx, first) - kRdfReach;  // cells rise along a row
            int x1 = __builtin_amdgcn_readlane(cx, last) + kRdfReach;
            x0 = x0 < 0 ? 0 : x0;
            x1 = x1 >= side ? side - 1 : x1;
            const int cz = r0 / side, cy = r0 - cz * side;
            for (int z = cz > kRdfReach ? cz - kRdfReach : 0; z <= cz + kRdfReach && z < side; ++z)
                for (int y = cy > kRdfReach ? cy - kRdfReach : 0; y <= cy + kRdfReach && y < side; ++y) {
                    const int base = (z * side + y) * side;
                    const int a = cd.rdf_start[base + x0], b = cd.rdf_start[base + x1 + 1];
                    for (int c = a; c < b; c += kGroup, ++turn) {
                        if ((turn & (kRdfWaves - 1)) != wave) continue;
                        const int m_end = b - c < kGroup ? b - c : kGroup;
                        if (lane < m_end) {
                            const T4 pj = ions[c + lane];
                            st[wave][lane] = make_double4((double)pj.x, (double)pj.y, (double)pj.z, (double)pj.w);
                        }
                        wave_lds_sync();
                        for (int m = 0; m < m_end; ++m) {
                            const double4 pj = st[wave][m];
                            const double dx = xi - pj.x, dy = yi - pj.y, dz = zi - pj.z;
                            const double d2 = dx * dx + dy * dy + dz * dz;
                            if (active && d2 < rmax2 && c + m != i) {
                                // floor(sqrt(d2) / dr): in float unless that
                                // lies near an integer (`near` is several
                                // times its error), then exactly as written
                                const float d = (float)d2;
                                const float v = d * __builtin_amdgcn_rsqf(d) * inv_dr;
                                const float f = __builtin_floorf(v);
                                int k = (int)f;
                                if (!(v - f > near && v - f < 1.f - near)) {
                                    const double r = __builtin_sqrt(d2);
                                    k = r < rmax ? (int)__builtin_floor(r / dr) : bins;
                                }
                                if (k < bins) atomicAdd(&mine[(int)pj.w * bins + k], 1u);
                            }
                        }
                        wave_lds_sync();
                    }
                }
        }
    }
    flush();
}

}  // namespace mcdev
