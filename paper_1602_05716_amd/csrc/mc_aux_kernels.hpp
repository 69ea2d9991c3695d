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

// Work item of a batched auxiliary launch: chain index and the block's index
// inside that chain.
struct BlockItem {
    int32_t chain;
    int32_t part;
};

// 1 / sqrt(d2) in double from the hardware estimate (v_rsq_f64, about 26
// bits) and one third-order step: with e = 1 - d2 y^2 (formed with a fused
// multiply-add, so its rounding does not matter), y (1 + e / 2 + 3 e^2 / 8)
// is off by e^3, far below a rounding; the result is within one unit in the
// last place, as a rounded sqrt followed by a rounded division is.  Six
// instructions instead of the 28 of those two.  NaN for d2 = 0 or infinity.
__device__ __forceinline__ double rsqrt_refined(double d2) {
    const double y = __builtin_amdgcn_rsq(d2);
    const double e = __builtin_fma(-(d2 * y), y, 1.0);
    return __builtin_fma(y * e, __builtin_fma(0.375, e, 0.5), y);
}

// Blocks per pair of super-rows of the re-sum (below) for a chain of nb
// groups in a handle whose chains have total_pairs such pairs: enough blocks
// for eight a CU (2048 in all), while every wave keeps at least two tiles.
__host__ __device__ inline int energy_split(int nb, int total_pairs) {
    const int want = (2048 + total_pairs - 1) / total_pairs;
    const int most = nb / 8;
    return want < most ? want : (most > 1 ? most : 1);
}
// Pairs of super-rows of a chain of nb groups.
__host__ __device__ inline int energy_pairs(int nb) { return ((nb + 1) / 2 + 1) / 2; }

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
            auto fast = [](double d2) { return rsqrt_refined(d2); };
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

}  // namespace mcdev
