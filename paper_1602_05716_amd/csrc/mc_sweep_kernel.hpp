// mc_sweep_kernel.hpp -- the persistent sequential-sweep kernel for gfx950.
//
// Method (Liang, Xing, Li, arXiv:1602.05716): sequential-update Metropolis
// Monte Carlo with the exact energy change of every trial (Sec. 2, Eq.
// (Delta E_ij)), hard-core overlap indicator (Sec. 3.3) and spherical hard
// wall (Sec. 5.2).  The kernel keeps the chain resident on the device for a
// whole mc_sweep call; there is no host round trip between trials.
//
// Decomposition (our own design for CDNA4; the paper's Sec. 3.2-3.7 scheme is
// prior art):
//   * Ions are cut into groups of 64 = one wavefront; group b of sweep s has
//     stream index g = s*B + b, and the trials form one sequence over g.
//   * Each target group g is served by one workgroup of M waves.  Lane i of
//     every wave is mover i of the group; wave w takes a 64/M-ion slice of
//     every partner group.  This is
//     the paper's "brush" (Sec. 3.4) turned so that the partner index is
//     uniform across the wave.
//   * By Eq. (Delta E_ij) the term of partner j is final as soon as j's own
//     latest trial is decided.  Partner groups decided more than `band`
//     groups before g are summed directly with their published positions, in
//     stream order, as they get decided (the upper/lower triangle split of
//     Sec. 2 applied continuously across sweep boundaries).
//   * For the last `band` groups and for the mover's own group, both possible
//     outcomes of partner j are evaluated at the start of the target's work
//     (old position and trial position), so that once j's accept bit is
//     known only a select and an add remain.
//   * The newest band groups' candidates (g-1, g-2) and the own group's go to
//     LDS for the chain step as soon as they are computed.  The older band
//     groups' accept masks are published before the compute waves finish;
//     each wave folds its slice of their candidates from the mask, then hands
//     over its partial sum and moves on to its next target.
//   * Wave 0 then decides the group: if the threshold lies outside the
//     interval spanned by the unknown corrections for every lane, at once.
//     Otherwise it solves the group's own accept bits, the fixed point of the
//     sequential rule a_i = f_i(a_0..a_{i-1}) (Jacobi sweeps over the wave;
//     the system is lower triangular, so the fixed point is unique, equals
//     the sequential outcome and is reached from any start), for a guess of
//     the pending band groups' masks (all rejected), while wave 1 sums the
//     older pending groups' masked rows as their masks arrive.  Each true
//     correction then costs one evaluation when the guess was right, a few
//     more iterations (updating the row sum by the flipped bits) when not.
//   * Publication: the accept mask goes out at once in the group record; the
//     new positions are written in place, double buffered by sweep parity,
//     each 16-byte record carrying the sweep index of the trial that produced
//     it in its fourth word, so a reader validates every record it loads and
//     no device-wide counter or cache flush is needed (agent-coherent
//     accesses only).
#pragma once

#include <type_traits>
#include <utility>

#include "mc_device.hpp"

namespace mcdev {

// Delayed-acceptance surrogate: sizes of the network and of its input.
constexpr int kDaBins = 64;               // bins of each neighbour histogram
constexpr int kDaIn = 2 * kDaBins;        // like- and unlike-charge histograms
constexpr int kDaHid = 128;               // hidden units of both hidden layers
constexpr int kDaParams = kDaIn * kDaHid + kDaHid + kDaHid * kDaHid + kDaHid + kDaHid + 1;

// Device state of a chain's delayed-acceptance stage and its drift monitor.
struct DAState {
    int32_t active;          // 1: two-stage test for moves without a conflict
    int32_t window;          // monitor window in sweeps (launches end on its multiples)
    int64_t fallback_sweep;  // sweep at which the monitor switched to the plain test, -1 = never
    double ref_rate;         // stage-2 rejection rate of stage-1 passes at training time (< 0: no monitor)
    double delta;            // switch to the plain test when a window's rate exceeds ref_rate + delta
    unsigned long long win_pass0, win_rej0;  // counters at the start of the window
    double last_rate;        // rate of the last complete window
    int64_t min_count;       // windows with fewer stage-1 passes are not judged
};

// Description of one chain inside a sweep launch (device memory).
struct ChainDesc {
    int32_t n;           // ions
    int32_t nb;          // groups of 64 (last one padded with inert ions)
    int32_t band;        // look-ahead band in groups, 0..min(kMaxBand, nb-1)
    int32_t wg_count;    // workgroups serving this chain
    int32_t npad;        // nb * 64
    uint32_t chain_id;   // Philox counter word 2
    uint64_t seed;       // Philox key
    double lB;           // Bjerrum length
    double D;            // trial cube side
    double half_uniform; // sigma/2 when every ion has the same diameter
    void* pos;           // versioned positions by sweep parity (see PosIO)
    void* charge;        // T[npad]: q_i
    void* half;          // T[npad]: sigma_i / 2
    const double* wall_a;// double[npad]: R - sigma_i / 2
    GroupRec* rec;       // [kRing]
    unsigned long long* stats;  // [7] counters: moves, accepted, wall, overlap, Metropolis rejections, iterations, early groups
    double* de_group;    // [launch groups] energy change of each group of the launch
    uint8_t* trace_acc;  // [trace_cap]
    double* trace_de;    // [trace_cap]
    int64_t trace_cap;   // moves traced from the start of the chain
    unsigned long long* clk;  // [2] wall clock at the launch start and when the
                              // chain's last group of the launch was published
    // energy bookkeeping and g(r) (auxiliary kernels)
    double* e_partial;   // re-sum partials, one per block of the re-sum launch
    int32_t e_split;     // re-sum blocks per pair of super-rows
    int32_t pad1;
    void* aux;           // EnergyAux
    double* e_state;     // running energy
    double* sweep_tot;   // [max sweeps per launch] scratch of the scan
    double* e_series;    // [e_capacity] running energy after each sweep
    int64_t e_capacity;
    const int32_t* type; // [npad] species index, -1 for padding
    int32_t ntypes;
    int32_t pad0;
    double rdf_rc;       // centres need |x| <= rdf_rc
    unsigned long long* rdf_counts;   // [ntypes * ntypes * bins]
    unsigned long long* rdf_centres;  // [ntypes]
    // ... the cell grid of its pair counts (cubic, over [-R, R]^3)
    int32_t rdf_side;    // cells per side
    int32_t pad2;
    double rdf_org;      // R
    double rdf_inv_h;    // 1 / side of a cell
    int32_t* rdf_cells;  // [rdf_side^3] ions per cell, zero between samples
    int32_t* rdf_start;  // [rdf_side^3 + 1] first ion of each cell in rdf_sorted
    int32_t* rdf_rank;   // [npad] an ion's place in its cell
    void* rdf_sorted;    // T4[npad]: {x, y, z, species} in cell order
    // delayed acceptance (kernels with DA = true only)
    const float* da_w;   // [kDaParams] network parameters (bfloat16 values held in float)
    const uint16_t* da_w1b;  // [128 x 128] W1 as bfloat16, transposed (row = hidden unit)
    const uint16_t* da_w2b;  // [128 x 128] W2 as bfloat16, transposed
    DAState* da;         // monitor state
    double da_rc;        // histogram range
    double da_dr;        // histogram bin width da_rc / 64
    uint32_t* log_feat;  // [log_cap][64] packed byte histograms of logged moves
    double* log_de;      // [log_cap] exact dE
    double* log_deh;     // [log_cap] surrogate dEh (0 when not evaluated)
    uint8_t* log_flags;  // [log_cap] bit0 wall, 1 overlap, 2 conflict, 3 stage-1 reject,
                         //           4 stage-2 reject, 5 accepted, 7 written
    int64_t log_cap;     // moves logged from the start of the chain
};

// A position record is {x, y, z, version}: version = sweep index (mod 2^32)
// of the trial that produced the position; slot pos[s & 1][i] holds the
// result of trial (s, i).  Float path: one 16-byte record.  Double path: two
// 16-byte halves {x, y}, {z, version}; the writer drains the first half
// before storing the second and the reader validates the second half before
// loading the first.
// Pause between two polls of a global-memory slot: the shortest sleep, or
// about 0.85 us (32 x 64 clocks) for a patient reader.
__device__ __forceinline__ void poll_pause(bool patient) {
    if (patient)
        __builtin_amdgcn_s_sleep(32);
    else
        __builtin_amdgcn_s_sleep(1);
}

template <typename T> struct PosIO;

template <> struct PosIO<float> {
    struct Rec { float x, y, z; uint32_t ver; };
    static constexpr uint32_t kBytes = 16;
    static __device__ __forceinline__ Rec load(__amdgpu_buffer_rsrc_t r, uint32_t idx) {
        return __builtin_bit_cast(Rec, __builtin_amdgcn_raw_buffer_load_b128(r, idx * 16u, 0, kCoherent));
    }
    static __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, uint32_t idx, float x, float y,
                                                 float z, uint32_t ver) {
        Rec v{x, y, z, ver};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, v), r, idx * 16u, 0, kCoherent);
    }
    // loads slot idx until its version is `ver` (all lanes with `active`);
    // a patient reader (one whose result is not needed for several groups)
    // polls about once a microsecond instead of back to back
    static __device__ __forceinline__ Rec load_valid(__amdgpu_buffer_rsrc_t r, uint32_t idx, uint32_t ver,
                                                     bool active, const Ctl& ctl, bool patient = false) {
        Rec v{0.f, 0.f, 0.f, ver};
        if (active) v = load(r, idx);
        if (__ballot(active && v.ver != ver) == 0ull) return v;
        PollGuard pg;
        for (;;) {
            poll_pause(patient);
            if (active && v.ver != ver) v = load(r, idx);
            if (__ballot(active && v.ver != ver) == 0ull) break;
            if (pg.stop(ctl)) break;
        }
        return v;
    }
};

template <> struct PosIO<double> {
    struct Rec { double x, y, z; uint32_t ver, pad; };
    struct Lo { double x, y; };
    struct Hi { double z; uint32_t ver, pad; };
    static constexpr uint32_t kBytes = 32;
    static __device__ __forceinline__ Hi load_hi(__amdgpu_buffer_rsrc_t r, uint32_t idx) {
        return __builtin_bit_cast(Hi, __builtin_amdgcn_raw_buffer_load_b128(r, idx * 32u + 16u, 0, kCoherent));
    }
    static __device__ __forceinline__ Lo load_lo(__amdgpu_buffer_rsrc_t r, uint32_t idx) {
        return __builtin_bit_cast(Lo, __builtin_amdgcn_raw_buffer_load_b128(r, idx * 32u, 0, kCoherent));
    }
    static __device__ __forceinline__ void store(__amdgpu_buffer_rsrc_t r, uint32_t idx, double x, double y,
                                                 double z, uint32_t ver) {
        Lo lo{x, y};
        Hi hi{z, ver, 0u};
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, lo), r, idx * 32u, 0, kCoherent);
        drain_memory();
        __builtin_amdgcn_raw_buffer_store_b128(__builtin_bit_cast(u32x4, hi), r, idx * 32u + 16u, 0, kCoherent);
    }
    static __device__ __forceinline__ Rec load_valid(__amdgpu_buffer_rsrc_t r, uint32_t idx, uint32_t ver,
                                                     bool active, const Ctl& ctl, bool patient = false) {
        Hi h{0.0, ver, 0u};
        if (active) h = load_hi(r, idx);
        if (__ballot(active && h.ver != ver) != 0ull) {
            PollGuard pg;
            for (;;) {
                poll_pause(patient);
                if (active && h.ver != ver) h = load_hi(r, idx);
                if (__ballot(active && h.ver != ver) == 0ull) break;
                if (pg.stop(ctl)) break;
            }
        }
        drain_memory();  // the high half is validated before the low half is read
        Lo l{0.0, 0.0};
        if (active) l = load_lo(r, idx);
        return Rec{l.x, l.y, h.z, h.ver, 0u};
    }
};

// Bit masks over one wave's slice of a partner group.
template <int P> struct SliceBits;
template <> struct SliceBits<8> { using type = uint8_t; };
template <> struct SliceBits<16> { using type = uint16_t; };

// Band groups with both-outcome candidates: up to kMaxBand (kDaMaxBand in
// the delayed-acceptance kernels, whose network would otherwise spill).
// The newest kChainSlots of them (g-1, g-2[, g-3]) go to the chain step
// through LDS; the accept masks of the older ones are out before the compute
// waves finish, and each wave resolves its own slice of their candidates
// itself.  (The four-wave float kernels keep two slots: a third would no
// longer let two workgroups share a CU's LDS.  The double kernels run one workgroup
// per CU and take three.  The delayed-acceptance kernels, whose LDS also
// holds the neighbour histograms and the network, take one.)
template <bool DA> constexpr int kBandSlots = DA ? kDaMaxBand : kMaxBand;
// ... and of the float kernels that hold fewer band groups in registers: the
// one for per-ion diameters, whose extra per-partner work leaves no room for
// a fourth (it would spill, and a spilling persistent kernel runs one
// workgroup per CU), and the eight-wave ones, which fit 128 registers so
// that two workgroups (sixteen waves) share a CU.
template <typename T, int M, bool UNIFORM_SIGMA, bool DA>
constexpr int kChainBand = DA ? kBandSlots<DA>
                              : sizeof(T) != 4 ? kMaxBand
                              : M == 8 ? (UNIFORM_SIGMA ? kMaxBandWide : kMaxBandWidePerIon)
                                       : (UNIFORM_SIGMA ? kMaxBand : kMaxBandPerIon);
// LDS chain slots; the eight-wave float kernels take one, which brings their
// LDS to 47.8 KB for two workgroups per CU.
template <typename T, int M, bool DA>
constexpr int kChainSlots = DA ? 1 : (sizeof(T) == 4 ? (M == 8 ? 1 : 2) : 3);
// Partners per wave in a tile of a decided partner group.  The eight-wave
// float kernels take 64: wave w takes every eighth decided group (w, w + 8,
// ... after the oldest) whole, so that a tile's fixed costs (its load and
// version check, the LDS staging and its waits, the double accumulation) fall
// on 64 pair terms a lane instead of 8, and every lane loads.  Measured 12-14 %
// faster where the pair terms bound (N >= 65536); with four waves, 32-partner
// slices were slower (the last decided tile lengthens the hand-off that the
// decision chain waits for).  The other kernels split every group over all
// their waves.
template <typename T, int M, bool DA>
constexpr int kDecidedSlice = (sizeof(T) == 4 && M == 8 && !DA) ? 64 : kGroup / M;
// A compute wave waiting for a partner group more than this many groups
// before its target polls patiently: the chain publishes about one group
// every two microseconds, far slower than a tile takes to compute.
constexpr int kPatientDistance = 6;

// Decided groups this close before the last one the target waits for are taken
// one at a time (at least one group, which empties the ring below).  Nearer, a
// round of four waits for its newest group: ten sweeps with 4 / 8 / 12 / 20 / 32
// of them 0.934 / 0.890 / 0.893 / 0.893 / 0.901 ms at N = 2048, 1.70 / 1.67 / 1.67 /
// 1.67 / 1.67 at 4096, 12.28 / 12.25 / 12.24 / 12.21 / 12.22 at 32768.
constexpr int kQuadMargin = 12;
static_assert(kQuadMargin >= 1, "the ring is emptied in the rounds of one group");
// Entries of a wave's ring of near partners: one partner adds up to 64, and
// the ring is emptied by 64 as soon as it holds that many.
constexpr int kNearRing = 128;

template <typename T, int M, bool DA = false>
struct SweepShared {
    using T4 = typename Prec<T>::T4;
    static constexpr int P = kGroup / M;
    static constexpr int PD = kDecidedSlice<T, M, DA>;
    static constexpr int KB = kBandSlots<DA>;
    static constexpr int LC = kChainSlots<T, M, DA>;
    using SB = typename SliceBits<P>::type;
    // per compute wave: staging of the current partner slice {x, y, z, q}
    // (a decided tile of PD > P partners continues in st_old2 / st_half2)
    // (the float delayed-acceptance kernels stage four decided slices at once)
    static constexpr int SW = sizeof(T) == 4 && DA ? 4 * P : 2 * P;
    T4 st[M][SW];
    __device__ T4* old_of(int w) { return st[w]; }
    __device__ T4* new_of(int w) { return st[w] + P; }
    T st_half[M][P];
    // hand-off from the compute waves to the chain wave (one target at a time)
    double part_s[M][kGroup];   // partial sums over each wave's partners
    uint64_t part_ov[M];        // overlap ballots over final partners
    T part_pn[M][2][kGroup];    // per wave: sums of the positive / negative
                                // corrections still unknown (groups g-1..g-LC, own group)
    // overlap bits per mover i, one 64-bit word over the partners j in which
    // wave w fills the slice of its own partners (bits w P .. w P + P - 1)
    static_assert(sizeof(SB) * M == 8, "the waves' slices tile a 64-bit word");
    alignas(8) SB ovo_own[kGroup][M];    // own group, j < i: overlap with j's old position
    alignas(8) SB ovt_own[kGroup][M];    //                   overlap with j's trial position
    alignas(8) SB ovo_b[LC][kGroup][M];  // group g-1-kb: overlap with j's old / trial position
    alignas(8) SB ovt_b[LC][kGroup][M];
    // corrections, one padded row per mover i (16-byte reads of 4 partners
    // are free of bank conflicts)
    static constexpr int CS = kGroup + (sizeof(T) == 4 ? 4 : 2);
    alignas(16) T c_own[kGroup][CS];    // own group [mover i][partner j]
    alignas(16) T c_b[LC][kGroup][CS];  // group g-1-kb [mover i][partner j]
    alignas(16) T fac[kGroup];          // chain wave: 0/1 factors of a row sum's mask
    int ready;                  // compute waves done filling the hand-off for the current target
    int consumed;               // local target index + 1 the chain wave last released
    // the helper wave's part of the chain step: band corrections of groups
    // g-LC..g-2 (summed oldest first), their overlap ballot, its factor row,
    // and the local target index + 1 it last finished
    double h_corr[LC > 1 ? kGroup : 1];
    uint64_t h_ov;
    alignas(LC > 1 ? 16 : alignof(T)) T fac_h[LC > 1 ? kGroup : 1];
    int h_done;
    // delayed acceptance: per mover, byte histograms of neighbour distances at
    // the old position (bytes 0..127) and at the trial position (128..255),
    // each like-charged bins 0..63 then unlike-charged; conflict ballots of
    // the waves; the surrogate's dEh
    uint32_t hist[DA ? kGroup : 1][DA ? 65 : 1];   // rows padded to 65 words (bank-conflict free)
    uint64_t part_conf[DA ? M : 1];
    double deh[DA ? kGroup : 1];
    float net_out[DA ? 2 * kGroup : 1];       // network output of each (position, mover)
    alignas(16) float bias[DA ? 3 : 1][DA ? kDaHid : 4];  // b1, b2, w3 and ...
    float bias3;                                          // ... b3; loaded once per launch
    // the network's two matrices, transposed ([hidden unit][input]), as
    // bfloat16, rows padded to 132 values (8-byte reads free of bank
    // conflicts); loaded once per launch
    static constexpr bool kWtsLds = DA && sizeof(T) == 4;  // (the double kernel reads them from memory)
    alignas(16) uint16_t wts[kWtsLds ? 2 * kDaHid : 1][kWtsLds ? kDaIn + 4 : 1];
    static_assert(!kWtsLds || sizeof(wts[0]) % 8 == 0, "rows of 8-byte pieces");
    // a decided tile's partners beyond the first P
    T4 st_old2[M][PD > P ? PD - P : 1];
    T st_half2[M][PD > P ? PD - P : 1];
    // delayed acceptance: per wave, a ring of partners found near a mover
    // {x, y, z, mover lane + 64 if unlike}, binned 64 at a time
    T4 near[DA ? M : 1][DA ? kNearRing : 1];
};

// The 64-bit word of overlap bits that the waves' slices tile.
template <typename SB, int M>
__device__ __forceinline__ uint64_t slice_word(const SB (&w)[M]) {
    uint64_t v;
    __builtin_memcpy(&v, &w[0], sizeof(v));
    return v;
}

// Bounded LDS wait used between the compute waves and the chain wave.
__device__ __forceinline__ void wait_lds_at_least(int* flag, int want, const Ctl& ctl) {
    if (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) < want) {
        PollGuard pg;
        for (;;) {
            __builtin_amdgcn_s_sleep(1);
            if (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP) >= want) break;
            if (pg.stop(ctl)) break;
        }
    }
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup");
}

// sum_j [bit j of mask] row[j] over the 64 partners, branch free.  The
// (wave-uniform) mask is spread over the lanes as 0/1 factors in LDS, one
// per partner, written lane-parallel; every lane then reads the factors as
// broadcasts beside its own row and multiply-adds: one vector instruction
// per partner (fma(1, v, a) rounds exactly as a + v, and fma(0, v, a) = a).
// 16-byte loads; fixed order, four independent accumulators: deterministic.
// Only the chain wave calls it, on its own factor row.
template <typename T>
__device__ __forceinline__ T masked_row_sum(const T* __restrict__ row, T* fac, uint64_t mask) {
    constexpr int V = 16 / (int)sizeof(T);  // values per 16-byte read
    typedef T VT __attribute__((ext_vector_type(V)));
    const int lane = threadIdx.x & 63;
    wave_lds_sync();  // the previous call's factor reads come first
    fac[lane] = (T)(uint32_t)((mask >> lane) & 1ull);
    wave_lds_sync();
    T a[4] = {0, 0, 0, 0};
#pragma unroll
    for (int j = 0; j < kGroup; j += V) {
        const VT v = *reinterpret_cast<const VT*>(row + j);
        const VT f = *reinterpret_cast<const VT*>(fac + j);
#pragma unroll
        for (int k = 0; k < V; ++k) a[(j + k) & 3] = Prec<T>::fma_exact(f[k], v[k], a[(j + k) & 3]);
    }
    return (a[0] + a[1]) + (a[2] + a[3]);
}

// The row sum of mask `to` from that of mask `from` (at most kFewFlips bits
// apart): for every bit that differs, in ascending order (a fixed order:
// deterministic), adds the entry if the bit is set in `to` and subtracts it
// otherwise.  Cheaper than a full masked_row_sum for a few flips: a scalar
// bit scan and one LDS read per flip, the reads issued before the first add.
constexpr int kFewFlips = 4;
template <typename T>
__device__ __forceinline__ T row_sum_update(const T* __restrict__ row, T own, uint64_t from, uint64_t to) {
    uint64_t f = from ^ to;
    T v[kFewFlips];
    bool up[kFewFlips];
#pragma unroll
    for (int q = 0; q < kFewFlips; ++q) {
        v[q] = 0;
        up[q] = true;
        if (f) {
            const int j = __builtin_ctzll(f);
            f &= f - 1;
            v[q] = row[j];
            up[q] = ((to >> j) & 1ull) != 0;
        }
    }
#pragma unroll
    for (int q = 0; q < kFewFlips; ++q) own = up[q] ? own + v[q] : own - v[q];
    return own;
}

// Publishes group g: its accept mask in the group record, then the new
// positions (trial position if accepted, old one otherwise), each tagged with
// the sweep index.
template <typename T>
__device__ __forceinline__ void publish_group(__amdgpu_buffer_rsrc_t rec_r, __amdgpu_buffer_rsrc_t pos_r,
                                              int64_t g, int64_t s, int npad, int ion, uint64_t acc,
                                              bool dec, T xi, T yi, T zi, T txi, T tyi, T tzi) {
    using IO = PosIO<T>;
    if ((threadIdx.x & 63) == 0) {
        GroupRec r;
        r.tag = (uint32_t)(g + 1);
        r.spare = 0;
        r.acc = acc;
        store_rec(rec_r, (uint32_t)(g & (kRing - 1)), r);
    }
    if (dec)
        IO::store(pos_r, (uint32_t)((s & 1) * npad + ion), txi, tyi, tzi, (uint32_t)s);
    else
        IO::store(pos_r, (uint32_t)((s & 1) * npad + ion), xi, yi, zi, (uint32_t)s);
}

// The sequential part of target group g, run by wave 0 after its own share
// of the pair terms: combine the waves' hand-off, decide the group (from the
// bounds, or after the band groups' accept masks by fixed-point iteration)
// and publish.
// Per-mover inputs of the chain step that do not depend on the other moves,
// formed at the start of the target's work, long before its decisions are
// due: the hard-wall test of the trial position (Sec. 5.2), the Metropolis
// threshold -log(u3) (u3 < exp(-dE) is evaluated as dE < -log(u3); the two
// forms can only disagree within rounding of the threshold itself, and
// dE <= 0 always accepts), and l_B q_i.
struct MoverInputs {
    bool wall;
    double thr;
    double lq;
    double log_u2;  // two-stage test: log of the second stage's uniform
};

template <typename T>
__device__ __forceinline__ MoverInputs mover_inputs(const ChainDesc& cd, int ion, T qi, T txi, T tyi, T tzi,
                                                    uint32_t w3) {
    MoverInputs mi;
    const double a = cd.wall_a[ion];
    const double X = (double)txi, Y = (double)tyi, Z = (double)tzi;
    int wall = (X * X + Y * Y + Z * Z > a * a) ? 1 : 0;
    double thr = -log(accept_uniform(w3));
    double lq = cd.lB * (double)qi;
    // evaluated here, not sunk to their first use behind the hand-off wait
    asm volatile("" : "+v"(wall), "+v"(thr), "+v"(lq));
    mi.wall = wall != 0;
    mi.thr = thr;
    mi.lq = lq;
    return mi;
}

// Counters of one workgroup, added to the chain's stats at the end.
struct WgCounters {
    unsigned long long moves = 0, acc = 0, wall = 0, ov = 0, iters = 0, early = 0;
    unsigned long long da_moves = 0, conflicts = 0, s1_rej = 0, s2_rej = 0, s1_pass = 0;
};

// The helper wave's part of the chain step of target g (wave 1, after its
// own hand-off): once every wave's candidates are in, the band corrections
// of groups g-LC..g-2 as their accept masks arrive, oldest first, for the
// chain wave -- which meanwhile solves the own group's fixed point.
template <typename T, int M, bool DA>
__device__ __forceinline__ void band_helper(SweepShared<T, M, DA>& sh, __amdgpu_buffer_rsrc_t rec_r, int64_t g,
                                            int t, int band, const Ctl& ctl) {
    constexpr int LC = SweepShared<T, M, DA>::LC;
    const int lane = threadIdx.x & 63;
    wait_lds_at_least(&sh.ready, M, ctl);
    double corr = 0.0;
    bool ov = false;
#pragma unroll
    for (int kb = LC - 1; kb >= 1; --kb) {
        if (kb < band) {
            const GroupRec r = wait_rec(rec_r, g - 1 - kb, ctl);
            corr += (double)masked_row_sum<T>(sh.c_b[kb][lane], sh.fac_h, r.acc);
            const uint64_t ovo = slice_word(sh.ovo_b[kb][lane]), ovt = slice_word(sh.ovt_b[kb][lane]);
            ov |= ((r.acc & ovt) | (~r.acc & ovo)) != 0;
        }
    }
    sh.h_corr[lane] = corr;
    const uint64_t ob = __ballot(ov);
    if (lane == 0) sh.h_ov = ob;
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
    if (lane == 0) __hip_atomic_store(&sh.h_done, t + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
}

#ifdef MC_TIMELINE
constexpr int kTlSlots = 32;  // diagnostic build: stamps per group in the dE trace buffer
#endif

template <typename T, int M, bool DA>
__device__ __forceinline__ void chain_step(SweepShared<T, M, DA>& sh, const ChainDesc& cd,
                                           __amdgpu_buffer_rsrc_t pos_r, __amdgpu_buffer_rsrc_t rec_r,
                                           int64_t g_begin, int64_t g, int t,
                                           T xi, T yi, T zi, T txi, T tyi, T tzi, const MoverInputs& mi, bool da_active,
                                           const Ctl& ctl, WgCounters& ctr)
{
    const int lane = threadIdx.x & 63;
    const int n = cd.n, nb = cd.nb, band = cd.band;
    const int npad = nb * kGroup;
    const int64_t s = g / nb;
    const int b = (int)(g - s * nb);
    const int ion = b * kGroup + lane;
    const bool valid = ion < n;
    const bool wall = mi.wall;
    const double thr = mi.thr;

#ifdef MC_TIMELINE
    // diagnostic build only: per-group wall-clock stamps in the dE trace buffer
    uint64_t tl0 = wall_clock64(), tl1 = 0, tl2 = 0, tl3 = 0, tl4 = 0, tl5 = 0, tl6 = 0, tlA = 0, tlB = 0, tlC = 0;
    uint64_t tlE = 0, tlR = 0, tlN = 0, tlN1 = 0;  // early check done, first row sum done, row sums (in the first solve)
#endif
    // the waves' partial sums
    wait_lds_at_least(&sh.ready, M, ctl);
#ifdef MC_TIMELINE
    tl1 = wall_clock64();
#endif
    double St = 0.0;
    constexpr int LC = SweepShared<T, M, DA>::LC;
    uint64_t ovo = 0, ovt = 0, ovob[LC], ovtb[LC];
    bool ovb = false;
    T cp = 0, cn = 0;
#pragma unroll
    for (int w = 0; w < M; ++w) {
        cp += sh.part_pn[w][0][lane];
        cn += sh.part_pn[w][1][lane];
        St += sh.part_s[w][lane];
        ovb |= ((sh.part_ov[w] >> lane) & 1ull) != 0;
    }
    ovo = slice_word(sh.ovo_own[lane]);
    ovt = slice_word(sh.ovt_own[lane]);
#pragma unroll
    for (int kb = 0; kb < LC; ++kb) {
        ovob[kb] = slice_word(sh.ovo_b[kb][lane]);
        ovtb[kb] = slice_word(sh.ovt_b[kb][lane]);
    }

#ifdef MC_TIMELINE
    tlA = wall_clock64();
#endif
    // Delayed acceptance (two-stage rule): a move without a conflict passes
    // stage 1 when dEh <= 0 or u3 < exp(-dEh), i.e. dEh < thr, and is then
    // accepted when dE - dEh <= 0 or u2 < exp(-(dE - dEh)), i.e. when
    // dE <= dEh or dE < dEh - log(u2).  The plain rule is the special case
    // shift = 0, thr_eff = thr; a stage-1 rejection sets both to -inf.
    double shift = 0.0, thr_eff = thr, deh = 0.0;
    bool conflict = false, da_lane = false, s1_rej = false;
    if constexpr (DA) {
        uint64_t cm = 0;
#pragma unroll
        for (int w = 0; w < M; ++w) cm |= sh.part_conf[w];
        conflict = ((cm >> lane) & 1ull) != 0;
        if (da_active && valid && !conflict) {
            da_lane = true;
            deh = sh.deh[lane];
            if (deh <= 0.0 || deh < thr) {
                shift = deh;
                thr_eff = deh - mi.log_u2;
            } else {
                s1_rej = true;
                shift = thr_eff = -1.0e300;
            }
        }
    }

    // ---- decisions.  dE = lB q (St + sum_kb corr_{g-1-kb} + own): the band
    // corrections and the own-group term stay unknown until the accept bits
    // of groups g-band..g-1 and of this group are known, but they are bounded
    // by the sums of their negative and positive candidate terms.  When the
    // threshold lies outside every lane's interval (with a margin far larger
    // than the rounding of these sums) and no hard-core overlap can flip, the
    // group's decisions are certain and are published before the band
    // groups' accept masks have even arrived; the exact dE follows.
    // Otherwise: solve the sequential rule's fixed point for a guess of the
    // pending masks, then correct it as the true masks arrive (below).
    __builtin_amdgcn_s_setprio(3);
    const double lq = mi.lq;
    const bool can = valid && !wall && !ovb;
    uint64_t acc = 0;
    double dE = 0.0;
    bool dec = false;
    int it = 0;
    bool early = false;
    {
        const double lo = St + (double)cn;
        const double hi = St + (double)cp;
        const double e_lo = lq >= 0 ? lq * lo : lq * hi;
        const double e_hi = lq >= 0 ? lq * hi : lq * lo;
        const double span = (double)(cp - cn);
        const double margin = fabs(lq) * (1e-4 * span + 1e-9 * (fabs(St) + 1.0)) + 1e-12;
        uint64_t ov_sure = 0, ov_flip = ovo ^ ovt;
#pragma unroll
        for (int kb = 0; kb < LC; ++kb) {
            ov_sure |= ovob[kb] & ovtb[kb];
            ov_flip |= ovob[kb] ^ ovtb[kb];
        }
        const bool reject_sure = !can || s1_rej || ov_sure != 0 || (ovo & ovt) != 0;
        const bool accept_sure = !reject_sure && ov_flip == 0 && e_hi < thr_eff - margin;
        const bool sure = reject_sure || accept_sure || (ov_flip == 0 && e_lo >= thr_eff + margin);
        // Not in a chain so short that a group whose mask is still unknown
        // here (the newest LC of the band) has this group's ions in its own band: it may
        // still be reading the positions, two sweeps old, that publishing
        // overwrites.
        if (nb > band + (band < LC ? band : LC) && __ballot(!sure) == 0ull) {
            early = true;
            acc = __ballot(accept_sure);
            dec = accept_sure;
            publish_group<T>(rec_r, pos_r, g, s, npad, ion, acc, dec, xi, yi, zi, txi, tyi, tzi);
#ifdef MC_TIMELINE
            tl3 = wall_clock64();
#endif
        }
    }
#ifdef MC_TIMELINE
    tlB = tlE = wall_clock64();
#endif
    // One evaluation of the sequential rule inside the group given an accept
    // mask `a` of the own group (row sum `own`): the decisions every lane
    // would take.  Lane i depends on lanes j < i only (the system is lower
    // triangular), so the iteration a <- rule(a) reaches the one fixed point
    // from any start within kGroup + 1 evaluations, and a mask that the rule
    // reproduces is that fixed point.
    auto rule = [&](double Sx, bool canx, uint64_t a, T own) {
        const bool ovown = ((a & ovt) | (~a & ovo)) != 0;
        dE = lq * (Sx + (double)own);
        dec = canx && !ovown && (dE <= shift || dE < thr_eff);
        return __ballot(dec);
    };
    // iterates from mask a (row sum own) to the fixed point; a step that
    // flips few bits updates the row sum by them instead of summing the row
    auto solve = [&](double Sx, bool canx, uint64_t a, T own) {
        uint64_t na = rule(Sx, canx, a, own);
        ++it;
        while (na != a && it <= kGroup + 2) {
            if (__popcll(na ^ a) <= kFewFlips)
                own = row_sum_update<T>(sh.c_own[lane], own, a, na);
            else
                own = masked_row_sum<T>(sh.c_own[lane], sh.fac, na);
#ifdef MC_TIMELINE
            if (tlN++ == 0) tlR = wall_clock64();
#endif
            a = na;
            na = rule(Sx, canx, a, own);
            ++it;
        }
        acc = na;
        return own;
    };
    double corr = 0.0;  // band corrections of groups g-LC..g-1, oldest first
#ifdef MC_TIMELINE
    tlC = wall_clock64();
#endif
    // groups g-LC..g-2 come from the helper wave: their sum, in the same
    // order, and the overlap ballot
    auto helper_part = [&]() {
        wait_lds_at_least(&sh.h_done, t + 1, ctl);
        corr = sh.h_corr[lane];
        ovb |= ((sh.h_ov >> lane) & 1ull) != 0;
    };
    // group g-1's correction, added to corr once its mask arrives
    auto g1_part = [&]() {
        const GroupRec r = wait_rec(rec_r, g - 1, ctl);
#ifdef MC_TIMELINE
        tl2 = wall_clock64();
#endif
        corr += (double)masked_row_sum<T>(sh.c_b[0][lane], sh.fac, r.acc);
        ovb |= ((r.acc & ovtb[0]) | (~r.acc & ovob[0])) != 0;
    };
    if (early) {
        if (LC > 1 && band >= 2) helper_part();
        if (band >= 1) g1_part();
        // exact energy change of the (already decided) trials
        const T own = acc ? masked_row_sum<T>(sh.c_own[lane], sh.fac, acc) : (T)0;
        dE = lq * ((St + corr) + (double)own);
        it = 1;
    } else {
        // While the accept masks of the chain band groups are on their way,
        // the fixed point is solved for a guess of them (every move
        // rejected).  As the true corrections come in (the helper's, then
        // g-1's) one evaluation confirms the solution, or the iteration goes
        // on from it.
        uint64_t pend = 0;  // overlaps with old positions of pending groups (rejected guess)
#pragma unroll
        for (int kb = 0; kb < LC; ++kb)
            if (kb < band) pend |= ovob[kb];
        T own = solve(St, valid && !wall && !ovb && pend == 0, 0, (T)0);
        if (LC > 1 && band >= 2) {
#ifdef MC_TIMELINE
            tlC = wall_clock64();  // end of the first solve
            tlN1 = tlN;
#endif
            helper_part();
#ifdef MC_TIMELINE
            tlB = wall_clock64();  // helper's part in
#endif
            pend = ovob[0];
            it = 0;
            own = solve(St + corr, valid && !wall && !ovb && pend == 0, acc, own);
        }
        if (band >= 1) {
#ifdef MC_TIMELINE
            tl6 = wall_clock64();
#endif
            g1_part();
#ifdef MC_TIMELINE
            tl4 = wall_clock64();
#endif
            it = 0;
            own = solve(St + corr, valid && !wall && !ovb, acc, own);
        }
#ifdef MC_TIMELINE
        if (band < 1) tl2 = tl4 = tl6 = wall_clock64();
        tl5 = wall_clock64();
#endif
        (void)own;
        publish_group<T>(rec_r, pos_r, g, s, npad, ion, acc, dec, xi, yi, zi, txi, tyi, tzi);
#ifdef MC_TIMELINE
        tl3 = wall_clock64();
#endif
    }
    const uint64_t m_ov = __ballot(valid && !wall && (ovb || ((acc & ovt) | (~acc & ovo)) != 0));

    // ---- release the hand-off buffer
    if (lane == 0) {
        __hip_atomic_store(&sh.ready, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
        __hip_atomic_store(&sh.consumed, t + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
    }

    __builtin_amdgcn_s_setprio(0);
#ifdef MC_TIMELINE
    if (lane == 0 && kTlSlots * (g + 1) <= cd.trace_cap) {
        uint64_t* tl = (uint64_t*)cd.trace_de + kTlSlots * g;
        tl[0] = tl0;
        tl[1] = tl1;
        tl[2] = tl2;
        tl[3] = tl3;
        {
            tl[4] = tl4;
            tl[5] = tl5;
            tl[6] = tl6;
            tl[7] = (uint64_t)it;
            tl[8] = tlA;
            tl[9] = tlB;
            tl[10] = tlC;
            tl[29] = tlE;
            tl[30] = tlR;
            tl[31] = tlN1;
        }
    }
#endif

    const double de_group = __shfl(wave_sum(dec ? dE : 0.0), 0, 64);
#ifndef MC_TIMELINE
    if (valid) {
#else
    if (false) {
#endif
        const int64_t mv = s * (int64_t)n + ion;
        if (mv < cd.trace_cap) {
            cd.trace_acc[mv] = (uint8_t)dec;
            cd.trace_de[mv] = dE;
        }
    }
    if (lane == 0) cd.de_group[g - g_begin] = de_group;
    const uint64_t m_wall = __ballot(valid && wall);
    const uint64_t m_valid = __ballot(valid);
    ctr.moves += __popcll(m_valid);
    ctr.acc += __popcll(acc);
    ctr.wall += __popcll(m_wall);
    ctr.ov += __popcll(m_ov);
    ctr.iters += it;
    ctr.early += early ? 1 : 0;
    if constexpr (DA) {
        const bool ov_final = ((m_ov >> lane) & 1ull) != 0;
        const bool passed = da_lane && !s1_rej && !wall && !ov_final;
        ctr.da_moves += __popcll(__ballot(da_lane));
        ctr.conflicts += __popcll(__ballot(valid && conflict));
        ctr.s1_rej += __popcll(__ballot(s1_rej));
        ctr.s1_pass += __popcll(__ballot(passed));
        ctr.s2_rej += __popcll(__ballot(passed && !dec));
        const int64_t mv = s * (int64_t)n + ion;
        if (valid && mv < cd.log_cap) {
            cd.log_de[mv] = dE;
            cd.log_deh[mv] = deh;
            cd.log_flags[mv] = (uint8_t)(0x80u | (uint32_t)wall | ((uint32_t)ov_final << 1) |
                                         ((uint32_t)conflict << 2) | ((uint32_t)s1_rej << 3) |
                                         ((uint32_t)(passed && !dec) << 4) | ((uint32_t)dec << 5));
        }
    }
}

// Occupancy asked of the compiler (waves per SIMD): two workgroups per CU.
// (the delayed-acceptance kernels take one wave per SIMD: their register use
// would otherwise spill; they run one workgroup per CU)
template <typename T, int M, bool DA = false>
constexpr int kWavesPerEU = DA ? 1 : (sizeof(T) == 4 ? (M == 8 ? 4 : 2) : 1);

// Squared distance in double, summed in the order x, y, z with no fused
// multiply-add: the neighbour-histogram bins and the conflict rule of the
// delayed-acceptance stage are decided on this value.
__device__ __forceinline__ double d2_exact(double ax, double ay, double az, double bx, double by, double bz) {
    const double dx = ax - bx, dy = ay - by, dz = az - bz;
    return dx * dx + dy * dy + dz * dz;
}

// Adds a neighbour at squared distance d2 to byte bin (pos, like/unlike, k)
// of mover `lane`'s histogram (four byte counters per LDS word).
template <typename SH>
__device__ __forceinline__ void da_hist_add(SH& sh, const ChainDesc& cd, float inv_dr, int lane, int pos, bool unlike,
                                            double d2) {
    if (!(d2 < cd.da_rc * cd.da_rc)) return;
    // floor(sqrt(d2) / dr): in float (off by less than 1e-4 up to bin 64)
    // unless that lies next to a bin's edge
    const float v = __builtin_amdgcn_sqrtf((float)d2) * inv_dr;
    const int k = __builtin_fabsf(v - __builtin_rintf(v)) > 1e-3f
                      ? (int)v
                      : (int)__builtin_floor(__builtin_sqrt(d2) / cd.da_dr);
    if (k >= kDaBins) return;
    const int byte = pos * kDaIn + (unlike ? kDaBins : 0) + k;
    atomicAdd(&sh.hist[lane][byte >> 2], 1u << (8 * (byte & 3)));
}

// Delayed-acceptance stage of one target group, run by all 4 waves after the
// last partner tile: logs the movers' histograms, evaluates the network eps
// at both positions of every mover, leaves dEh = l_B (eps(trial) - eps(old))
// in sh.deh and clears the histograms.  Both hidden layers run on the matrix
// cores (v_mfma_f32_32x32x8bf16_1k) as [128 units x 128] x [128 x 128 rows],
// row r = 64 * position + mover, bfloat16 values with float sums: wave w
// takes rows 32 w .. 32 w + 31 and all four 32-unit tiles.  Lane l gives
// A[l % 32][4 (l / 32) + v] (weights, from LDS where the kernel put them at
// its start) and B[4 (l / 32) + v][l % 32], and gets D[8 (i / 4) + 4 (l / 32)
// + i % 4][l % 32]: what it gets of a layer is what it gives of the next, so
// nothing passes through LDS between the layers, and a row's last sum is
// all but four additions within a lane.  Hidden activations are rounded to
// bfloat16.  Bound: latency, on the path from a partner group's accept mask
// to this group's: 4.2 us; as rows x units, with the activations
// through LDS and each output summed over 32 lanes, 7.4 us.
typedef short da_bf16x4 __attribute__((ext_vector_type(4)));
typedef float da_f32x16 __attribute__((ext_vector_type(16)));
typedef float da_f32x2 __attribute__((ext_vector_type(2)));
typedef float da_f32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 da_pair __attribute__((ext_vector_type(2)));

// two floats rounded to bfloat16 (to nearest even), in one word
__device__ __forceinline__ uint32_t bf16_pair(float a, float b) {
    const da_f32x2 v = {a, b};
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, da_pair));
}

// The network's matrix instructions in pairs: tiles t and t + 1 of step j (8
// inputs) of a layer.
struct DaPair {
    int layer, t, j;
};
constexpr DaPair da_pair_at(int p) {
    return p < 32   ? DaPair{0, 2 * (p / 16), p % 16}
           : p < 48 ? DaPair{1, 2 * (p & 1), (p - 32) / 2}
                    : DaPair{1, 2 * ((p - 48) / 8), 8 + p % 8};
}

// f(0), f(1), .., f(N - 1) with constant arguments
template <typename F, int... I>
__device__ __forceinline__ void static_for_each(F& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_each(f, std::make_integer_sequence<int, N>{});
}

// (before_sums() runs when the matrix instructions are out)
template <typename T, int M, typename F>
__device__ __forceinline__ void da_network(SweepShared<T, M, true>& sh, const ChainDesc& cd, int wave, int lane,
                                           bool da_on, int64_t mv0, int n_movers, int64_t g, F&& before_sums) {
#ifdef MC_TIMELINE
    // diagnostic build only: stamps of the network phase after the chain stamps
    uint64_t* tln = (uint64_t*)cd.trace_de + kTlSlots * g + 11;
    const bool stamp = wave == 0 && lane == 0 && kTlSlots * (g + 1) <= cd.trace_cap;
    if (stamp) tln[0] = wall_clock64();
#else
    (void)g;
#endif
    static_assert(M == 4, "the network phase assumes 4 waves");
    const int half = lane >> 5, row = wave * 32 + (lane & 31), mover = row & 63, pos = row >> 6;
    const __amdgpu_buffer_rsrc_t wbr = make_rsrc((void*)cd.da_w1b, (uint32_t)(4u * kDaIn * kDaHid));
    // inputs 8 j + 4 half .. + 3 of hidden unit 32 t + lane % 32 of layer
    // `layer` (the part common to all in one register, worked out here: kept
    // from target to target, an offset each would not fit the registers)
    int w_lane = (lane & 31) * kDaIn + 4 * half;
    if constexpr (!SweepShared<T, M, true>::kWtsLds) asm volatile("" : "+v"(w_lane));
    auto weights = [&](int layer, int t, int j) __attribute__((always_inline)) -> da_bf16x4 {
        if constexpr (SweepShared<T, M, true>::kWtsLds)
            return *reinterpret_cast<const da_bf16x4*>(&sh.wts[layer * kDaHid + 32 * t + (lane & 31)][8 * j + 4 * half]);
        else
            return __builtin_bit_cast(da_bf16x4, __builtin_amdgcn_raw_buffer_load_b64(
                                                     wbr, 2 * w_lane, 2 * ((layer * kDaHid + 32 * t) * kDaIn + 8 * j), 0));
    };
    __syncthreads();  // every histogram add of this target is done
#ifdef MC_TIMELINE
    if (stamp) tln[1] = wall_clock64();
#endif
    // this lane's words of its row: counts 8 j + 4 half .. + 3
    uint32_t words[kDaIn / 8];
#pragma unroll
    for (int j = 0; j < kDaIn / 8; ++j) {
        uint32_t& w = sh.hist[mover][pos * 32 + 2 * j + half];
        words[j] = w;
        w = 0u;
    }
    if (mover < n_movers && mv0 + mover < cd.log_cap) {
        uint32_t* dst = cd.log_feat + (mv0 + mover) * 64 + pos * 32 + half;
#pragma unroll
        for (int j = 0; j < kDaIn / 8; ++j) dst[2 * j] = words[j];
    }
    if (da_on) {
        // The 128 matrix instructions go out as 64 pairs, tiles t and t + 1 of
        // one step of 8 inputs, in an order that leaves the lane work of the
        // finished tiles (bias, relu, rounding, last layer) to run beside
        // the next ones; the weights are loaded kAhead pairs ahead.
        constexpr int kPairs = 64, kAhead = 4;
        da_bf16x4 wt[kAhead][2];
        auto fetch = [&](auto pc) __attribute__((always_inline)) {
            constexpr int p = decltype(pc)::value;
            constexpr DaPair d = da_pair_at(p);
#pragma unroll
            for (int u = 0; u < 2; ++u)
                wt[p % kAhead][u] = weights(d.layer, d.t + u, d.j);
        };
        // (one address for every bias read, worked out here: an address each
        // would be kept from target to target, a register each)
        typedef __attribute__((address_space(3))) const da_f32x4 lds_f32x4;
        lds_f32x4* bias = (lds_f32x4*)&sh.bias[0][4 * half];
        asm volatile("" : "+v"(bias));
        uint2 x[kDaIn / 8], h[kDaHid / 8];
        auto convert = [&](int j) {
            // counts up to 255 are bfloat16 values: the upper halves of the floats
            uint32_t f[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) f[v] = __builtin_bit_cast(uint32_t, (float)((words[j] >> (8 * v)) & 0xFFu));
            x[j] = make_uint2(__builtin_amdgcn_perm(f[1], f[0], 0x07060302u),
                              __builtin_amdgcn_perm(f[3], f[2], 0x07060302u));
        };
        da_f32x16 acc1[4], acc2[4];
        // bf16(relu(acc + bias)) of units 8 j + 4 half .. + 3
        auto activation = [&](const da_f32x16 (&acc)[4], int which, int j) {
            const da_f32x4 b = bias[which * (kDaHid / 4) + 2 * j];
            const float bv[4] = {b.x, b.y, b.z, b.w};
            float r[4];
#pragma unroll
            for (int v = 0; v < 4; ++v) {
                const float z = acc[j / 4][4 * (j & 3) + v] + bv[v];
                r[v] = z > 0.f ? z : 0.f;
            }
            return make_uint2(bf16_pair(r[0], r[1]), bf16_pair(r[2], r[3]));
        };
        // last layer: sum over the units of bf16(relu(Z2 + b2)) w3; unit
        // 32 t + c, c = 8 q + 4 half + v: over t in order, then over the bits
        // of c from the lowest
        float part[4][4];
        auto last_layer = [&](int j) {
            const uint2 a = activation(acc2, 1, j);
            const da_f32x4 w = bias[2 * (kDaHid / 4) + 2 * j];
            const float wv[4] = {w.x, w.y, w.z, w.w};
            const uint32_t hb[4] = {a.x << 16, a.x & 0xFFFF0000u, a.y << 16, a.y & 0xFFFF0000u};
#pragma unroll
            for (int v = 0; v < 4; ++v)
                part[j & 3][v] = __builtin_fmaf(__builtin_bit_cast(float, hb[v]), wv[v], j < 4 ? 0.f : part[j & 3][v]);
        };
        static_for<kAhead>(fetch);
        convert(0);
        convert(1);
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc1[t][r] = acc2[t][r] = 0.f;
        static_for<kPairs>([&](auto pc) __attribute__((always_inline)) {
            constexpr int p = decltype(pc)::value;
            constexpr DaPair d = da_pair_at(p);
            const da_bf16x4 in = __builtin_bit_cast(da_bf16x4, d.layer ? h[d.j] : x[d.j]);
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                da_f32x16& c = d.layer ? acc2[d.t + u] : acc1[d.t + u];
                c = __builtin_amdgcn_mfma_f32_32x32x8bf16_1k(wt[p % kAhead][u], in, c, 0, 0, 0);
            }
            if constexpr (p + kAhead < kPairs) fetch(std::integral_constant<int, p + kAhead>{});
            if constexpr (p + 2 < 16) convert(p + 2);
            if constexpr (p >= 16 && p < 48 && (p & 1)) h[(p - 16) / 2] = activation(acc1, 0, (p - 16) / 2);
            if constexpr (p > 56) last_layer(p - 57);
            __builtin_amdgcn_sched_barrier(0);
#ifdef MC_TIMELINE
            if (p == 31 && stamp) tln[2] = wall_clock64();
#endif
        });
        before_sums();
#pragma unroll
        for (int j = 7; j < 16; ++j) last_layer(j);
        float sum[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            sum[q] = (part[q][0] + part[q][1]) + (part[q][2] + part[q][3]);
            sum[q] += __shfl_xor(sum[q], 32, 64);
        }
        sh.net_out[row] = (sum[0] + sum[1]) + (sum[2] + sum[3]);
    } else {
        before_sums();
    }
    __syncthreads();  // outputs complete, histograms clear
#ifdef MC_TIMELINE
    if (stamp) tln[3] = wall_clock64();
#endif
    if (da_on && wave == 0) {
        const float b3 = sh.bias3;
        const float o0 = b3 + sh.net_out[lane], o1 = b3 + sh.net_out[64 + lane];
        sh.deh[lane] = cd.lB * ((double)o1 - (double)o0);
    }
}

// One workgroup's share of one chain for sweeps s0 .. s0 + n_sweeps - 1:
// the targets g = k_wg (mod the chain's workgroup count).
template <typename T, int M, bool UNIFORM_SIGMA, bool DA>
__device__ __forceinline__ void sweep_chain(SweepShared<T, M, DA>& sh, const ChainDesc& cd, const int k_wg,
                                            uint32_t s0, int32_t n_sweeps, const Ctl& ctl, const int wave,
                                            const int lane)
{
    using T4 = typename Prec<T>::T4;
    using IO = PosIO<T>;
    constexpr int P = kGroup / M;
    constexpr int KB = kChainBand<T, M, UNIFORM_SIGMA, DA>;
    constexpr int LC = SweepShared<T, M, DA>::LC;
    static_assert(KB >= LC, "the chain step's band slots are band groups");
    using SB = typename SliceBits<P>::type;

    const int tid = 64 * wave + lane;  // (threadIdx.x itself would hold a register throughout)
    const int nb = cd.nb, band = cd.band;
    const int npad = nb * kGroup;
    const __amdgpu_buffer_rsrc_t pos_r = make_rsrc(cd.pos, (uint32_t)(2u * npad * IO::kBytes));
    const __amdgpu_buffer_rsrc_t rec_r = make_rsrc(cd.rec, (uint32_t)(kRing * sizeof(GroupRec)));
    const T* __restrict__ charge = (const T*)cd.charge;
    const T* __restrict__ half = (const T*)cd.half;
    const T D = (T)cd.D;
    const T hu = (T)cd.half_uniform;
    const int64_t g_begin = (int64_t)s0 * nb;
    const int64_t g_end = g_begin + (int64_t)n_sweeps * nb;

    if (tid == 0) {
        // one store each (a merged 64-bit store of zeros has kept a register
        // pair live through the whole kernel)
        __hip_atomic_store(&sh.ready, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_store(&sh.consumed, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        __hip_atomic_store(&sh.h_done, 0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
        if (k_wg == 0) cd.clk[0] = wall_clock64();
    }
    if constexpr (DA) {
        static_assert(sizeof(sh.hist) == sizeof(uint32_t) * kGroup * 65, "histogram rows");
        for (int k = tid; k < kGroup * 65; k += 64 * M) (&sh.hist[0][0])[k] = 0u;
    }
    // the delayed-acceptance switch is constant during a launch (the drift
    // monitor changes it between launches)
    const bool da_on = DA && cd.da != nullptr && cd.da->active != 0 && cd.da_w != nullptr;
    const float inv_dr = DA ? (float)(1.0 / cd.da_dr) : 0.f;
    if constexpr (DA) {
        if (da_on) {
            if (tid == 0) sh.bias3 = cd.da_w[kDaParams - 1];
            for (int k = tid; k < 3 * kDaHid; k += 64 * M) {
                const int u = k % kDaHid, o_b2 = kDaIn * kDaHid + kDaHid + kDaHid * kDaHid;
                sh.bias[k / kDaHid][u] = cd.da_w[(k < kDaHid ? kDaIn * kDaHid : k < 2 * kDaHid ? o_b2 : o_b2 + kDaHid) + u];
            }
        }
    }
    if constexpr (SweepShared<T, M, DA>::kWtsLds) {
        if (da_on) {
            static_assert(kDaIn == kDaHid, "both matrices are 128 x 128");
            for (int k = tid; k < 2 * kDaHid * kDaIn / 4; k += 64 * M) {
                const int row = k / (kDaIn / 4), c4 = k % (kDaIn / 4);  // row of the two stacked matrices
                const uint16_t* src = row < kDaHid ? cd.da_w1b + row * kDaIn : cd.da_w2b + (row - kDaHid) * kDaIn;
                *reinterpret_cast<uint2*>(&sh.wts[row][4 * c4]) = *reinterpret_cast<const uint2*>(src + 4 * c4);
            }
        }
    }
    __syncthreads();

    WgCounters ctr;
    {
        int t = 0;
        for (int64_t g = g_begin + k_wg; g < g_end; g += cd.wg_count, ++t) {
            const int64_t s = g / nb;
            const int b = (int)(g - s * nb);
            const int ion = b * kGroup + lane;

            // the movers: old position = result of the group's previous trial
            const auto xr = IO::load_valid(pos_r, (uint32_t)(((s - 1) & 1) * npad + ion), (uint32_t)(s - 1),
                                           true, ctl);
            const T xi = xr.x, yi = xr.y, zi = xr.z, qi = charge[ion];
            const uint4 wd = move_words(cd.seed, cd.chain_id, (uint32_t)s, (uint32_t)ion);
            const T txi = trial_coord(xi, wd.x, D), tyi = trial_coord(yi, wd.y, D),
                    tzi = trial_coord(zi, wd.z, D);
            const T hi = UNIFORM_SIGMA ? hu : half[ion];
            MoverInputs mi{};
            if (wave == 0) mi = mover_inputs(cd, ion, qi, txi, tyi, tzi, wd.w);
            if constexpr (DA) {
                if (wave == 0 && da_on) {  // here, not in the chain step that the next groups wait for
                    mi.log_u2 = log(accept_uniform(move_words(cd.seed, cd.chain_id, (uint32_t)s, (uint32_t)ion, 2u).x));
                    asm volatile("" : "+v"(mi.log_u2));
                }
            }

#ifdef MC_TIMELINE
            if (!DA && wave == 0 && lane == 0 && kTlSlots * (g + 1) <= cd.trace_cap)
                ((uint64_t*)cd.trace_de)[kTlSlots * g + 11] = wall_clock64();
#endif
            double S = 0.0;     // sum_j q_j (1/|x~_i - x_j| - 1/|x_i - x_j|)
            bool ov = false;    // overlap with a partner whose position is final
            bool conf = false;  // delayed acceptance: a pending partner is near (conflict rule)

            // ---- own group: both outcomes of every partner j != i
            T c_own[P];
            SB ovo_own = 0, ovt_own = 0;
            {
                if (lane >= wave * P && lane < wave * P + P) {
                    const int m = lane - wave * P;
                    sh.old_of(wave)[m] = mk4<T>(xi, yi, zi, qi);
                    sh.new_of(wave)[m] = mk4<T>(txi, tyi, tzi, qi);
                    sh.st_half[wave][m] = hi;
                }
                wave_lds_sync();
                T sf = 0;
#pragma unroll
                for (int m = 0; m < P; ++m) {
                    const int j = wave * P + m;
                    const T4 po = sh.old_of(wave)[m];
                    const T4 pt = sh.new_of(wave)[m];
                    const T hj = UNIFORM_SIGMA ? hu : sh.st_half[wave][m];
                    const T s_ij = hi + hj;
                    const T d2o = Prec<T>::norm2(po.x - xi, po.y - yi, po.z - zi);
                    const T d2ot = Prec<T>::norm2(po.x - txi, po.y - tyi, po.z - tzi);
                    const T d2t = Prec<T>::norm2(pt.x - xi, pt.y - yi, pt.z - zi);
                    const T d2tt = Prec<T>::norm2(pt.x - txi, pt.y - tyi, pt.z - tzi);
                    const T o = po.w * (Prec<T>::rinv(d2ot) - Prec<T>::rinv(d2o));
                    const T tt = pt.w * (Prec<T>::rinv(d2tt) - Prec<T>::rinv(d2t));
                    const bool oo = d2ot < s_ij * s_ij, ot = d2tt < s_ij * s_ij;
                    if (j > lane) {
                        sf += o;
                        ov |= oo;
                        c_own[m] = 0;
                    } else if (j < lane) {
                        sf += o;
                        c_own[m] = tt - o;
                        ovo_own |= (SB)((SB)oo << m);
                        ovt_own |= (SB)((SB)ot << m);
                    } else {
                        c_own[m] = 0;
                    }
                    if constexpr (DA) {
                        if (j > lane) {  // not moved yet: its current position counts
                            const double qq = (double)po.w * (double)qi;
                            if (qq != 0.0) {
                                da_hist_add(sh, cd, inv_dr, lane, 0, qq < 0.0, d2_exact(xi, yi, zi, po.x, po.y, po.z));
                                da_hist_add(sh, cd, inv_dr, lane, 1, qq < 0.0, d2_exact(txi, tyi, tzi, po.x, po.y, po.z));
                            }
                        } else if (j < lane) {  // decision pending: conflict rule
                            const double rc2 = cd.da_rc * cd.da_rc;
                            conf |= d2_exact(xi, yi, zi, po.x, po.y, po.z) < rc2 ||
                                    d2_exact(xi, yi, zi, pt.x, pt.y, pt.z) < rc2 ||
                                    d2_exact(txi, tyi, tzi, po.x, po.y, po.z) < rc2 ||
                                    d2_exact(txi, tyi, tzi, pt.x, pt.y, pt.z) < rc2;
                        }
                    }
                }
                S += (double)sf;
                wave_lds_sync();
            }

            // ---- band groups g-1..g-band: both outcomes, evaluated ahead of their decisions
            T c_band[KB][P];
            SB ovo_band[KB], ovt_band[KB];
#pragma unroll
            for (int kb = 0; kb < KB; ++kb) {
                ovo_band[kb] = 0;
                ovt_band[kb] = 0;
#pragma unroll
                for (int m = 0; m < P; ++m) c_band[kb][m] = 0;
                if (kb < band) {
                    const int64_t gp = g - 1 - kb;
                    const int64_t sp = floor_div(gp, nb);
                    const int bp = (int)(gp - sp * nb);
                    // old position of j = result of its trial one sweep before
                    const int j = bp * kGroup + wave * P + (lane < P ? lane : 0);
                    const auto pr = IO::load_valid(pos_r, (uint32_t)(((sp - 1) & 1) * npad + j),
                                                   (uint32_t)(sp - 1), lane < P, ctl);
                    if (lane < P) {
                        const T qj = charge[j];
                        const uint4 wj = move_words(cd.seed, cd.chain_id, (uint32_t)sp, (uint32_t)j);
                        sh.old_of(wave)[lane] = mk4<T>(pr.x, pr.y, pr.z, qj);
                        sh.new_of(wave)[lane] = mk4<T>(trial_coord((T)pr.x, wj.x, D), trial_coord((T)pr.y, wj.y, D),
                                                        trial_coord((T)pr.z, wj.z, D), qj);
                        if (!UNIFORM_SIGMA) sh.st_half[wave][lane] = half[j];
                    }
                    wave_lds_sync();
                    T sf = 0;
#pragma unroll
                    for (int m = 0; m < P; ++m) {
                        const T4 po = sh.old_of(wave)[m];
                        const T4 pt = sh.new_of(wave)[m];
                        const T hj = UNIFORM_SIGMA ? hu : sh.st_half[wave][m];
                        const T s_ij = hi + hj;
                        const T d2o = Prec<T>::norm2(po.x - xi, po.y - yi, po.z - zi);
                        const T d2ot = Prec<T>::norm2(po.x - txi, po.y - tyi, po.z - tzi);
                        const T d2t = Prec<T>::norm2(pt.x - xi, pt.y - yi, pt.z - zi);
                        const T d2tt = Prec<T>::norm2(pt.x - txi, pt.y - tyi, pt.z - tzi);
                        const T o = po.w * (Prec<T>::rinv(d2ot) - Prec<T>::rinv(d2o));
                        const T tt = pt.w * (Prec<T>::rinv(d2tt) - Prec<T>::rinv(d2t));
                        sf += o;
                        c_band[kb][m] = tt - o;
                        ovo_band[kb] |= (SB)((SB)(d2ot < s_ij * s_ij) << m);
                        ovt_band[kb] |= (SB)((SB)(d2tt < s_ij * s_ij) << m);
                        if constexpr (DA) {
                            if (gp >= 0) {  // decision pending: conflict rule
                                const double rc2 = cd.da_rc * cd.da_rc;
                                conf |= d2_exact(xi, yi, zi, po.x, po.y, po.z) < rc2 ||
                                        d2_exact(xi, yi, zi, pt.x, pt.y, pt.z) < rc2 ||
                                        d2_exact(txi, tyi, tzi, po.x, po.y, po.z) < rc2 ||
                                        d2_exact(txi, tyi, tzi, pt.x, pt.y, pt.z) < rc2;
                            } else {
                                // before the chain's first group: nothing moved, the
                                // ion sits at its starting position, which counts
                                const double qq = (double)po.w * (double)qi;
                                if (qq != 0.0) {
                                    da_hist_add(sh, cd, inv_dr, lane, 0, qq < 0.0, d2_exact(xi, yi, zi, po.x, po.y, po.z));
                                    da_hist_add(sh, cd, inv_dr, lane, 1, qq < 0.0, d2_exact(txi, tyi, tzi, po.x, po.y, po.z));
                                }
                            }
                        }
                    }
                    S += (double)sf;
                    wave_lds_sync();
                }
            }

            // the candidates of group g-1 and of the own group for the chain
            // wave: overlap slices, the sums of their positive and negative
            // parts (bounds of the corrections still unknown) and the rows
            auto hand_off_candidates = [&]() {
                sh.ovo_own[lane][wave] = ovo_own;
                sh.ovt_own[lane][wave] = ovt_own;
#pragma unroll
                for (int kb = 0; kb < LC; ++kb) {
                    sh.ovo_b[kb][lane][wave] = ovo_band[kb];
                    sh.ovt_b[kb][lane][wave] = ovt_band[kb];
                }
                T cp = 0, cn = 0;
#pragma unroll
                for (int m = 0; m < P; ++m) {
#pragma unroll
                    for (int kb = 0; kb < LC; ++kb) {
                        cp += c_band[kb][m] > 0 ? c_band[kb][m] : (T)0;
                        cn += c_band[kb][m] < 0 ? c_band[kb][m] : (T)0;
                    }
                    cp += c_own[m] > 0 ? c_own[m] : (T)0;
                    cn += c_own[m] < 0 ? c_own[m] : (T)0;
                }
                sh.part_pn[wave][0][lane] = cp;
                sh.part_pn[wave][1][lane] = cn;
#pragma unroll
                for (int m = 0; m < P; ++m) {
                    sh.c_own[lane][wave * P + m] = c_own[m];
#pragma unroll
                    for (int kb = 0; kb < LC; ++kb)
                        sh.c_b[kb][lane][wave * P + m] = c_band[kb][m];  // zero beyond the band
                }
            };
            // complete from here on: handed off now, off the critical path,
            // once the chain wave has released the previous target
            wait_lds_at_least(&sh.consumed, t, ctl);
            hand_off_candidates();

            // ---- decided partner groups g-nb+1 .. g-band-1, in stream order.  The next
            // tile is loaded speculatively while this one is computed (float path); a
            // record whose version is not the expected one yet is loaded again.
            // A round of tiles covers KD decided groups, each shared by M / KD
            // waves with PD partners a wave: KD = 1 in most kernels (every
            // wave a P-partner slice of every group), KD = 8 in the eight-wave
            // float kernels (every wave one group whole).
            {
                constexpr int PD = kDecidedSlice<T, M, DA>;
                constexpr int KD = PD / P;
                static_assert(KD * P == PD && M % KD == 0 && (!DA || KD == 1), "decided tiles");
                const int64_t g_last = g - band - 1;
                int64_t sp = (b + 1 < nb) ? s - 1 : s;   // sweep and group of g-nb+1
                int bp = (b + 1 < nb) ? b + 1 : 0;
                const int dphase = wave / (M / KD);      // this wave's first group: g-nb+1+dphase
                for (int k = 0; k < dphase; ++k)
                    if (++bp == nb) {
                        bp = 0;
                        ++sp;
                    }
                const int jl = (wave % (M / KD)) * PD + (lane < PD ? lane : 0);
                typename IO::Rec nxt{};
                bool have_next = false;
                // uniform diameters: overlap with any of these partners iff the
                // smallest trial distance is below the contact distance
                T d2t_min = (T)3.0e38;
                // Delayed acceptance: the partners within range of a mover are
                // few (one in a thousand pairs in a large system), so they
                // are only noted in the pair loop, as a ballot per partner,
                // and go to the wave's ring; the exact distances and bins (a
                // double sqrt and division each) are worked out for 64 of
                // them at a time, a lane each.  Bound: the pair terms.
                // Binning each tile's few at once, one or two lanes at work,
                // cost every tile that had any the whole chain of double
                // operations.
                uint32_t q_in = 0, q_out = 0;
                auto bin_near = [&](uint32_t count) {
                    wave_lds_sync();
                    const uint32_t k = (uint32_t)lane < count ? (uint32_t)lane : count - 1u;
                    const T4 e = sh.near[wave][(q_out + k) & (kNearRing - 1)];
                    const int code = (int)e.w;
                    const int l = code & 63;
                    const T ox = __shfl(xi, l, 64), oy = __shfl(yi, l, 64), oz = __shfl(zi, l, 64);
                    const T nx = __shfl(txi, l, 64), ny = __shfl(tyi, l, 64), nz = __shfl(tzi, l, 64);
                    if ((uint32_t)lane < count) {
                        da_hist_add(sh, cd, inv_dr, l, 0, code >= 64, d2_exact(ox, oy, oz, e.x, e.y, e.z));
                        da_hist_add(sh, cd, inv_dr, l, 1, code >= 64, d2_exact(nx, ny, nz, e.x, e.y, e.z));
                    }
                    q_out += count;
                    wave_lds_sync();
                };
                // to the ring: the movers near_of[m] near partner st[m], every
                // lane one of its own partners a turn.  Partner by partner, a tile
                // with several near pairs, as in small systems, took up to 16
                // turns of a few lanes: ten sweeps of the 2:1 system at N = 8001
                // with a move log 3.58 ms, 2.7 so.  A turn of 40 lanes and more is
                // binned at once: of the same system with every partner in range
                // four sweeps take 4.85 ms instead of 6.0 (8001, log), at the
                // cost of 1 % where near pairs are few (ten of N = 32768 12.2 ms,
                // 12.1 without; lines at 32 to 48 within 1 %, 56 up to 2.5 % slower).
                auto note_near = [&](const T4* st, const uint64_t (&near_of)[DA ? P : 1], uint64_t near_any) {
                    if (near_any == 0ull) return;
                    uint32_t mine = 0;
#pragma unroll
                    for (int m = 0; m < (DA ? P : 1); ++m)
                        mine |= __builtin_amdgcn_inverse_ballot_w64(near_of[m]) ? 1u << m : 0u;
                    while (__ballot(mine != 0u) != 0ull) {
                        const T4 p = st[mine ? __builtin_ctz(mine) : 0];
                        const double qq = (double)p.w * (double)qi;
                        const bool put = mine != 0u && qq != 0.0;
                        mine &= mine - 1u;
                        const uint64_t who = __ballot(put);
                        if (__popcll(who) >= 40) {
                            if (put) {
                                da_hist_add(sh, cd, inv_dr, lane, 0, qq < 0.0, d2_exact(xi, yi, zi, p.x, p.y, p.z));
                                da_hist_add(sh, cd, inv_dr, lane, 1, qq < 0.0, d2_exact(txi, tyi, tzi, p.x, p.y, p.z));
                            }
                            continue;
                        }
                        if (put)
                            sh.near[wave][(q_in + __builtin_amdgcn_mbcnt_hi((uint32_t)(who >> 32),
                                                                            __builtin_amdgcn_mbcnt_lo((uint32_t)who, 0u))) &
                                          (kNearRing - 1)] = mk4<T>(p.x, p.y, p.z, (T)(lane + (qq < 0.0 ? 64 : 0)));
                        q_in += (uint32_t)__popcll(who);
                        if (q_in - q_out >= 64u) bin_near(64u);
                    }
                };
                // a working-precision squared distance below this bound may be
                // below rc^2 exactly (the bound is a relative 1e-5 above it)
                const T rc2_wide = (T)(cd.da_rc * cd.da_rc * (1.0 + 1e-5));
                // the terms of one staged slice of P partners of one diameter
                auto slice_sum = [&](const T4* st) {
                    T sf = 0;
                    uint64_t near_of[DA ? P : 1], near_any = 0;  // delayed acceptance: movers possibly within rc
#pragma unroll
                    for (int m = 0; m < P; ++m) {
                        const T4 p = st[m];
                        const T d2 = Prec<T>::norm2(p.x - xi, p.y - yi, p.z - zi);
                        const T d2t = Prec<T>::norm2(p.x - txi, p.y - tyi, p.z - tzi);
                        sf = Prec<T>::fma(p.w, Prec<T>::rinv(d2t) - Prec<T>::rinv(d2), sf);
                        d2t_min = Prec<T>::min(d2t, d2t_min);
                        near_of[m] = __ballot(Prec<T>::min(d2, d2t) < rc2_wide);
                        near_any |= near_of[m];
                    }
                    note_near(st, near_of, near_any);
                    S += (double)sf;
                };
                int64_t gp = g - nb + 1 + dphase;
                // Delayed acceptance, float, uniform diameters: while the
                // groups are well before the target, a wave takes its slices
                // of four of them at once, a record a lane (16 of 64 lanes
                // load for one slice), loaded four slices ahead.  The slices'
                // sums stay as they are.  Not for the last kQuadMargin groups,
                // which the chain is still deciding.  Bound: the pair terms;
                // one slice at a time, with one workgroup a CU, every slice
                // waited for its records (ten sweeps of N = 32768 14.6 ms,
                // 13.0 so, with near partners still taken one by one).  The
                // plain kernels have a second workgroup to fill that wait: no
                // gain at N = 32768, 3 % lost at 4001.
                if constexpr (DA && UNIFORM_SIGMA && SweepShared<T, M, DA>::SW == kGroup) {
                    const int64_t q_last = g_last - kQuadMargin;
                    const int sub = lane / P, jq = wave * P + lane % P;
                    typename IO::Rec rec{};
                    T qc = 0;
                    uint32_t slot = 0, ver = 0;
                    auto next = [&]() {
                        int bl = bp + sub;
                        ver = (uint32_t)sp;
                        if (bl >= nb) {
                            bl -= nb;
                            ++ver;
                        }
                        const int j = bl * kGroup + jq;
                        slot = (ver & 1u) * (uint32_t)npad + (uint32_t)j;
                        rec = IO::load(pos_r, slot);
                        qc = charge[j];
                    };
                    if (gp + 3 <= q_last) next();
                    for (; gp + 3 <= q_last; gp += 4) {
                        if (__ballot(rec.ver != ver) != 0ull) rec = IO::load_valid(pos_r, slot, ver, true, ctl, true);
                        sh.st[wave][lane] = mk4<T>(rec.x, rec.y, rec.z, qc);
                        wave_lds_sync();
                        bp += 4;
                        if (bp >= nb) {
                            bp -= nb;
                            ++sp;
                        }
                        if (gp + 7 <= q_last) next();
#pragma nounroll
                        for (int u = 0; u < 4; ++u) slice_sum(sh.st[wave] + u * P);
                        wave_lds_sync();
                    }
                }
                for (; gp <= g_last; gp += KD) {
                    const int j = bp * kGroup + jl;
                    typename IO::Rec cur;
                    if (have_next && __ballot(lane < PD && nxt.ver != (uint32_t)sp) == 0ull)
                        cur = nxt;
                    else
                        cur = IO::load_valid(pos_r, (uint32_t)((sp & 1) * npad + j), (uint32_t)sp, lane < PD, ctl,
                                             g - gp > kPatientDistance);
#ifdef MC_TIMELINE
                    if (!DA && gp + KD > g_last && lane == 0 && kTlSlots * (g + 1) <= cd.trace_cap)
                        ((uint64_t*)cd.trace_de)[kTlSlots * g + (wave == 0 ? 14 : 24 + wave)] = wall_clock64();
#endif
                    // per-ion diameters: a slice whose partners all have one
                    // diameter (every slice but those at a species boundary)
                    // takes the running-minimum contact test of the uniform case
                    T hj0 = (T)0;
                    bool slice_uniform = true;
                    if (lane < PD) {
                        const bool lo = PD == P || lane < P;
                        const int ls = lo ? lane : lane - P;
                        (lo ? sh.old_of(wave) : sh.st_old2[wave])[ls] = mk4<T>(cur.x, cur.y, cur.z, charge[j]);
                        if (!UNIFORM_SIGMA) {
                            hj0 = half[j];
                            (lo ? sh.st_half[wave] : sh.st_half2[wave])[ls] = hj0;
                        }
                    }
                    if constexpr (!UNIFORM_SIGMA && !DA) {
                        const T hjl = hj0;
                        hj0 = __shfl(hjl, 0, 64);
                        slice_uniform = __ballot(lane < PD && hjl != hj0) == 0ull;
                    }
                    wave_lds_sync();
                    // (KD steps of one, compared one by one, were about 1 % of a
                    // sweep of N = 131072: 7.95 ms, 7.86 so, of runs that differ by
                    // 0.3 %)
                    int bn = bp + KD;
                    int64_t sn = sp;
                    while (bn >= nb) {
                        bn -= nb;
                        ++sn;
                    }
                    have_next = false;
                    if constexpr (sizeof(T) == 4) {
                        if (gp + KD <= g_last) {
                            if (lane < PD) nxt = IO::load(pos_r, (uint32_t)((sn & 1) * npad + bn * kGroup + jl));
                            have_next = true;
                        }
                    }
                    T sf = 0;
                    uint64_t near_of[DA ? P : 1], near_any = 0;  // delayed acceptance: movers possibly within rc
                    if constexpr (UNIFORM_SIGMA || DA) {
                        // P partners at a time (a loop, not unrolled, so that a
                        // round needs the registers of one P-partner slice)
#pragma nounroll
                        for (int c = 0; c < KD; ++c)
#pragma unroll
                        for (int mm = 0; mm < P; ++mm) {
                            const int m = c * P + mm;
                            const T4 p = c == 0 ? sh.old_of(wave)[mm] : sh.st_old2[wave][(c - 1) * P + mm];
                            const T hj = UNIFORM_SIGMA ? hu
                                         : c == 0 ? sh.st_half[wave][mm] : sh.st_half2[wave][(c - 1) * P + mm];
                            const T s_ij = hi + hj;
                            const T d2 = Prec<T>::norm2(p.x - xi, p.y - yi, p.z - zi);
                            const T d2t = Prec<T>::norm2(p.x - txi, p.y - tyi, p.z - tzi);
                            sf = Prec<T>::fma(p.w, Prec<T>::rinv(d2t) - Prec<T>::rinv(d2), sf);
                            if (UNIFORM_SIGMA)
                                d2t_min = Prec<T>::min(d2t, d2t_min);
                            else
                                ov |= d2t < s_ij * s_ij;
                            if constexpr (DA) {
                                near_of[m] = __ballot(Prec<T>::min(d2, d2t) < rc2_wide);
                                near_any |= near_of[m];
                            }
                        }
                    } else {
                        // per-ion diameters: the contact test per pair, or as a
                        // running minimum of the trial distances for a slice
                        // with one diameter -- exact: min_j d2t_j < s^2 iff some
                        // d2t_j < s^2, with the one s = hi + hj the per-pair
                        // test forms for every partner of the slice
                        auto slice_terms = [&](auto per_pair_c) {
                            constexpr bool PER_PAIR = decltype(per_pair_c)::value;
                            T tmin = (T)3.0e38;
#pragma nounroll
                            for (int c = 0; c < KD; ++c) {
                            // (one base address a chunk: a choice per partner
                            // cost an address move each, 11 % of the loop)
                            const T4* st = c == 0 ? sh.old_of(wave) : sh.st_old2[wave] + (c - 1) * P;
                            const T* st_h = c == 0 ? sh.st_half[wave] : sh.st_half2[wave] + (c - 1) * P;
#pragma unroll
                            for (int mm = 0; mm < P; ++mm) {
                                const T4 p = st[mm];
                                const T d2 = Prec<T>::norm2(p.x - xi, p.y - yi, p.z - zi);
                                const T d2t = Prec<T>::norm2(p.x - txi, p.y - tyi, p.z - tzi);
                                sf = Prec<T>::fma(p.w, Prec<T>::rinv(d2t) - Prec<T>::rinv(d2), sf);
                                if constexpr (PER_PAIR) {
                                    const T s_ij = hi + st_h[mm];
                                    ov |= d2t < s_ij * s_ij;
                                } else {
                                    tmin = Prec<T>::min(d2t, tmin);
                                }
                            }
                            }
                            if constexpr (!PER_PAIR) {
                                const T s_ij = hi + hj0;
                                ov |= tmin < s_ij * s_ij;
                            }
                        };
                        if (slice_uniform)
                            slice_terms(std::false_type{});
                        else
                            slice_terms(std::true_type{});
                    }
                    if constexpr (DA) {
                        note_near(sh.old_of(wave), near_of, near_any);
                    }
                    S += (double)sf;
                    wave_lds_sync();
                    if constexpr (DA) {
                        // the ring is empty but for the last tile's when that comes
                        if (gp + 2 * KD > g_last && q_in != q_out) bin_near(q_in - q_out);
                    }
                    bp = bn;
                    sp = sn;
                }
                if (UNIFORM_SIGMA) ov |= d2t_min < (hu + hu) * (hu + hu);
            }
#ifdef MC_TIMELINE
            if (!DA && wave == 0 && lane == 0 && kTlSlots * (g + 1) <= cd.trace_cap)
                ((uint64_t*)cd.trace_de)[kTlSlots * g + 12] = wall_clock64();
#endif

            GroupRec rb[KB];
            auto load_band_recs = [&]() {  // all loads in flight at once
#pragma unroll
                for (int kb = LC; kb < KB; ++kb)
                    if (kb < band) rb[kb] = load_rec(rec_r, (uint32_t)((g - 1 - kb) & (kRing - 1)));
            };
            // ---- delayed acceptance: the features are complete after the
            // last partner tile, so the network runs here, while the older
            // band groups' accept masks are still on their way
            if constexpr (DA) {
                const uint64_t cb = __ballot(conf);
                if (lane == 0) sh.part_conf[wave] = cb;
                da_network<T, M>(sh, cd, wave, lane, da_on, s * (int64_t)cd.n + b * kGroup, cd.n - b * kGroup, g,
                                 load_band_recs);
            }

            if constexpr (!DA) load_band_recs();
            // ---- band groups older than the chain step's: their accept
            // masks are out by now (published about one group after the last
            // partner tile); this wave's slice of their candidates becomes final
#pragma unroll
            for (int kb = KB - 1; kb >= LC; --kb) {
                if (kb < band) {
                    const GroupRec r = rb[kb].tag == (uint32_t)(g - kb) ? rb[kb] : wait_rec(rec_r, g - 1 - kb, ctl);
                    const uint32_t a = (uint32_t)(r.acc >> (wave * P));
                    T sf = 0;
                    SB hit = 0;
#pragma unroll
                    for (int m = 0; m < P; ++m) {
                        const bool am = ((a >> m) & 1u) != 0;
                        sf += am ? c_band[kb][m] : (T)0;
                        hit |= am ? (ovt_band[kb] & (SB)(1u << m)) : (ovo_band[kb] & (SB)(1u << m));
                    }
                    S += (double)sf;
                    ov |= hit != 0;
                }
            }

#ifdef MC_TIMELINE
            if (!DA && lane == 0 && kTlSlots * (g + 1) <= cd.trace_cap)
                ((uint64_t*)cd.trace_de)[kTlSlots * g + (wave == 0 ? 13 : 20 + wave)] = wall_clock64();
#endif
            // ---- hand off the sums to the chain wave
            sh.part_s[wave][lane] = S;
            {
                const uint64_t ob = __ballot(ov);
                if (lane == 0) sh.part_ov[wave] = ob;
            }
            __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
            if (lane == 0)
                __hip_atomic_fetch_add(&sh.ready, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
#ifdef MC_TIMELINE
            if (!DA && lane == 0 && wave < 4 && kTlSlots * (g + 1) <= cd.trace_cap)
                ((uint64_t*)cd.trace_de)[kTlSlots * g + 16 + wave] = wall_clock64();
#endif

            // ---- wave 1 helps with the older chain band groups, wave 0
            // finishes the group: decisions and publication
            if constexpr (LC > 1) {
                if (wave == 1 && band >= 2) {
                    band_helper<T, M, DA>(sh, rec_r, g, t, band, ctl);
#ifdef MC_TIMELINE
                    if (lane == 0 && kTlSlots * (g + 1) <= cd.trace_cap)
                        ((uint64_t*)cd.trace_de)[kTlSlots * g + 28] = wall_clock64();
#endif
                }
            }
            if (wave == 0) {
                chain_step<T, M, DA>(sh, cd, pos_r, rec_r, g_begin, g, t, xi, yi, zi, txi, tyi, tzi, mi, da_on,
                                     ctl, ctr);
                if (g == g_end - 1 && lane == 0) cd.clk[1] = wall_clock64();
            }
        }
    }
    if (wave == 0 && lane == 0 && ctr.moves) {
        atomicAdd(&cd.stats[0], ctr.moves);
        atomicAdd(&cd.stats[1], ctr.acc);
        atomicAdd(&cd.stats[2], ctr.wall);
        atomicAdd(&cd.stats[3], ctr.ov);
        atomicAdd(&cd.stats[4], ctr.moves - ctr.acc - ctr.wall - ctr.ov);
        atomicAdd(&cd.stats[5], ctr.iters);
        atomicAdd(&cd.stats[6], ctr.early);
        if constexpr (DA) {
            atomicAdd(&cd.stats[7], ctr.da_moves);
            atomicAdd(&cd.stats[8], ctr.conflicts);
            atomicAdd(&cd.stats[9], ctr.s1_rej);
            atomicAdd(&cd.stats[10], ctr.s1_pass);
            atomicAdd(&cd.stats[11], ctr.s2_rej);
        }
    }
    __syncthreads();  // every wave is done with this chain's LDS state
}

// The sweep launch.  Workgroup w runs its items (chain, index of the
// workgroup among the chain's) one after another: a chain served by several
// workgroups is their only item; chains served by one workgroup alone may
// share it (a chain never waits on a workgroup busy with another chain).
template <typename T, int M, bool UNIFORM_SIGMA, bool DA = false>
__global__ void __launch_bounds__(64 * M)
__attribute__((amdgpu_waves_per_eu(kWavesPerEU<T, M, DA>)))
sweep_kernel(const ChainDesc* __restrict__ chains, const int2* __restrict__ wg_range,
             const int2* __restrict__ items, uint32_t s0, int32_t n_sweeps, Ctl ctl)
{
    __shared__ SweepShared<T, M, DA> sh;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int2 r = wg_range[blockIdx.x];
    for (int q = r.x; q < r.y; ++q) {
        const int2 it = items[q];
        sweep_chain<T, M, UNIFORM_SIGMA, DA>(sh, chains[it.x], it.y, s0, n_sweeps, ctl, wave, lane);
    }
}

// Running energy after each sweep of a launch, one block per chain:
// per-sweep totals of the group energy changes, one wave a sweep (lane l
// sums the groups l, l + 64, ...; then a butterfly: the order depends on the
// sweep alone, not on the launch it belongs to), then a serial prefix from
// the previous running energy.  Deterministic.  Latency bound; with one
// thread a sweep, summing its groups one after another, the scan of 100
// sweeps of 512 groups took 155 us.
__global__ void __launch_bounds__(1024)
energy_scan_kernel(const ChainDesc* __restrict__ chains, int32_t n_sweeps, int64_t s0)
{
    const ChainDesc& cd = chains[blockIdx.x];
    const int nb = cd.nb;
    const int lane = threadIdx.x & 63;
    for (int s = threadIdx.x >> 6; s < n_sweeps; s += blockDim.x >> 6) {
        double t = 0.0;
        for (int b = lane; b < nb; b += 64) t += cd.de_group[(int64_t)s * nb + b];
        t = wave_sum(t);
        if (lane == 0) cd.sweep_tot[s] = t;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        double e = *cd.e_state;
        for (int k = 0; k < n_sweeps; k += 8) {
            double v[8];  // loaded together: the prefix waits for memory once in eight sweeps
#pragma unroll
            for (int q = 0; q < 8; ++q) v[q] = k + q < n_sweeps ? cd.sweep_tot[k + q] : 0.0;
#pragma unroll
            for (int q = 0; q < 8; ++q) {
                if (k + q >= n_sweeps) break;
                e += v[q];
                if (s0 + k + q < cd.e_capacity) cd.e_series[s0 + k + q] = e;
            }
        }
        *cd.e_state = e;
        // delayed-acceptance drift monitor: at the end of each window, the
        // stage-2 rejection rate of stage-1 passes against its training-time
        // value; above ref_rate + delta the chain falls back to the plain
        // test for good (from the next launch, i.e. the next window)
        DAState* da = cd.da;
        const int64_t s_end = s0 + n_sweeps;
        if (da != nullptr && da->window > 0 && s_end % da->window == 0) {
            const unsigned long long pass = cd.stats[10], rej = cd.stats[11];
            const unsigned long long dp = pass - da->win_pass0, dr = rej - da->win_rej0;
            if (dp > 0) da->last_rate = (double)dr / (double)dp;
            if (da->active && da->ref_rate >= 0.0 && (int64_t)dp >= da->min_count &&
                da->last_rate > da->ref_rate + da->delta) {
                da->active = 0;
                da->fallback_sweep = s_end;
            }
            da->win_pass0 = pass;
            da->win_rej0 = rej;
        }
    }
}

}  // namespace mcdev
