// The simulation kernel template.  Resident form (RR = L): one workgroup
// advances one (protocol, replica) instance through all of its steps without
// leaving the compute unit.  Slab form (RR < L): one workgroup advances RR
// rows of a larger lattice by one step, from one state buffer in device memory
// to the other (see Geo).
//
// Layout.  Row pitch L = 64 * CPL; the lattice side LW <= L is a multiple of
// CPL.  Wave w owns rows [w*RPT, (w+1)*RPT) of the workgroup's RR rows; lane l
// owns columns [l*CPL, (l+1)*CPL).  The three float32 fields of a thread's
// RPT x CPL sites live in VGPRs for the whole run (resident) or step (slab);
// the uint16 cell words live in LDS.  One diffusion sub-step needs, per wave,
// only the row above and the row below its slab from the neighbouring waves (an
// LDS exchange of 2 rows), while left/right neighbours come from the adjacent lane through DPP lane
// shifts fused into the VALU adds.  A wave's 64 lanes span a whole lattice row,
// so the lane shifts' zero fill at lanes 0 and 63 is exactly the missing
// neighbour outside the lattice (the Dirichlet value is 0 in field units).
//
// Padding.  When LW < L the columns past the lattice hold padding sites:
// fields 0 with a diffusion number of 0 and no clamp, so they stay 0 and the
// last lattice column reads the boundary value from its right neighbour as
// lane 63 does; cell words EMPTY, never free and never irradiated.  Whole
// lanes are padding when LW is a multiple of CPL; otherwise one lane holds
// both kinds and keeps its diffusion numbers and clamps per column.  Philox
// counters and device-memory state use lattice coordinates (row pitch LW).
//
// Slabs.  A slab edge that is not a lattice edge is treated as if it were
// one; the error this makes reaches `substeps` rows into the slab through the
// diffusion and two rows further through the division proposals and their
// conflicts, so the rows within substeps + 2 of such an edge are a halo:
// computed, not stored, and owned by the neighbouring slab.  Every site's
// arithmetic is the resident form's, so both give identical results.
//
// Teams (TEAM): the slabs of one instance are a team of co-resident
// workgroups (a cooperative launch) that keep their rows on the CU for the
// whole horizon.  After each step a workgroup publishes the own rows its
// neighbours hold as halo (into one of two exchange buffers, by step parity)
// and a per-slab step count; before the next step it waits for both
// neighbours' counts, with a bounded spin, and reloads only its halo rows.
// A wait that runs out marks the instance's live count negative and the
// workgroup leaves the instance: every wait ends, so every workgroup exits.  It
// then publishes nothing any more in this launch: its counts would run on into
// its next instances, past neighbours that have yet to read the rows of the
// last one it finished.  Instances of a later turn that need an exchange it
// marks without computing them; those of fewer than two steps it computes.
//
// The method (Materials and Methods: nutrient and waste diffusion, cell
// cycle, quiescence and death driven by the local environment, irradiation
// damage; fitness from the final number of occupied sites, equation
// final_fit_fun) with the synthetic model's rules:
//   step n:  (1) fraction at n?  live cell of class c survives iff w1 < T_c
//            (2) activity a = act[state], frozen until the next fraction
//            (3) `substeps` FTCS sub-steps
//                c' = c + lam (N + S + E + W - 4c) - kappa a  (O, G; then max(., 0))
//                H' = H + lam (N + S + E + W - 4H) + kappa a
//                (protocols timed in half-hours, the paper's 30-minute slots:
//                a fraction at the half hour runs (1) and (2) again after
//                substeps / 2 of them)
//            (4) synchronous cell update from the snapshot (lysis, environment,
//                division proposals into free von Neumann neighbours, conflict
//                resolution by the smallest key)
//            (5) live count (PROLIF + QUIESC) by wave reduction.
#pragma once
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

#include "gga_device.h"
#include "gga_internal.h"

namespace gga {
namespace {

constexpr uint32_t NONE_KEY = 0xFFFFFFFFu;
constexpr uint32_t INIT_STEP = 0xFFFFFFFFu;
constexpr int EMPTY = 0, PROLIF = 1, QUIESC = 2, DEAD = 3;
constexpr uint32_t DOOM_BIT = 1u << 14;    // cell word: lethally hit, awaiting mitotic death
// The bits of a cell word that state buffers hold: state, age and mark.  The
// cell update uses the others within a step, so a caller's words are loaded
// without them.
constexpr uint32_t WORD_BITS = 0x3FFu | DOOM_BIT;

// The word of a seeded cell: age floor(w0 A0 / 2^32), saturating at 255 like
// every age (a larger one would run into the bits above it).
__device__ __forceinline__ uint16_t seed_word(uint32_t w0, int A0) {
    const uint32_t age = (uint32_t)(((uint64_t)w0 * (uint32_t)A0) >> 32);
    return (uint16_t)(PROLIF | (min(age, 255u) << 2));
}

// 32-bit linear-quadratic survival threshold, evaluated in float64 exactly as
// written: x = m d, y = m D, S = exp(-alpha x - beta x (x + 2 y)),
// T = min(floor(S 2^32), 2^32-1).  D is the unrepaired dose of earlier
// fractions (incomplete repair, see prior_damage); D = 0 is the plain law.
#pragma clang fp contract(off)
__device__ uint32_t lq_threshold(double d, double m, double alpha, double beta, double D) {
    const double x = m * d, y = m * D;
    const double e = -(alpha * x) - (beta * x) * (x + 2.0 * y);
    const double s = exp(e) * 4294967296.0;
    const double f = floor(s);
    return f >= 4294967295.0 ? 0xFFFFFFFFu : (uint32_t)f;
}

// Unrepaired dose before fraction j of protocol p: the sum over earlier
// fractions i of d_i 2^(-(t_j - t_i) / half_time), in index order (times in
// hours, or half-hours scaled by 0.5); 0 when half_time is 0.
__device__ double prior_damage(const float* dose, const int32_t* gap, int j, long long tj, double half_time,
                               double unit) {
    if (!(half_time > 0.0)) return 0.0;
    double acc = 0.0;
    long long ti = 0;
    for (int i = 0; i < j; ++i) {
        ti += gap[i];
        const float di = dose[i];
        if (di > 0.0f) acc += (double)di * exp2(-(((double)(tj - ti) * unit) / half_time));
    }
    return acc;
}

// Oxygen modification factor of oxygen bin b (the oxygen effect, oer_max > 1):
// (oer_max o + K) / (oer_max (o + K)) at the bin's midpoint
// o = (b + 1/2) ghost_O / GGA_OER_BINS.
__device__ double oxygen_modification(const gga_params& P, int b) {
    const double o = (((double)b + 0.5) * (double)P.ghost[0]) / GGA_OER_BINS;
    return (P.oer_max * o + P.oer_k) / (P.oer_max * (o + P.oer_k));
}

// Oxygen bin of a site from its O in field units (O = o^ + ghost_O, rho_O = 1):
// floor(GGA_OER_BINS O / ghost_O) clamped to 0 .. GGA_OER_BINS - 1, in float64.
__device__ __forceinline__ int oxygen_bin(float o_hat, const gga_params& P) {
    const double q = ((double)o_hat + (double)P.ghost[0]) / (double)P.ghost[0];
    const double b = floor(q * GGA_OER_BINS);
    return b < 0.0 ? 0 : (b > GGA_OER_BINS - 1 ? GGA_OER_BINS - 1 : (int)b);
}
#pragma clang fp contract(on)

// CPL consecutive uint16 cell words of one row, read or written with one
// LDS access (the address is 2*CPL-byte aligned: x0 = lane * CPL; three
// columns per lane take one access per word).
template <int CPL>
__device__ __forceinline__ void load_words(const uint16_t* p, uint32_t (&w)[CPL]) {
    if constexpr (CPL == 1) {
        w[0] = p[0];
    } else if constexpr (CPL == 2) {
        const uint32_t v = *reinterpret_cast<const uint32_t*>(p);
        w[0] = v & 0xFFFFu; w[1] = v >> 16;
    } else if constexpr (CPL == 3) {
        w[0] = p[0]; w[1] = p[1]; w[2] = p[2];
    } else {
        static_assert(CPL == 4, "CPL must be 1, 2, 3 or 4");
        const uint2 v = *reinterpret_cast<const uint2*>(p);
        w[0] = v.x & 0xFFFFu; w[1] = v.x >> 16; w[2] = v.y & 0xFFFFu; w[3] = v.y >> 16;
    }
}
template <int CPL>
__device__ __forceinline__ void store_words(uint16_t* p, const uint32_t (&w)[CPL]) {
    if constexpr (CPL == 1) {
        p[0] = (uint16_t)w[0];
    } else if constexpr (CPL == 2) {
        *reinterpret_cast<uint32_t*>(p) = w[0] | (w[1] << 16);
    } else if constexpr (CPL == 3) {
        p[0] = (uint16_t)w[0]; p[1] = (uint16_t)w[1]; p[2] = (uint16_t)w[2];
    } else {
        *reinterpret_cast<uint2*>(p) = make_uint2(w[0] | (w[1] << 16), w[2] | (w[3] << 16));
    }
}

// Fields are held in kernel units c^ = (c - g_f) / rho_f: shifted by the
// field's Dirichlet boundary value g_f and scaled by rho_f = kappa'_f / kappa'_O
// (kappa' the signed reaction rate: -uptake for O and G, +production for H).
// In these units the boundary is 0 and every field's reaction term is the
// oxygen one, kappa'_O a, so one per-site term serves all three fields.  The
// FTCS update keeps its form: c' = lam S + (1 - 4 lam) c + r carries over to
// c^' = lam S^ + (1 - 4 lam) c^ + r / rho_f, because the shift g_f cancels
// (4 lam + (1 - 4 lam) - 1 = 0) and a neighbour on the boundary is g_f, i.e. 0.
__host__ __device__ __forceinline__ double field_rho(const gga_params& P, int f) {
    const double k0 = -(double)P.kappa[0];
    const double kf = f < 2 ? -(double)P.kappa[f] : (double)P.kappa[f];
    return kf / k0;
}
__host__ __device__ __forceinline__ float to_field_units(const gga_params& P, int f, double c) {
    return (float)((c - (double)P.ghost[f]) / field_rho(P, f));
}

// Constants of the cell update.  They sit in LDS and are read at their point
// of use after a barrier, so they do not occupy scalar registers across the
// diffusion loop.
struct CellConst {
    float thOq, thGq, thOd, thGd, thHd;
    int T_min, T_lys, ca0, ca1;
    uint32_t T_div;
    float low[2];       // O and G above these at a step's start: its sub-steps need no clamp
};

// Register slot of row i after k forward rotating sub-steps (S = RPT + 1 slots).
template <int S>
constexpr int rot_slot(int i, int k) { return ((i - k) % S + S) % S; }

// L = 64 * CPL columns (LW of them the lattice's); NW waves of RPT rows hold
// RR = NW * RPT rows.  RR = LW: the whole lattice (resident).  RR < LW: a slab of
// a larger lattice advanced by one step per launch, or through all of them as
// part of a team (the rows within `substeps + 2` of a slab edge that is not a
// lattice edge are a halo, recomputed by the neighbouring slab).
template <int CPL, int RPT, int NW, int LW = 64 * CPL>
struct Geo {
    static constexpr int L = 64 * CPL;                // row pitch on the CU
    static constexpr int SIDE = LW;                   // lattice side
    static constexpr bool PAD = LW < L;               // columns past the lattice hold padding
    static constexpr bool PADC = PAD && LW % CPL != 0; // one lane holds lattice and padding columns
    static constexpr int NWAVE = NW;
    static constexpr int RR = NW * RPT;
    static constexpr bool SLAB = RR < LW;
    static constexpr int NT = 64 * NWAVE;
    // Halo area: [3 ghost rows][per wave: 3 top rows, 3 bottom rows], a row per
    // field, once per parity of the sub-step count, and 3 ghost rows at the end.
    // The ghost rows hold the boundary values, so the first and last wave read
    // their outer neighbour row like every other one.
    static constexpr int HALO = (6 * NW + 3) * L;
    static constexpr int AREA = 2 * HALO + 3 * L;
    static constexpr int POOL = (AREA > RR * L) ? AREA : RR * L;
    static_assert(RR <= LW && NWAVE <= 16, "workgroup above 1024 threads");
    static_assert(LW <= L && L % 32 == 0, "rows of whole claim words");
    static constexpr int SITES = RPT * CPL;           // sites per thread, bit i * CPL + c of the masks
    static_assert(SITES <= 64, "per-thread site masks are 64 bits wide at most");
    using Mask = std::conditional_t<(SITES > 32), uint64_t, uint32_t>;
    // Cell update: UR units of RPU rows per wave (two rows, a half-wave each,
    // on 64 columns; else one), every NW-th of the workgroup's, UC columns per
    // lane in NP pairs (as many lanes as a row needs), the units in NB blocks
    // of UB; bit j * UC + c of a block's masks: column c of its j-th unit.
    static constexpr int UC = L <= 128 ? 2 : 4, NP = UC / 2, RPU = L == 64 ? 2 : 1, UR = RR / RPU / NW;
    static constexpr int NB = (UR * UC + 63) / 64, UB = UR / NB;
    using UMask = std::conditional_t<(UB * UC > 32), uint64_t, uint32_t>;
    static_assert(L <= 256 && L % UC == 0 && UR % NB == 0 && UR <= 32 && RR % (RPU * NW) == 0, "rows of the cell update");
};

// Lowest set bit of a site mask.
__device__ __forceinline__ int first_bit(uint32_t m) { return __builtin_ctz(m); }
__device__ __forceinline__ int first_bit(uint64_t m) { return __builtin_ctzll(m); }

// Two 16-bit lanes in a register (two cell words): subtraction, addition and
// minimum per half, and each half's sign spread over it.
typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
typedef int16_t i16x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk_sub(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, a) - __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pk_add(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, (u16x2)(__builtin_bit_cast(u16x2, a) + __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pk_min(uint32_t a, uint32_t b) {
    return __builtin_bit_cast(uint32_t, __builtin_elementwise_min(__builtin_bit_cast(u16x2, a), __builtin_bit_cast(u16x2, b)));
}
__device__ __forceinline__ uint32_t pk_sign(uint32_t a) {
    return __builtin_bit_cast(uint32_t, (i16x2)(__builtin_bit_cast(i16x2, a) >> 15));
}
// a where the mask is set, b elsewhere
__device__ __forceinline__ uint32_t bit_select(uint32_t mask, uint32_t a, uint32_t b) { return (a & mask) | (b & ~mask); }

// EXT: the extended radiobiology (the oxygen effect on radiosensitivity,
// gga_params.oer_max > 1, and mitotic death, gga_params.mitotic_death), a
// separate instantiation so that runs without them keep their register budget.
template <int CPL, int RPT, int NW, int LW, bool EXT, bool TEAM = false>
__global__ __launch_bounds__(64 * NW) void sim_kernel(SimArgs arg) {
    using G = Geo<CPL, RPT, NW, LW>;
    constexpr int L = G::L;
    constexpr bool PAD = G::PAD, PADC = G::PADC;
    static_assert(!TEAM || G::SLAB, "teams are made of slabs");
    constexpr int RR = G::RR;
    constexpr int NWAVE = G::NWAVE;
    constexpr bool SLAB = G::SLAB;
    // cells may be marked for mitotic death (teams load no state: without the
    // option they never hold a mark)
    constexpr bool MARKS = EXT || !TEAM;
    using Mask = typename G::Mask;
    using UMask = typename G::UMask;

    __shared__ __attribute__((aligned(16))) uint16_t s_cell[RR * L];
    __shared__ __attribute__((aligned(16))) uint32_t s_pool[G::POOL];   // halo buffer(s), then claim slots
    // one "has a daughter" bit per site (and a word that nothing reads: with it the
    // arrays behind lie so that the teams' kernels spill 3 to 4 registers less)
    __shared__ uint32_t s_claim[RR * L / 32 + 1];
    __shared__ uint32_t s_ev_step[GGA_KMAX];   // half-hours since step n0 (2 (n - n0), + 1 at the half hour)
    __shared__ float s_ev_dose[GGA_KMAX];
    __shared__ double s_ev_prior[GGA_KMAX];    // unrepaired dose of the earlier fractions (incomplete repair)
    __shared__ uint32_t s_ev_thr[GGA_KMAX][4];
    // the current fraction's thresholds per class and oxygen bin (oxygen effect only)
    __shared__ uint32_t s_oer_thr[EXT ? 4 : 1][EXT ? GGA_OER_BINS : 1];
    __shared__ int s_nev, s_valid, s_evj[2];
    __shared__ int s_count[2];
    __shared__ int s_team_ok;
    __shared__ uint32_t s_rows[NWAVE];         // per wave: which of its rows of the cell update hold a cell
    __shared__ int s_low[2], s_dirty;          // the sub-steps of step n may reach the clamp (by parity of n); see `low`
    __shared__ float s_react[4];               // reaction term per cell state
    __shared__ float2 s_react2[16];            // and of two cells, by their states (the first in the low bits)
    __shared__ CellConst s_k;                  // cell-update constants, read where used

    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    // instance (and slab) of this workgroup
    int inst = 0, slab = 0, slab_row = 0;
    if constexpr (SLAB) {
        // Workgroups are dealt to the 8 XCDs in turn (block b to XCD b mod 8), so
        // all slabs of list position k go to XCD k mod 8: slab rows shared by
        // neighbouring slabs come from that XCD's L2.  b = (y * 8 + x) with
        // x = k mod 8 and y = (k / 8) * n_slabs + slab; positions past the list
        // are idle workgroups.
        const int x = (int)(blockIdx.x & 7u), y = (int)(blockIdx.x >> 3);
        const int kq = y / arg.n_slabs;
        slab = y - kq * arg.n_slabs;
        slab_row = kq * 8 + x;
        if (slab_row >= arg.n_active) return;              // uniform across the workgroup
        inst = arg.inst_list && !TEAM ? arg.inst_list[slab_row] : slab_row;
    } else {
        inst = arg.inst_list ? arg.inst_list[blockIdx.x] : (int)blockIdx.x;
    }
    // A team takes list positions in turns of n_active, every other turn
    // backwards: lists come with the longest horizons first, so the teams' sums
    // stay even, and no team waits for the others between its instances (the
    // uneven batch of 256 protocols x 4 in launches of one instance per team
    // took 316 ms, now 252).  The step counts run on from instance to instance.
    int flag_base = 0;
    if (TEAM && tid == 0) s_team_ok = 1;             // until a wait runs out
    for (int turn = 0; turn < (TEAM ? arg.turns : 1); ++turn) {
    // a team's arguments are read from the kernel argument segment by a pointer
    // that is opaque in each turn, so that nothing derived from them is held
    // in registers from one instance to the next
    const SimArgs* args = &arg;
    if constexpr (TEAM) {
        auto* segment = __builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(segment));
        args = (const SimArgs*)segment;
    }
    const SimArgs& a = *args;
    if constexpr (TEAM) {
        const int pos = turn * a.n_active + ((turn & 1) ? a.n_active - 1 - slab_row : slab_row);
        if (pos >= a.n_list) continue;
        inst = a.inst_list[pos];
        if (turn) __syncthreads();                       // the last instance's LDS words are read
    }
    inst = __builtin_amdgcn_readfirstlane(inst);     // uniform, as all that follows from it
    const int p = inst / a.R;
    const int r = inst - p * a.R;
    // state buffer row: the slab's list position; a library tumour (replica r
    // starts from library state r mod lib_n); or the instance
    const int slot = SLAB ? slab_row : (a.lib_n ? r % a.lib_n : inst);
    // the slab's first lattice row, and its own (non-halo) rows [iy0, iy1) of the slab
    const int ys = SLAB ? a.slab_ys[slab] : 0;
    int iy0 = SLAB ? a.slab_i0[slab] : 0, iy1 = SLAB ? a.slab_i1[slab] : RR;
    const int lat0 = ys * LW;                        // lattice index of the slab's first site
    const int nsteps = __builtin_amdgcn_readfirstlane(((!SLAB || TEAM) && a.horizon) ? a.horizon[p] : a.nsteps);
    const int y0 = wave * RPT;
    const int x0 = lane * CPL;
    // columns past the lattice hold padding: column x0 + c is the lattice's
    // when realc(c); real: the lane holds at least one lattice column
    auto realc = [&](int c) { return !PAD || x0 + c < LW; };
    const bool real = realc(0);
    // lattice index (the Philox site counter) of slab site index `site` (pitch L)
    auto lat_id = [&](int site) { return PAD ? (site / L) * LW + site % L + lat0 : site + lat0; };
    const gga_params& P = a.prm;
    // Philox key; `a` itself stays unmodified (a written kernel argument would
    // be copied to scratch memory)
    uint32_t seed_lo = a.seed_lo, seed_hi = a.seed_hi;
    if (a.generation) {             // per-generation key of a replayed GA generation
        const uint64_t key = a.seed + (uint64_t)(uint32_t)*a.generation * 0x9E3779B97F4A7C15ull;
        seed_lo = (uint32_t)key;
        seed_hi = (uint32_t)(key >> 32);
    }

    // ---- protocol: validity and irradiation events ----
    if constexpr (SLAB && !TEAM) {
        // event table (times in half-hours; at most one fraction at the start of
        // step n0 and one at its middle): lane j of wave 0 checks fraction j
        if (wave == 0) {
            const int k = a.ev_count[p];
            int j0 = -1, j1 = -1;
            for (int j = lane; j < k; j += 64) {
                const int tau = a.ev_step[(size_t)p * a.K + j];
                if (tau == 2 * a.n0) j0 = j;
                if (tau == 2 * a.n0 + 1) j1 = j;
            }
            const uint64_t m0 = __builtin_amdgcn_ballot_w64(j0 >= 0), m1 = __builtin_amdgcn_ballot_w64(j1 >= 0);
            const int J0 = m0 ? __shfl(j0, __builtin_ctzll(m0)) : -1;
            const int J1 = m1 ? __shfl(j1, __builtin_ctzll(m1)) : -1;
            if (lane == 0) {
                s_valid = a.ev_valid[p];
                int e = 0;
                if (J0 >= 0) { s_ev_step[e] = 0u; s_evj[e] = J0; ++e; }
                if (J1 >= 0) { s_ev_step[e] = 1u; s_evj[e] = J1; ++e; }
                s_nev = e;
            }
        }
    }
    if (tid == 0) {
        const int k = a.nfrac ? a.nfrac[p] : 0;
        int valid = (k >= 0 && k <= a.K);
        int nev = 0;
        double total = 0.0;
        long long t = 0;
        for (int j = 0; (!SLAB || TEAM) && valid && j < k; ++j) {
            const float d = a.dose[(size_t)p * a.K + j];
            const int g = a.gap[(size_t)p * a.K + j];
            if (!(d >= 0.0f) || !isfinite(d)) { valid = 0; break; }
            if (g < (j == 0 ? 0 : 1)) { valid = 0; break; }
            total += (double)d;
            t += g;
            // event time in half-hours (delays count half-hours with a.half)
            const long long tau = a.half ? t : 2 * t;
            if (d > 0.0f && tau >= 2LL * a.n0 && tau < 2LL * ((long long)a.n0 + nsteps)) {
                s_ev_step[nev] = (uint32_t)(tau - 2LL * a.n0);
                s_ev_dose[nev] = d;
                s_ev_prior[nev] = prior_damage(a.dose + (size_t)p * a.K, a.gap + (size_t)p * a.K, j, t,
                                               a.prm.repair_half_time, a.half ? 0.5 : 1.0);
                ++nev;
            }
        }
        if (valid && total > a.dose_cap + 1e-6) valid = 0;
        if (TEAM && valid && nsteps > 1 && !s_team_ok) {   // a wait has run out: no exchange any more
            if (a.live) atomicExch(&a.live[inst], (int)0x80000000);
            valid = 0;
        }
        if (!SLAB || TEAM) {
            s_valid = valid;
            s_nev = nev;
        }
        const gga_params& Q = a.prm;
        // thresholds in field units (rho_O = 1, rho_G > 0, rho_H < 0: the host
        // requires positive rates, so "H above its threshold" reads H^ < th^)
        s_k.thOq = to_field_units(Q, 0, Q.theta_O_quiesce); s_k.thGq = to_field_units(Q, 1, Q.theta_G_quiesce);
        s_k.thOd = to_field_units(Q, 0, Q.theta_O_death); s_k.thGd = to_field_units(Q, 1, Q.theta_G_death);
        s_k.thHd = to_field_units(Q, 2, Q.theta_H_death);
        s_k.T_min = Q.T_min; s_k.T_lys = Q.T_lys;
        s_k.ca0 = Q.class_age[0]; s_k.ca1 = Q.class_age[1];
        s_k.T_div = (Q.P_div >= 1.0) ? 0xFFFFFFFFu : (uint32_t)floor(Q.P_div * 4294967296.0);
        s_count[0] = 0;
        s_count[1] = 0;
        s_low[0] = 0;
        s_low[1] = 0;
        s_dirty = 0;
    }
    __syncthreads();
    if (!__builtin_amdgcn_readfirstlane(s_valid)) {
        if (!SLAB && tid == 0 && a.live) a.live[inst] = -1;   // slabs: set before the first step
        continue;                                 // uniform across the workgroup
    }
    const int nev = __builtin_amdgcn_readfirstlane(s_nev);
    if constexpr (SLAB && !TEAM) {
        if (tid < nev) {
            const EventFraction ef = a.ev_frac[(size_t)p * a.K + s_evj[tid]];
            s_ev_dose[tid] = ef.dose;
            s_ev_prior[tid] = ef.prior;
        }
        __syncthreads();
    }
    for (int e = tid; e < 4 * nev; e += G::NT)
        s_ev_thr[e >> 2][e & 3] = lq_threshold((double)s_ev_dose[e >> 2], P.m[e & 3], P.alpha, P.beta,
                                               s_ev_prior[e >> 2]);

    // ---- state: fields in registers, cells in LDS ----
    float F[3][RPT + 1][CPL];                  // slot RPT: spare row for the rotating sub-steps
    const size_t plane = (size_t)LW * LW;      // device-memory state: [3][LW][LW] fields, [LW][LW] cells
    if ((SLAB && !TEAM) || (!TEAM && (a.mode & MODE_LOAD))) {      // teams start from the initial state
        const float* src = a.fields + (size_t)slot * 3 * plane + lat0;
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
            for (int i = 0; i < RPT; ++i)
#pragma unroll
                for (int c = 0; c < CPL; ++c)
                    F[f][i][c] = realc(c) ? src[f * plane + (size_t)(y0 + i) * LW + x0 + c] : 0.0f;
        const uint16_t* cs = a.cells + (size_t)slot * plane + lat0;
#pragma unroll
        for (int i = 0; i < RPT; ++i)
#pragma unroll
            for (int c = 0; c < CPL; ++c)
                s_cell[(y0 + i) * L + x0 + c] = realc(c) ? (uint16_t)(cs[(size_t)(y0 + i) * LW + x0 + c] & WORD_BITS) : (uint16_t)0;
    } else {
        const int ctr = LW / 2;
        const int rad2 = P.seed_radius * P.seed_radius;
        float f0[3];
#pragma unroll
        for (int f = 0; f < 3; ++f) f0[f] = to_field_units(P, f, P.init[f]);
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
            for (int i = 0; i < RPT; ++i)
#pragma unroll
                for (int c = 0; c < CPL; ++c) F[f][i][c] = realc(c) ? f0[f] : 0.0f;
#pragma nounroll
        for (int i = 0; i < RPT; ++i)
#pragma nounroll
            for (int c = 0; c < CPL; ++c) {
                const int y = ys + y0 + i, x = x0 + c;       // lattice row and column
                uint16_t w = 0;
                if (realc(c) && (x - ctr) * (x - ctr) + (y - ctr) * (y - ctr) <= rad2) {
                    const Block4 b = philox10(y * LW + x, INIT_STEP, r, p, seed_lo, seed_hi);
                    w = seed_word(b.w0, P.A0);
                }
                s_cell[(y0 + i) * L + x] = w;
            }
    }

    // Per-field constants (field units, see to_field_units): the update and the
    // lower clamp of O and G (c >= 0 reads c^ >= -g / rho, rho_O = 1 and
    // rho_G > 0); the one reaction rate kappa'_O enters through s_react.
    // Padding columns take lam = 0 and no clamp, so their fields stay 0 (per
    // column when a lane holds both kinds, else per lane).
    constexpr int NC = PADC ? CPL : 1;
    float lam[3][NC], cen[3], lo[2][NC];
#pragma unroll
    for (int f = 0; f < 3; ++f) {
#pragma unroll
        for (int c = 0; c < NC; ++c) lam[f][c] = realc(c) ? P.lambda[f] : 0.0f;
        cen[f] = 1.0f - 4.0f * P.lambda[f];
    }
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
        for (int c = 0; c < NC; ++c) lo[f][c] = realc(c) ? to_field_units(P, f, 0.0) : -INFINITY;
    // reaction term per cell state, -kappa'_O a[state], looked up in LDS by
    // each site's state (one LDS read instead of a chain of selects)
    if (tid < 4) s_react[tid] = -P.kappa[0] * P.activity[tid];
    if (tid < 16) s_react2[tid] = make_float2(-P.kappa[0] * P.activity[tid & 3], -P.kappa[0] * P.activity[tid >> 2]);

    // Sub-steps without the clamp.  Every field's update rises with each of its
    // inputs (lambda in [0, 1/4]) and so does its rounded value, so with O and G
    // at least m <= 0 everywhere (0 is the boundary) the next values are at
    // least m - r up to three roundings of that size, r the largest reaction
    // rate: when low[f] < m for the step's first fields, with
    // low[f] = lo[f] / (1 + 2^-14) + substeps r (64 sub-steps round by less than
    // 2^-16 relatively), no site can reach its clamp within the step and the
    // maximum leaves every value as it is.  Fields that are not finite or
    // beyond 1e20 (a caller's state; O and G never grow) keep the clamp always.
    // Saves 2 of 17 instructions per site and sub-step.
    if (tid == 0) {
        float act = P.activity[0];
        for (int k = 1; k < 4; ++k) act = fmaxf(act, P.activity[k]);
        const double r = (double)a.substeps * ((double)P.kappa[0] * (double)act);
        for (int f = 0; f < 2; ++f) s_k.low[f] = (float)((double)to_field_units(P, f, 0.0) / (1.0 + 1.0 / 16384.0) + r);
    }
    __syncthreads();
    // smallest value of field f over the thread's sites
    auto least = [&](int f) {
        float m = F[f][0][0];
#pragma unroll
        for (int k = 1; k + 1 < RPT * CPL; k += 2)
            asm("v_min3_f32 %0, %0, %1, %2" : "+v"(m) : "v"(F[f][k / CPL][k % CPL]), "v"(F[f][(k + 1) / CPL][(k + 1) % CPL]));
        if constexpr (RPT * CPL % 2 == 0) asm("v_min_f32 %0, %0, %1" : "+v"(m) : "v"(F[f][RPT - 1][CPL - 1]));
        return m;
    };
    // marks step m's clamp when one of this wave's sites needs it
    auto mark_low = [&](float least_O, float least_G, int m) {
        const float low_O = s_k.low[0], low_G = s_k.low[1];
        if (__builtin_amdgcn_ballot_w64(!(least_O > low_O && least_G > low_G && 0.0f > low_O && 0.0f > low_G)) != 0 && lane == 0)
            s_low[m & 1] = 1;
    };
    {
        uint32_t most = 0;                               // magnitudes as integers: NaN above infinity above 1e20
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
            for (int i = 0; i < RPT; ++i)
#pragma unroll
                for (int c = 0; c < CPL; ++c) most = max(most, __float_as_uint(F[f][i][c]) & 0x7FFFFFFFu);
        if (__builtin_amdgcn_ballot_w64(most >= __float_as_uint(1e20f)) != 0 && lane == 0) s_dirty = 1;
        mark_low(least(0), least(1), a.n0);
    }

    // Rows of the cell update (see there): packed words of row y's pairs, EMPTY
    // for lanes past the row; which of the wave's rows hold a cell, for s_rows.
    constexpr int UC = G::UC, NP = G::NP, RPU = G::RPU, UR = G::UR, NB = G::NB, UB = G::UB;
    auto load_pairs = [&](int y, int ux, uint32_t (&w)[NP]) {
#pragma unroll
        for (int q = 0; q < NP; ++q) w[q] = 0;
        if (L == 64 * UC || ux < L) {
            if constexpr (NP == 1) {
                w[0] = *reinterpret_cast<const uint32_t*>(s_cell + y * L + ux);
            } else {
                const uint2 v = *reinterpret_cast<const uint2*>(s_cell + y * L + ux);
                w[0] = v.x;
                w[NP - 1] = v.y;
            }
        }
    };
    auto store_pairs = [&](int y, int ux, const uint32_t (&w)[NP]) {
        if (L == 64 * UC || ux < L) {
            if constexpr (NP == 1) *reinterpret_cast<uint32_t*>(s_cell + y * L + ux) = w[0];
            else *reinterpret_cast<uint2*>(s_cell + y * L + ux) = make_uint2(w[0], w[NP - 1]);
        }
    };
    auto scan_rows = [&] {
        uint32_t rows = 0;
        int at = lane % (64 / RPU) * UC, sub = RPU > 1 ? lane / 32 : 0;
        asm volatile("" : "+v"(at), "+v"(sub));
        uint32_t any[UR];
#pragma unroll
        for (int k = 0; k < UR; ++k) {
            uint32_t w[NP];
            load_pairs((wave + NWAVE * k) * RPU + (RPU > 1 ? sub : 0), at, w);
            any[k] = w[0] | w[NP - 1];
        }
#pragma unroll
        for (int k = 0; k < UR; ++k) rows |= (uint32_t)(__builtin_amdgcn_ballot_w64(any[k] != 0u) != 0) << k;
        if (lane == 0) s_rows[wave] = rows;
    };

    int ev = 0;
    int count = 0;
    __syncthreads();
    scan_rows();
    const bool dirty = __builtin_amdgcn_readfirstlane(s_dirty) != 0;

    // Teams: a step count is published with its publisher's XCD in its low bits
    // (while the count leaves room for them).  A workgroup whose neighbours run
    // on its own XCD, as the block numbering arranges, shares their L2: its
    // stores have reached it when they are acknowledged and device-scope loads
    // (SC1) read it past the compute unit's cache, so neither side needs the
    // fences that write the L2 back and invalidate it for the other XCDs.
    // Otherwise, and for the first count, both do.
    constexpr int SC1 = 16;
    const int xcc_bits = TEAM ? a.flag_bits : 0;
    const int xcc = TEAM && xcc_bits ? (int)(__builtin_amdgcn_s_getreg(20 | (3 << 11)) & 15u) : 0;   // HW_REG_XCC_ID
    bool same_xcd = false, team_ok = true;
    for (int n = a.n0; n < a.n0 + nsteps; ++n) {
        // Every LDS access below addresses a row as base + constant offset.  The
        // base is opaque to the compiler at the top of each step, so per-row
        // addresses are not hoisted out of the loop into registers.
        int own = y0 * L + x0;
        asm volatile("" : "+v"(own));
        // nor are the per-row comparisons with the slab's own rows, into scalar ones
        if constexpr (SLAB) asm volatile("" : "+s"(iy0), "+s"(iy1));
        asm volatile("" : "+s"(seed_lo), "+s"(seed_hi));   // nor is Philox's key schedule
        uint16_t* const cellp = s_cell + own;            // row i: cellp + i * L
        float Ro[RPT][CPL];                              // reaction term, set below
        bool occupied = false;                           // one of the wave's sites holds a cell
        const bool clamp = dirty || __builtin_amdgcn_readfirstlane(s_low[n & 1]) != 0;
        // (3) diffusion sub-steps, in pairs over the RPT + 1 register slots with
        // no row copied: a forward sub-step (rows top to bottom) writes new row
        // i over old row i - 1, which row i was the last to read, moving every
        // row one slot down; the reverse sub-step that follows (rows bottom to
        // top) writes new row i over old row i + 1 and moves them back, so after
        // each pair every row is in its own slot again.
        // Exchange.  The order gives every exchanged row half a sub-step or more
        // between its publication and its use, so one barrier in the middle of
        // each sub-step is all they need and no wave waits at its end: a forward
        // sub-step publishes its new top row first and its new bottom row last.
        // The neighbour above needs the old top row (published last by the
        // reverse sub-step before) for its own bottom row, computed last, and the
        // new top row for the start of the reverse sub-step that follows: it
        // reads both after the barrier.  Mirrored for the reverse sub-step.  Rows
        // are buffered by state parity: a buffer is rewritten two sub-steps
        // later, behind the barrier that its readers passed after using it.
        // (The form before, publish, barrier, read, compute, left every wave
        // waiting on the LDS reads at once: 1.95 against 1.77 us per sub-step of
        // 256 instances on 128 x 128, of which issuing its 15 instructions a
        // site takes 1.67.)
        float* const hw = reinterpret_cast<float*>(s_pool) + (3 + 6 * wave) * L + x0;
        constexpr int TOP = 0, BOT = 3 * L, UP = -3 * L, DN = 6 * L, ODD = G::HALO;
        auto put = [&](int at, int slot) {
#pragma unroll
            for (int f = 0; f < 3; ++f)
#pragma unroll
                for (int c = 0; c < CPL; ++c) hw[at + f * L + c] = F[f][slot][c];
        };
        auto get = [&](int at, float (&h)[3][CPL]) {
#pragma unroll
            for (int f = 0; f < 3; ++f)
#pragma unroll
                for (int c = 0; c < CPL; ++c) h[f][c] = hw[at + f * L + c];
        };
        // new row i, rows in the slots of map k, into slot `to`; `edge`: the
        // neighbouring wave's row above row 0 or below the last row.  Per field
        // and column c' = lam (up + below + west + east) + (c cen + r).
        auto row = [&](int k, int i, int to, const float (&edge)[3][CPL]) {
            const int si = rot_slot<RPT + 1>(i, k);
#pragma unroll
            for (int f = 0; f < 3; ++f)
#pragma unroll
                for (int c = 0; c < CPL; ++c) {
                    const float above = (i == 0) ? edge[f][c] : F[f][rot_slot<RPT + 1>(i - 1, k)][c];
                    const float below = (i < RPT - 1) ? F[f][rot_slot<RPT + 1>(i + 1, k)][c] : edge[f][c];
                    const float west = (c > 0) ? F[f][si][c - 1] : lane_from_left(F[f][si][CPL - 1]);
                    const float east = (c < CPL - 1) ? F[f][si][c + 1] : lane_from_right(F[f][si][0]);
                    const float sum = (above + below) + (west + east);
                    F[f][to][c] = fmaf(lam[f][PADC ? c : 0], sum, fmaf(F[f][si][c], cen[f], Ro[i][c]));
                }
        };
        // the clamp of O and G on slots first .. last, in steps that may need it
        // (the pin keeps H's rows from being computed behind the branch, where
        // the lane shifts would no longer fold into the adds)
        auto clamp_slots = [&](int first, int last) {
#pragma unroll
            for (int f = 0; f < 3; ++f)
#pragma unroll
                for (int j = first; j <= last; ++j)
#pragma unroll
                    for (int c = 0; c < CPL; ++c) asm volatile("" : "+v"(F[f][j][c]));
            if (clamp) {
#pragma unroll
                for (int f = 0; f < 2; ++f)
#pragma unroll
                    for (int j = first; j <= last; ++j)
#pragma unroll
                        for (int c = 0; c < CPL; ++c) asm("v_max_f32 %0, %0, %1" : "+v"(F[f][j][c]) : "v"(lo[f][PADC ? c : 0]));
            }
        };
        // sub-steps stay in order: no work moves across this point, and nothing
        // derived from Ro is held in registers across it
        auto pin = [&] {
#pragma unroll
            for (int f = 0; f < 3; ++f)
#pragma unroll
                for (int j = 0; j <= RPT; ++j)
#pragma unroll
                    for (int c = 0; c < CPL; ++c) asm volatile("" : "+v"(F[f][j][c]));
#pragma unroll
            for (int i = 0; i < RPT; ++i)
#pragma unroll
                for (int c = 0; c < CPL; ++c) asm volatile("" : "+v"(Ro[i][c]));
        };
        constexpr int MID = RPT / 2;
        static_assert(RPT >= 2, "the first and last row of a thread differ");
        float hn[3][CPL], hd[3][CPL];                    // halo rows: for the next sub-step's first row, for the last row
        // even sub-step: state in buffer 0, new state into buffer 1
        auto forward = [&] {
            pin();
            row(0, 0, RPT, hn);
            clamp_slots(RPT, RPT);
            put(TOP + ODD, RPT);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 1; i < MID; ++i) row(0, i, i - 1, hn);
            __syncthreads();
            get(DN, hd);
            get(DN + ODD, hn);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = MID; i < RPT; ++i) row(0, i, i - 1, hd);
            clamp_slots(0, RPT - 2);
            put(BOT + ODD, RPT - 2);
        };
        // odd sub-step: state in buffer 1, new state into buffer 0
        auto reverse = [&] {
            pin();
            row(1, RPT - 1, RPT - 1, hn);
            clamp_slots(RPT - 1, RPT - 1);
            put(BOT, RPT - 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = RPT - 2; i >= RPT - MID; --i) row(1, i, i, hn);
            __syncthreads();
            get(UP + ODD, hd);
            get(UP, hn);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = RPT - MID - 1; i >= 0; --i) row(1, i, i, hd);
            clamp_slots(0, RPT - 2);
            put(TOP, 0);
        };
        // ghost rows (the cell update's claim slots share this memory); the
        // first barrier of the sub-steps orders these writes before any read
        for (int k = tid; k < 3 * 3 * L; k += G::NT) {
            const int blk = k / (3 * L);
            reinterpret_cast<float*>(s_pool)[blk * (G::HALO - 3 * L) + k] = 0.0f;
        }
        const uint32_t rel = 2u * (uint32_t)(n - a.n0);  // the hour's start, in half-hours since step n0
#pragma nounroll
        for (uint32_t half = 0;; half = 1) {
            // this segment's first halo rows (after the reads of the half hour's first segment)
            if (half) __syncthreads();
            put(TOP, 0);
            put(BOT, RPT - 1);
            // (1) irradiation: every live cell draws w1 against its class
            // threshold, at the start of the hour or, for a fraction timed at
            // the half hour, after half of the hour's sub-steps (its words from
            // the block of step word n | 2^31)
            if (ev < nev && s_ev_step[ev] == rel + half) {
                // with the oxygen effect: this fraction's thresholds per class
                // and oxygen bin, and each site's bin from its current O
                const bool oer = EXT && P.oer_max > 1.0, mitotic = EXT && P.mitotic_death != 0;
                if (oer) {
                    __syncthreads();                      // the previous fraction's table is read
                    if (tid < 4 * GGA_OER_BINS) {
                        const double f = oxygen_modification(P, tid % GGA_OER_BINS);
                        s_oer_thr[tid / GGA_OER_BINS][tid % GGA_OER_BINS] =
                            lq_threshold(f * (double)s_ev_dose[ev], P.m[tid / GGA_OER_BINS], P.alpha, P.beta,
                                         f * s_ev_prior[ev]);
                    }
                    __syncthreads();
                }
                const uint32_t t0 = s_ev_thr[ev][0], t1 = s_ev_thr[ev][1];
                const uint32_t t2 = s_ev_thr[ev][2], t3 = s_ev_thr[ev][3];
                const int ca0 = s_k.ca0, ca1 = s_k.ca1;
                Mask live_mask = 0;
#pragma unroll
                for (int i = 0; i < RPT; ++i)
#pragma unroll
                    for (int c = 0; c < CPL; ++c) {
                        const uint32_t w = cellp[i * L + c];
                        const int st = w & 3;
                        if (st == PROLIF || st == QUIESC) {
                            live_mask |= (Mask)1 << (i * CPL + c);
                            // the site's oxygen bin rides in the word's free bits 10-13
                            // until this fraction is done
                            if (oer) cellp[i * L + c] = (uint16_t)(w | ((uint32_t)oxygen_bin(F[0][i][c], P) << 10));
                        }
                    }
                while (live_mask) {
                    const int idx = first_bit(live_mask);
                    live_mask &= live_mask - 1;
                    const int site = own + (idx / CPL) * L + idx % CPL;
                    const uint32_t w = s_cell[site];
                    const int st = w & 3, age = (w >> 2) & 255;
                    uint32_t thr = (st == QUIESC) ? t3 : (age < ca0 ? t0 : (age < ca1 ? t1 : t2));
                    if (oer) {
                        const int cls = (st == QUIESC) ? 3 : (age < ca0 ? 0 : (age < ca1 ? 1 : 2));
                        thr = s_oer_thr[cls][(w >> 10) & 15u];
                    }
                    const Block4 b = philox10(lat_id(site), (uint32_t)n | (half << 31), r, p, seed_lo, seed_hi);
                    // mitotic death: the cell lives on, marked, until it next divides
                    if (b.w1 >= thr) s_cell[site] = mitotic ? (uint16_t)(w | DOOM_BIT) : (uint16_t)DEAD;
                }
                if (oer) {
#pragma unroll
                    for (int i = 0; i < RPT; ++i)
#pragma unroll
                        for (int c = 0; c < CPL; ++c) cellp[i * L + c] = (uint16_t)(cellp[i * L + c] & ~0x3C00u);
                }
                ++ev;
            }

            // (2) reaction term until the next fraction or the end of the hour,
            // one per site for all three fields in field units: Ro = -kappa_O a.
            // A wave without a cell (padding is EMPTY too) takes the EMPTY term
            // without looking its sites up.
            {
                uint32_t w[RPT][CPL], any = 0;
#pragma unroll
                for (int i = 0; i < RPT; ++i) {
                    load_words<CPL>(cellp + i * L, w[i]);
#pragma unroll
                    for (int c = 0; c < CPL; ++c) any |= w[i][c];
                }
                occupied = __builtin_amdgcn_ballot_w64(any != 0u) != 0;
                const float empty = s_react[EMPTY];
#pragma unroll
                for (int i = 0; i < RPT; ++i)
#pragma unroll
                    for (int c = 0; c < CPL; ++c) Ro[i][c] = realc(c) ? empty : 0.0f;
                if (occupied) {
#pragma unroll
                    for (int i = 0; i < RPT; ++i) {
#pragma unroll
                        for (int c = 0; c + 1 < CPL; c += 2) {   // one look-up for two cells
                            const float2 v = s_react2[(w[i][c] & 3) | ((w[i][c + 1] & 3) << 2)];
                            Ro[i][c] = realc(c) ? v.x : 0.0f;
                            Ro[i][c + 1] = realc(c + 1) ? v.y : 0.0f;
                        }
                        if constexpr (CPL % 2) Ro[i][CPL - 1] = realc(CPL - 1) ? s_react[w[i][CPL - 1] & 3] : 0.0f;
                    }
                }
            }
            // (3) the sub-steps up to a fraction at the half hour, or to the end of the hour
            const bool split = half == 0 && ev < nev && s_ev_step[ev] == rel + 1;
            const int count = split ? a.substeps / 2 : half ? a.substeps - a.substeps / 2 : a.substeps;
            __syncthreads();
            get(UP, hn);
#pragma unroll
            for (int f = 0; f < 3; ++f)                  // the spare row holds nothing outside the sub-steps
#pragma unroll
                for (int c = 0; c < CPL; ++c) F[f][RPT][c] = 0.0f;
            int left = count;
#pragma nounroll
            for (; left >= 2; left -= 2) {
                forward();
                reverse();
            }
            if (left) {                                  // a last single one, its rows moved back by a copy
                forward();
#pragma unroll
                for (int f = 0; f < 3; ++f)
#pragma unroll
                    for (int i = RPT - 1; i >= 0; --i)
#pragma unroll
                        for (int c = 0; c < CPL; ++c) F[f][i][c] = F[f][i ? i - 1 : RPT][c];
            }
            if (!split) break;
        }
        if constexpr (TEAM) {
            // The fields of the rows the neighbours hold as halo are final
            // now (the cell update does not change them): their stores go out
            // here and drain during the cell update; the cell words and the
            // step count follow it.
            if (n + 1 < a.n0 + nsteps) {
                const int t1 = flag_base + n + 1 - a.n0;
                size_t at = (size_t)slot * 3 * plane + lat0;
                asm volatile("" : "+s"(at));
                float* fd = ((t1 & 1) ? a.fields_out : a.fields) + at;
                int exA = a.slab_exA[slab], exB = a.slab_exB[slab];
                int yt = y0;
                asm volatile("" : "+s"(exA), "+s"(exB), "+s"(yt));
#pragma unroll
                for (int i = 0; i < RPT; ++i) {
                    const int y = yt + i;
                    if (real && y >= iy0 && y < iy1 && (y < exA || y >= exB)) {
#pragma unroll
                        for (int f = 0; f < 3; ++f)
#pragma unroll
                            for (int c = 0; c < CPL; ++c)
                                if (realc(c)) fd[f * plane + (size_t)y * LW + x0 + c] = F[f][i][c];
                    }
                }
            }
        }

        const float least_O = least(0), least_G = least(1);
        // (4) cell update.  A tumour fills neighbouring rows, so a wave updating the
        // rows whose fields it holds would leave most waves idle while one or two
        // work; instead wave w takes rows w, w + NW, .. of the workgroup, UC
        // columns per lane, and only rows that hold a cell or touch one.  The
        // fields reach it as two bits in the words of the cells past a
        // threshold.  Bit-parallel over the lane's sites (masks, bit
        // k * UC + c).  Proposers claim an EMPTY target with ds_min_u32 on
        // best[t] (one slot per site, sharing the halo pool) and set the
        // target's bit in s_claim; the smallest key's low two bits name the
        // winner's direction, so no key is kept.
        constexpr uint32_t NEC_BIT = 1u << 10, STARV_BIT = 1u << 11;
        // Environment (none when the wave's smallest values are at or above every
        // threshold, which no value is of a threshold that is no number; x < th
        // <=>  sign bit of x - th: the difference of two finite floats is zero only
        // when they are equal and otherwise keeps the sign of the exact difference).
        if (occupied) {
            const float thOq = s_k.thOq, thGq = s_k.thGq, thOd = s_k.thOd, thGd = s_k.thGd, thHd = s_k.thHd;
            if (dirty || __builtin_amdgcn_ballot_w64(!(least_O >= thOq && least_O >= thOd && least_G >= thGq &&
                                                       least_G >= thGd && least(2) >= thHd)) != 0) {
#pragma unroll
                for (int i = 0; i < RPT; ++i) {
                    uint32_t w[CPL];
                    load_words<CPL>(cellp + i * L, w);
#pragma unroll
                    for (int c = 0; c < CPL; ++c) {
                        const float O = F[0][i][c], Gl = F[1][i][c], H = F[2][i][c];
                        const uint32_t nec = (__float_as_uint(Gl - thGd) | __float_as_uint(O - thOd) | __float_as_uint(H - thHd)) >> 31;
                        const uint32_t starv = (__float_as_uint(O - thOq) | __float_as_uint(Gl - thGq)) >> 31;
                        if ((w[c] & 3u) != EMPTY) w[c] |= nec * NEC_BIT | starv * STARV_BIT;
                    }
                    store_words<CPL>(cellp + i * L, w);
                    __builtin_amdgcn_sched_barrier(0);   // row by row: few registers beside the fields
                }
            }
        }
        __syncthreads();   // the flags are in, the last sub-step's halo reads are done
        uint32_t* best = s_pool;
        // this lane's first column and the wave, opaque: nothing derived from
        // them is held in registers across the step loop
        int ux = lane % (64 / RPU) * UC, uw = wave;
        uint32_t none = NONE_KEY;
        asm volatile("" : "+v"(ux), "+s"(uw), "+v"(none));
        auto row_at = [&](int k) {                       // the row of unit k
            if constexpr (RPU == 1) return uw + NWAVE * k;
            else return (uw + NWAVE * k) * RPU + lane / 32;
        };
        const bool ulane = L == 64 * UC || ux < L;
        constexpr uint32_t ONE = 0x00010001u, AGE4 = 0x03FC03FCu;
        uint32_t in_lattice[NP];                         // bits 0 and 16: the pair's columns are the lattice's
#pragma unroll
        for (int q = 0; q < NP; ++q)
            in_lattice[q] = LW == 64 * UC ? ONE : (uint32_t)(ux + 2 * q < LW) | ((uint32_t)(ux + 2 * q + 1 < LW) << 16);
        // rows that hold a cell, those above or below one, and both
        const uint32_t cell_rows = __builtin_amdgcn_readfirstlane(s_rows[uw]);
        const uint32_t up_rows = uw > 0 ? __builtin_amdgcn_readfirstlane(s_rows[uw > 0 ? uw - 1 : 0])
                                          : __builtin_amdgcn_readfirstlane(s_rows[NWAVE - 1]) << 1;
        const uint32_t dn_rows = uw < NWAVE - 1 ? __builtin_amdgcn_readfirstlane(s_rows[uw < NWAVE - 1 ? uw + 1 : 0])
                                                  : __builtin_amdgcn_readfirstlane(s_rows[0]) >> 1;
        uint32_t near_rows = (cell_rows | up_rows | dn_rows) & (UR == 32 ? ~0u : (1u << UR) - 1u);
        uint32_t own_rows = near_rows;                   // counted: a slab counts its own rows only
        if constexpr (SLAB) {
            uint32_t need = 0, mine = 0;
#pragma unroll
            for (int k = 0; k < UR; ++k) {
                const int y = row_at(k);
                if (RPU == 1) need |= (uint32_t)(y >= iy0 - 2 && y < iy1 + 2) << k;
                mine |= (uint32_t)(y >= iy0 && y < iy1) << k;
            }
            if (RPU == 1) near_rows &= need;
            own_rows = near_rows & mine;
        }
        // The rows' new words before births, two cells per register: bits 0 and 16
        // of a pair hold a flag each, spread over the halves by a packed
        // negation.  A rewritten cell that was no EMPTY one carries WAS_BIT until
        // the births, so that whoever reads it, before or after, sees the
        // snapshot: EMPTY has neither a state nor that bit.
        constexpr uint32_t WAS_BIT = 1u << 15;
        auto empties = [&](uint32_t w) { return ~(w | (w >> 1) | (w >> 15)); };   // in bits 0 and 16 (mask the rest)
        constexpr uint32_t block = UB == 32 ? ~0u : (1u << (UB % 32)) - 1u;
        UMask cand_m[NB], empty_m[NB], doom_m[NB];
        int live = 0;
        {
            const int T_lys = min(s_k.T_lys, 256), T_min = min(s_k.T_min, 256);
            const uint32_t lys4 = (uint32_t)(4 * T_lys) * ONE, min4 = (uint32_t)(4 * T_min) * ONE;
            const uint32_t mitotic = EXT && P.mitotic_death ? ONE : 0u;   // else marks mean nothing
#pragma unroll
            for (int b = 0; b < NB; ++b) {
            cand_m[b] = empty_m[b] = doom_m[b] = 0;
#pragma nounroll                                         // (kept small: the step's code has to stay in the instruction cache)
            for (uint32_t todo = (near_rows >> (b * UB)) & block; todo; todo &= todo - 1) {
                const int j = __builtin_ctz(todo), k = b * UB + j, y = row_at(k);
                uint32_t w[NP], e[NP];
                load_pairs(y, ux, w);
                // keys and claim bits of the row (EMPTY lanes past it excepted)
                if (ulane) {
                    if constexpr (NP == 1) *reinterpret_cast<uint2*>(best + y * L + ux) = make_uint2(none, none);
                    else *reinterpret_cast<uint4*>(best + y * L + ux) = make_uint4(none, none, none, none);
                }
                if (lane % (64 / RPU) < L / 32) s_claim[y * (L / 32) + lane % (64 / RPU)] = 0u;
#pragma unroll
                for (int q = 0; q < NP; ++q) {
                    e[q] = ~(w[q] | (w[q] >> 1)) & in_lattice[q];
                    empty_m[b] |= (UMask)((e[q] | (e[q] >> 15)) & 3u) << (j * UC + 2 * q);
                }
                if (!((cell_rows >> k) & 1u)) continue;  // all EMPTY: births only
                uint32_t free[NP];                       // EMPTY neighbours
#pragma unroll
                for (int q = 0; q < NP; ++q) {
                    uint32_t left = q > 0 ? e[q - 1] : lane_from_left_u32(e[NP - 1]);
                    uint32_t right = q < NP - 1 ? e[q + 1] : lane_from_right_u32(e[0]);
                    if (RPU > 1 && ux == 0) left = 0u;   // the other half's row
                    if (RPU > 1 && ux == L - UC) right = 0u;
                    free[q] = __builtin_amdgcn_alignbit(e[q], left, 16) | __builtin_amdgcn_alignbit(right, e[q], 16);
                }
                auto vertical = [&](bool inside, uint32_t rows, int yn) {
                    if (!inside) return;                 // beyond the slab: not free
                    uint32_t v[NP];
                    if (RPU > 1 || ((rows >> k) & 1u)) {
                        load_pairs(yn, ux, v);
#pragma unroll
                        for (int q = 0; q < NP; ++q) free[q] |= empties(v[q]);
                    } else {
#pragma unroll
                        for (int q = 0; q < NP; ++q) free[q] = ONE;
                    }
                };
                vertical(y > 0, up_rows, y - 1);
                vertical(y < RR - 1, dn_rows, y + 1);
#pragma unroll
                for (int q = 0; q < NP; ++q) {
                    const uint32_t s0 = w[q] & ONE, s1 = (w[q] >> 1) & ONE;
                    const uint32_t alive = s0 ^ s1;      // PROLIF or QUIESC
                    const uint32_t nec = (w[q] >> 10) & ONE, starv = (w[q] >> 11) & ONE;
                    const uint32_t age4 = w[q] & AGE4, older4 = pk_min(pk_add(age4, 4 * ONE), AGE4);
                    // a live cell: DEAD, or QUIESC at its age, or PROLIF and older
                    uint32_t v = bit_select(pk_sub(0u, starv), age4 | (QUIESC * ONE), older4 | (PROLIF * ONE));
                    v = bit_select(pk_sub(0u, nec), DEAD * ONE, v);
                    // a DEAD one: older, or lysed
                    const uint32_t gone = pk_sub(0u, s0 & s1) & pk_sign(pk_sub(older4, lys4)) & (older4 | (DEAD * ONE));
                    const uint32_t was = (s0 | s1) * WAS_BIT;
                    const uint32_t ready = alive & ~(nec | starv) & ~pk_sign(pk_sub(age4, min4));
                    const uint32_t marked = EXT ? ready & (w[q] >> 14) & mitotic : 0u;
                    const uint32_t cand = ready & ~marked & free[q];
                    cand_m[b] |= (UMask)((cand | (cand >> 15)) & 3u) << (j * UC + 2 * q);
                    if constexpr (EXT) doom_m[b] |= (UMask)((marked | (marked >> 15)) & 3u) << (j * UC + 2 * q);
                    if ((own_rows >> k) & 1u) live += __builtin_popcount(alive & ~nec);
                    // what lives keeps its mark, though only mitotic death reads it
                    const uint32_t mark = MARKS ? w[q] & pk_sub(0u, alive & ~nec) & (DOOM_BIT * ONE) : 0u;
                    w[q] = bit_select(pk_sub(0u, alive), v, gone) | was | mark;
                }
                store_pairs(y, ux, w);
            }
            }
        }
        __syncthreads();   // keys and claim bits are reset
        // row and column of bit idx of block b
        auto row_of = [&](int b, int idx) { return row_at(b * UB + idx / UC); };
        auto lat_of = [&](int y, int x) { return (PAD ? y * LW : y * L) + x + lat0; };
        if constexpr (EXT) {
            // marked cells never divide: they draw their block whatever their
            // neighbours and die when ready (mitotic death)
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                UMask m = doom_m[b];
                doom_m[b] = 0;
                while (m) {
                    const int idx = first_bit(m), y = row_of(b, idx), x = ux + idx % UC;
                    m &= m - 1;
                    const Block4 w = philox10(lat_of(y, x), n, r, p, seed_lo, seed_hi);
                    if (w.w3 < s_k.T_div) {
                        doom_m[b] |= (UMask)1 << idx;    // those that die
                        live -= (int)((own_rows >> (b * UB + idx / UC)) & 1u);
                    }
                }
            }
        }
        UMask prop_m[NB], dir0_m[NB], dir1_m[NB];        // proposers, and the two bits of their direction
#pragma unroll
        for (int b = 0; b < NB; ++b) {
            prop_m[b] = dir0_m[b] = dir1_m[b] = 0;
            UMask m = cand_m[b];
            while (m) {
                const int idx = first_bit(m), y = row_of(b, idx), x = ux + idx % UC;
                m &= m - 1;
                const Block4 w = philox10(lat_of(y, x), n, r, p, seed_lo, seed_hi);
                if (w.w3 < s_k.T_div) {
                    const uint16_t* at = s_cell + y * L + x;
                    const uint32_t fm = (uint32_t)(y > 0 && (at[y > 0 ? -L : 0] & (WAS_BIT | 3u)) == EMPTY) |
                                        ((uint32_t)(x + 1 < LW && (at[x + 1 < LW ? 1 : 0] & (WAS_BIT | 3u)) == EMPTY) << 1) |
                                        ((uint32_t)(y < RR - 1 && (at[y < RR - 1 ? L : 0] & (WAS_BIT | 3u)) == EMPTY) << 2) |
                                        ((uint32_t)(x > 0 && (at[x > 0 ? -1 : 0] & (WAS_BIT | 3u)) == EMPTY) << 3);
                    const uint32_t kth = (uint32_t)(((uint64_t)w.w0 * __builtin_popcount(fm)) >> 32);
                    uint32_t rest = fm;
                    for (uint32_t j = 0; j < kth; ++j) rest &= rest - 1;
                    const uint32_t dir = __builtin_ctz(rest);                 // 0 N, 1 E, 2 S, 3 W
                    const int t = y * L + x + (dir == 0 ? -L : dir == 1 ? 1 : dir == 2 ? L : -1);
                    atomicMin(&best[t], ((w.w2 >> 3) << 2) | ((dir + 2) & 3u));
                    atomicOr(&s_claim[t >> 5], 1u << (t & 31));
                    prop_m[b] |= (UMask)1 << idx;
                    dir0_m[b] |= (UMask)(dir & 1u) << idx;
                    dir1_m[b] |= (UMask)(dir >> 1) << idx;
                }
            }
        }
        __syncthreads();   // all claims are in, the snapshot is read
        if (near_rows) {
            UMask fresh_m[NB];                           // winning parents and daughters, at age 0
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                fresh_m[b] = 0;
                UMask m = prop_m[b];
                while (m) {
                    const int idx = first_bit(m);
                    m &= m - 1;
                    const uint32_t dir = ((uint32_t)(dir0_m[b] >> idx) & 1u) | (((uint32_t)(dir1_m[b] >> idx) & 1u) << 1);
                    const int t = row_of(b, idx) * L + ux + idx % UC + (dir == 0 ? -L : dir == 1 ? 1 : dir == 2 ? L : -1);
                    if ((best[t] & 3u) == ((dir + 2) & 3u)) fresh_m[b] |= (UMask)1 << idx;
                }
            }
            uint32_t rows = 0;
#pragma unroll
            for (int b = 0; b < NB; ++b)
#pragma nounroll
            for (uint32_t todo = (near_rows >> (b * UB)) & block; todo; todo &= todo - 1) {
                const int j = __builtin_ctz(todo), k = b * UB + j, y = row_at(k), bit = j * UC, at = y * L + ux;
                const uint32_t born = (s_claim[(ulane ? at : 0) >> 5] >> (at & 31)) & (uint32_t)(empty_m[b] >> bit) &
                                      ((1u << UC) - 1u);
                if ((own_rows >> k) & 1u) live += __builtin_popcount(born);
                const uint32_t fresh = born | (uint32_t)(fresh_m[b] >> bit);
                uint32_t w[NP], any = 0;
                load_pairs(y, ux, w);
#pragma unroll
                for (int q = 0; q < NP; ++q) {
                    // bits 2q and 2q + 1 spread over the halves
                    const uint32_t to = bit_select(0xFFFFu, (uint32_t)((int)(fresh << (31 - 2 * q)) >> 31),
                                                   (uint32_t)((int)(fresh << (30 - 2 * q)) >> 31));
                    if constexpr (EXT) {
                        const uint32_t dies = (uint32_t)(doom_m[b] >> bit);
                        w[q] = bit_select(bit_select(0xFFFFu, (uint32_t)((int)(dies << (31 - 2 * q)) >> 31),
                                                     (uint32_t)((int)(dies << (30 - 2 * q)) >> 31)),
                                          DEAD * ONE, w[q]);
                    }
                    // a winning parent keeps its mark (a daughter's site holds none)
                    w[q] &= ~(WAS_BIT * ONE);
                    w[q] = bit_select(to, PROLIF * ONE | (MARKS ? w[q] & (DOOM_BIT * ONE) : 0u), w[q]);
                    any |= w[q];
                }
                store_pairs(y, ux, w);
                rows |= (uint32_t)(__builtin_amdgcn_ballot_w64(any != 0u) != 0) << k;
            }
            // (5) live count: wave reduction, one LDS atomic per wave
            live = wave_sum(live);
            if (lane == 0) {
                atomicAdd(&s_count[n & 1], live);
                s_rows[uw] = rows;
            }
        }
        if constexpr (!TEAM) mark_low(least_O, least_G, n + 1);   // the cell update changes no field
        __syncthreads();
        if (tid == 0) {
            count = s_count[n & 1];
            s_count[(n + 1) & 1] = 0;
            s_low[n & 1] = 0;                            // for step n + 2
            if (!SLAB && a.traj) a.traj[(size_t)inst * a.nsteps + (n - a.n0)] = count;
            // slabs: this slab's share of step n's count
            if (SLAB && a.traj) atomicAdd(&a.traj[(size_t)inst * a.count_at + n], count);
        }
        if constexpr (TEAM) {
            // publish the cell words of the own rows the neighbours hold as
            // halo (their fields went out after the sub-steps), then the step
            // count
            if (n + 1 >= a.n0 + nsteps) break;
            const int t = n + 1 - a.n0;
            {
                const int t1 = flag_base + t;
                size_t at = (size_t)slot * plane + lat0;
                asm volatile("" : "+s"(at));
                uint16_t* cd = ((t1 & 1) ? a.cells_out : a.cells) + at;
                // (whole rows, dealt to the waves)
                const int exA = a.slab_exA[slab], exB = a.slab_exB[slab], na = exA - iy0, ne = na + iy1 - exB;
                for (int j = wave; j < ne; j += NWAVE) {
                    const int y = j < na ? iy0 + j : exB + j - na;
                    uint32_t w[NP];
                    load_pairs(y, lane * UC, w);
                    if (lane * UC < LW) {
                        uint32_t* row = reinterpret_cast<uint32_t*>(cd + (size_t)y * LW + lane * UC);
                        if constexpr (NP == 1) *row = w[0];
                        else *reinterpret_cast<uint2*>(row) = make_uint2(w[0], w[NP - 1]);
                    }
                }
                // every wave's rows have reached the cache hierarchy before the
                // barrier; one device-scope release then publishes them all
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
                __syncthreads();
                if (tid == 0) {
                    int32_t* flag = a.team_flags + (size_t)slot * a.n_slabs + slab;
                    if (!same_xcd) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
                    else __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup");
                    __hip_atomic_store(flag, (t1 << xcc_bits) | xcc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                }
            }
            // The neighbouring slabs' rows of step n + 1: wait for their step
            // counts, then reload this slab's halo rows from the exchange.
            // Polls are relaxed device-scope loads of both neighbours' counts
            // (its own where there is none), one memory round trip; one
            // acquire fence follows the last.  The compute unit's caches are
            // shared by the workgroup's waves, and none of them reads the
            // exchange rows before the barrier that follows the fence.
            if (tid == 0) {
                int ok = a.spin_limit >= 0;
                const int32_t* flags = a.team_flags + (size_t)slot * a.n_slabs;
                const int up = slab > 0 ? slab - 1 : slab, dn = slab + 1 < a.n_slabs ? slab + 1 : slab;
                int k = 0;
                while (ok) {
                    const int fu = __hip_atomic_load(flags + up, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    const int fd = __hip_atomic_load(flags + dn, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    if ((fu >> xcc_bits) >= flag_base + t && (fd >> xcc_bits) >= flag_base + t) {
                        if (xcc_bits && ((fu ^ xcc) & 15) == 0 && ((fd ^ xcc) & 15) == 0) ok = 2;
                        break;
                    }
                    if (++k > a.spin_limit) { ok = 0; break; }
                    __builtin_amdgcn_s_sleep(1);
                }
                if (ok != 2) __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
                s_team_ok = ok;
            }
            __syncthreads();
            const int waited = __builtin_amdgcn_readfirstlane(s_team_ok);
            team_ok = waited != 0;
            if (!team_ok) break;                     // this workgroup leaves the instance
            // The halo rows [0, iy0) and [iy1, RR) come by LDS DMA, all waves
            // sharing the copy whichever rows are theirs: cell words into
            // their LDS rows (padding columns past LW are not touched and stay
            // EMPTY), fields into the pool, which the sub-steps do not use
            // yet, and from there into their rows' registers.  No register
            // waits for memory, so everything is in flight together.  (One
            // wave loading its own 8 to 14 halo rows into registers, a memory
            // round trip for each, and the fences: 26 us of a 256 x 256 step
            // in slabs of 88 rows beside its sub-steps, now 15.)
            same_xcd = waited == 2;
            int yb = iy0, nh = iy0 + RR - iy1;       // rows above, halo rows in all
            const float* src = (((flag_base + t) & 1) ? a.fields_out : a.fields);
            const uint16_t* cs = (((flag_base + t) & 1) ? a.cells_out : a.cells);
            size_t at = (size_t)slot * plane + lat0; // opaque: row addresses are not hoisted out of the step loop
            asm volatile("" : "+s"(at));
            for (int j = wave; j < nh; j += NWAVE) {
                const int y = j < yb ? j : j + iy1 - yb;
                if (lane < LW / 8)                   // 16 bytes a lane: a row is one instruction
                    __builtin_amdgcn_global_load_lds(
                        (__attribute__((address_space(1))) void*)(cs + at + (size_t)y * LW + 8 * lane),
                        (__attribute__((address_space(3))) void*)(s_cell + y * L), 16, 0, SC1);
            }
            // Pool [field][halo row][LW], or field by field where the rows of all
            // three do not fit (above 15 sub-steps).  Every wave reads a row for
            // each of its own and selects, with no branch: one per row or wave
            // would hold the fields twice.
            const float* gf = src + at + (size_t)slot * 2 * plane;
            const bool one = 3 * nh * LW > G::POOL;
            const float* lf = reinterpret_cast<const float*>(s_pool) + x0;
            int yt = y0;
            asm volatile("" : "+s"(yt));
#pragma unroll
            for (int f = 0; f < 3; ++f) {
                if (f == 0 || one) {
                    if (f > 0) __syncthreads();          // the field before has been read
#pragma nounroll
                    for (int g = f; g < (one ? f + 1 : 3); ++g)
                        for (int j = wave; j < nh; j += NWAVE) {
                            const int y = j < yb ? j : j + iy1 - yb;
                            if (lane < LW / 4)
                                __builtin_amdgcn_global_load_lds(
                                    (__attribute__((address_space(1))) void*)(gf + (size_t)g * plane + (size_t)y * LW + 4 * lane),
                                    (__attribute__((address_space(3))) void*)(s_pool + ((g - f) * nh + j) * LW), 16, 0, SC1);
                        }
                    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the DMA writes are in LDS
                    __syncthreads();
                }
#pragma unroll
                for (int i = 0; i < RPT; ++i) {
                    const int y = yt + i;
                    const bool halo = y < iy0 || y >= iy1;
                    const float* row = lf + (halo ? (one ? 0 : f * nh) + (y < iy0 ? y : y - iy1 + yb) : 0) * LW;
#pragma unroll
                    for (int c = 0; c < CPL; ++c) {
                        const float v = row[c];
                        F[f][i][c] = halo && realc(c) ? v : F[f][i][c];
                        asm volatile("" : "+v"(F[f][i][c]));
                    }
                    if (i % 4 == 3) __builtin_amdgcn_sched_barrier(0);   // few rows in flight beside the fields
                }
            }
            mark_low(least(0), least(1), n + 1);          // the halo rows changed
            __syncthreads();                          // halo cells in before anyone reads them
            scan_rows();
        }
    }

    // The lane and thread index again, from the lane count: keeping them live
    // across the step loop for the uses below would take a register.
    const int lane_end = (int)__builtin_amdgcn_mbcnt_hi(~0u, __builtin_amdgcn_mbcnt_lo(~0u, 0u));
    const int tid_end = wave * 64 + lane_end;
    if ((!SLAB || TEAM) && nsteps == 0) {
        int live = 0;
#pragma unroll
        for (int i = 0; i < RPT; ++i)
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                const int st = s_cell[(y0 + i) * L + x0 + c] & 3;
                live += (st == PROLIF || st == QUIESC) && (!SLAB || (y0 + i >= iy0 && y0 + i < iy1));
            }
        live = wave_sum(live);
        if (lane_end == 0) atomicAdd(&s_count[0], live);
        __syncthreads();
        if (tid_end == 0) count = s_count[0];
    }
    if constexpr (TEAM) {
        // the instance's last step (or its initial state): this slab's share
        if (tid_end == 0 && a.live) {
            if (team_ok) atomicAdd(&a.live[inst], count);
            else atomicExch(&a.live[inst], (int)0x80000000);
        }
        flag_base += nsteps > 1 ? nsteps - 1 : 0;
    } else if constexpr (SLAB) {
        // the instance's last step: add this slab's share of the live count
        if (tid_end == 0 && a.live && a.n0 + 1 == (a.horizon ? a.horizon[p] : a.count_at)) atomicAdd(&a.live[inst], count);
    } else {
        if (tid_end == 0 && a.live) a.live[inst] = count;
    }

    if ((SLAB && !TEAM) || (!TEAM && (a.mode & MODE_STORE))) {
        // slabs write their own rows into the other state buffer
        float* dst = (SLAB ? a.fields_out : a.fields) + (size_t)slot * 3 * plane + lat0;
#pragma unroll
        for (int f = 0; f < 3; ++f)
#pragma unroll
            for (int i = 0; i < RPT; ++i)
                if (real && (!SLAB || (y0 + i >= iy0 && y0 + i < iy1)))
#pragma unroll
                    for (int c = 0; c < CPL; ++c)
                        if (realc(c)) dst[f * plane + (size_t)(y0 + i) * LW + x0 + c] = F[f][i][c];
        __syncthreads();
        uint16_t* cd = (SLAB ? a.cells_out : a.cells) + (size_t)slot * plane + lat0;
#pragma unroll
        for (int i = 0; i < RPT; ++i)
            if (real && (!SLAB || (y0 + i >= iy0 && y0 + i < iy1)))
#pragma unroll
                for (int c = 0; c < CPL; ++c)
                    if (realc(c)) cd[(size_t)(y0 + i) * LW + x0 + c] = s_cell[(y0 + i) * L + x0 + c];
    }
    }
}

}  // namespace
}  // namespace gga
