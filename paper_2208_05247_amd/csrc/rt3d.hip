// rt3d.hip -- Monte Carlo solar photon tracer for gfx950 (MI355X) behind the
// C ABI declared in include/rt3d.h.
//
// Method: the forward Monte Carlo ray tracer of Veerman, van Stratum and van
// Heerwaarden (GRL 2022), sec. 2.3 -- null-collision tracking on a one-level
// acceleration grid, absorption by weights at every scattering or null
// collision, Rayleigh (gas) / Henyey-Greenstein (cloud) scattering, Russian
// roulette below weight 0.5, Lambertian surface, heating and flux tallies.
//
// Design for CDNA4 (not the paper's CUDA design):
//   * persistent kernel, one photon per lane, lanes refilled from a
//     per-wave pool of photon ids that is topped up with one global atomic
//     per pool, so divergent photon lifetimes do not idle the wave; a wave
//     refills once 16 of its lanes are idle, so the emission code runs for
//     many lanes at once;
//   * one loop pass = at most a few acceleration-grid crossings (3 by
//     default) and then the event reached, if any (tentative collision,
//     surface, top): a lane on a long clear-sky walk does not hold its wave
//     through all of it;
//   * majorants staged in LDS when they fit, else read through L1/L2;
//   * integer weights (units of 2^-31) and uint64 tallies: order-independent
//     atomics, bitwise-reproducible results and an exactly closing ledger;
//   * deposits into the same cell by consecutive events of one lane are
//     merged in registers and written with one atomic when the lane moves on;
//   * event counters live in registers and are folded into LDS per photon
//     and into global memory once per workgroup.
#include <hip/hip_runtime.h>

#include <stdint.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <mutex>
#include <type_traits>

#include "rt3d.h"

namespace {

constexpr uint32_t kWOne = 0x80000000u;  // weight one in units of 2^-31
constexpr uint32_t kNoCell = 0xffffffffu;
constexpr uint32_t kNoMajorant = 0x7fffffffu;  // a NaN: never a majorant (those are >= 0, or negated as a flag)
constexpr size_t kLdsMajorantBytes = 64 * 1024;  // automatic LDS staging limit (two workgroups per CU)

// ---------------------------------------------------------------------------
// Philox4x32-10 (Salmon et al., SC'11): per round the counter becomes
// (hi(M1 c2) ^ c1 ^ k0, lo(M1 c2), hi(M0 c0) ^ c3 ^ k1, lo(M0 c0)); the key
// is bumped by the Weyl constants between rounds.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t xor3(uint32_t a, uint32_t b, uint32_t c) {
    return __builtin_amdgcn_bitop3_b32(a, b, c, 0x96);
}

__device__ __forceinline__ uint4 philox(uint4 c, uint32_t k0, uint32_t k1) {
#pragma unroll
    for (int r = 0; r < 10; ++r) {
        if (r) {
            k0 += 0x9E3779B9u;
            k1 += 0xBB67AE85u;
        }
        // both halves of a product from one v_mad_u64_u32 (5.4 cycles a wave
        // against 9.6 for v_mul_lo_u32 + v_mul_hi_u32), three-way xors as one
        // v_bitop3_b32
        const uint64_t p0 = (uint64_t)0xD2511F53u * c.x;
        const uint64_t p1 = (uint64_t)0xCD9E8D57u * c.z;
        c = make_uint4(xor3((uint32_t)(p1 >> 32), c.y, k0), (uint32_t)p1, xor3((uint32_t)(p0 >> 32), c.w, k1),
                       (uint32_t)p0);
    }
    return c;
}

__device__ __forceinline__ uint4 philox(uint4 c, unsigned long long key) {
    return philox(c, (uint32_t)key, (uint32_t)(key >> 32));
}

// 24-bit uniforms: [0,1) for comparisons and positions, (0,1] for logs.
__device__ __forceinline__ float u01(uint32_t u) { return (float)(u >> 8) * 0x1p-24f; }
__device__ __forceinline__ float u01_open(uint32_t u) { return (float)((u >> 8) + 1u) * 0x1p-24f; }

__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// ---------------------------------------------------------------------------
// Scrambled Sobol entry points (sec. 2.3: rays start at the top of the domain
// following a scrambled Sobol sequence).  The p-th photon to enter a column
// takes the p-th point of the 2D Sobol sequence, nested-uniform scrambled
// per column and run.  Dimension 1 is the base-2 radical inverse (bit
// reversal); dimension 2 uses the primitive polynomial x + 1, whose
// direction numbers follow v_1 = 2^31, v_j = v_{j-1} ^ (v_{j-1} >> 1).
__device__ __forceinline__ uint32_t sobol_dim2(uint32_t p) {
    uint32_t v = 0x80000000u, r = 0;
    while (p) {
        if (p & 1u) r ^= v;
        v ^= v >> 1;
        p >>= 1;
    }
    return r;
}

// MurmurHash3's finaliser (a bijective 32-bit mix).
__device__ __forceinline__ uint32_t fmix32(uint32_t h) {
    h ^= h >> 16;
    h *= 0x85ebca6bu;
    h ^= h >> 13;
    h *= 0xc2b2ae35u;
    h ^= h >> 16;
    return h;
}

// Owen's nested uniform scramble of the first kDigits binary digits of v:
// digit d is flipped by the top bit of fmix32(node ^ seed), node = (v's
// first d digits) | 2^d numbering the binary-tree node above that digit.
// Digit d depends only on digits before it, so the first 24 digits of the
// 32-digit scramble are the 24-digit scramble.
template <int kDigits>
__device__ __forceinline__ uint32_t owen_scramble(uint32_t v, uint32_t seed) {
    uint32_t out = 0;
#pragma unroll 4
    for (int d = 0; d < kDigits; ++d) {
        const uint32_t node = (d ? v >> (32 - d) : 0u) | (1u << d);
        out |= (((v >> (31 - d)) ^ (fmix32(node ^ seed) >> 31)) & 1u) << (31 - d);
    }
    return out;
}

// Henyey-Greenstein cos(theta) by inversion of its cumulative distribution,
// mu = (1 + g^2 - s^2) / (2 g) with s = (1 - g^2) / (1 + g a), a = 2 xi - 1.
// For small |g| that quotient cancels catastrophically in FP32; multiplied
// out it is the same function
//   mu = (a + g (a^2 + 3)/2 + g^2 a + g^3 (a^2 - 1)/2) / (1 + g a)^2,
// which is exact at g = 0 (mu = a) and well conditioned while 1 + g a stays
// near 1, so each form is used where it is accurate (|mu error| < 1e-6).
__device__ __forceinline__ float hg_cos(float g, float xi) {
    if (g >= 1.0f) return 1.0f;  // pure forward scattering (0/0 at xi = 0 otherwise)
    const float a = 2.0f * xi - 1.0f;
    float mu;
    if (fabsf(g) < 0.1f) {
        const float d = 1.0f + g * a;
        const float a2 = a * a;
        mu = (a + g * (0.5f * (a2 + 3.0f) + g * (a + g * (0.5f * (a2 - 1.0f))))) / (d * d);
    } else {
        const float s = (1.0f - g * g) / (1.0f - g + 2.0f * g * xi);
        mu = (1.0f + g * g - s * s) / (2.0f * g);
    }
    return fminf(1.0f, fmaxf(-1.0f, mu));
}

// Rayleigh cos(theta): root of mu^3 + 3 mu + 4 - 8 xi = 0 (Cardano).
__device__ __forceinline__ float rayleigh_cos(float xi) {
    const float q = 4.0f * xi - 2.0f;
    const float u = cbrtf(q + sqrtf(q * q + 1.0f));
    return fminf(1.0f, fmaxf(-1.0f, u - rcp(u)));
}

// Turn direction (x,y,z) by polar cosine mu and azimuth 2*pi*t, in the
// frame e1 = (x z, y z, -s^2)/s, e2 = (-y, x, 0)/s with s = |(x, y)|.  s is
// taken from the horizontal components (not sqrt(1 - z^2), which cancels for
// near-vertical d), so the frame stays accurate down to s ~ 1e-12; only a
// direction closer to vertical than that uses the fixed frame (x, y axes).
__device__ __forceinline__ void turn(float& x, float& y, float& z, float mu, float t) {
    float sp, cp;
    __sincosf(6.28318530717958647f * t, &sp, &cp);
    const float st = sqrtf(fmaxf(0.0f, 1.0f - mu * mu));
    float nx, ny, nz;
    // the order of every rounding is written out (see mul_rounded): for a sum
    // of two products the compiler may fuse either, and does not choose the
    // same one in every kernel
    const float s2 = __builtin_fmaf(y, y, x * x);
    if (s2 < 1e-24f) {
        nx = st * cp;
        ny = st * sp;
        nz = z > 0.0f ? mu : -mu;
    } else {
        const float is = rsqrtf(s2);
        const float s = s2 * is;
        nx = __builtin_fmaf(x, mu, st * __builtin_fmaf(x * z, cp, -(y * sp)) * is);
        ny = __builtin_fmaf(y, mu, st * __builtin_fmaf(x, sp, y * z * cp) * is);
        nz = __builtin_fmaf(z, mu, -(cp * st * s));
    }
    const float n = rsqrtf(__builtin_fmaf(nz, nz, __builtin_fmaf(ny, ny, nx * nx)));
    x = nx * n;
    y = ny * n;
    z = nz * n;
}

// ---------------------------------------------------------------------------
// Photon schedule: the order in which the work queue hands out photons.
// Photon k of g-point n (id = photon_offset + k) enters column
// (id + o_n) mod ncol (systematic column sampling with a random offset o_n),
// so every column receives P_n = count_n div ncol photons of g-point n in
// full passes, and the columns of one cyclic range one more.  Queue slots
// run through the full passes entry tile by entry tile (tiles of
// tile_x x tile_y columns, row-major; inside a tile pass by pass over all
// g-points, its columns row-major), then through the remaining photons
// g-point by g-point.  The photons in flight at one time then enter a few
// neighbouring tiles, and the cells and tallies they touch form a small
// working set instead of the whole domain.  Which photons are traced, with
// which random numbers, does not depend on the order, and neither do the
// integer tallies.
// ---------------------------------------------------------------------------
// Division by a launch constant: quotients of 32-bit values below 2^31 as one
// high product and a shift, of 64-bit values below 2^33 by the reciprocal in
// FP64 and a correction by one.  A 64-bit division by a run-time value is
// about 150 instructions, a 32-bit one 22; a photon's emission has six of
// them.
struct FastDiv {
    uint32_t d, mul, shift;
};

inline FastDiv fast_div(uint32_t d) {
    FastDiv f;
    f.d = d;
    f.shift = 0;
    while (((uint64_t)1 << f.shift) < d) ++f.shift;
    f.mul = (uint32_t)(((uint64_t)1 << (31 + f.shift)) / d + 1);
    return f;
}

__device__ __host__ __forceinline__ uint32_t quotient(uint32_t n, const FastDiv& f) {
    return (uint32_t)(((uint64_t)(n << 1) * f.mul) >> 32) >> f.shift;
}

struct FastDiv33 {
    unsigned long long d;
    double inv;
};

inline FastDiv33 fast_div33(unsigned long long d) { return FastDiv33{d, 1.0 / (double)d}; }

__device__ __host__ __forceinline__ unsigned long long quotient(unsigned long long n, const FastDiv33& f,
                                                                unsigned long long* rem) {
#ifndef __HIP_DEVICE_COMPILE__
    if (n >> 33) {  // (a launch has fewer photons; rt3d_schedule_slots takes any number)
        *rem = n % f.d;
        return n / f.d;
    }
#endif
    unsigned long long q = (unsigned long long)((double)n * f.inv);
    long long r = (long long)(n - q * f.d);
    if (r < 0) {
        --q;
        r += (long long)f.d;
    } else if (r >= (long long)f.d) {
        ++q;
        r -= (long long)f.d;
    }
    *rem = (unsigned long long)r;
    return q;
}

struct Schedule {
    const unsigned long long* pass_first;  // [ngp + 1] prefix sums of P_n
    const unsigned long long* rem_first;   // [ngp + 1] prefix sums of count_n mod ncol
    const unsigned long long* col_offset;  // [ngp] o_n
    unsigned long long full_slots;         // ncol * sum P_n
    FastDiv33 tile_slots;                  // tile_cols * sum P_n
    FastDiv33 tile_cols;
    unsigned long long photon_offset;
    FastDiv nx, ntx, tile_x;
    uint32_t ncol, tile_y;
    uint32_t po_mod;  // photon_offset mod ncol
    int ngp;
};

struct Slot {
    int gp;
    unsigned long long id;
    uint32_t col, i, j;  // entry column, col = j nx + i
};

// Prefix sums of the full passes and of the photons left over per g-point.
template <typename Count>
inline void schedule_tables(const Count* photons, int ngp, unsigned long long ncol,
                                                unsigned long long* pass_first, unsigned long long* rem_first) {
    unsigned long long passes = 0, rest = 0;
    for (int n = 0; n < ngp; ++n) {
        pass_first[n] = passes;
        rem_first[n] = rest;
        passes += (unsigned long long)photons[n] / ncol;
        rest += (unsigned long long)photons[n] % ncol;
    }
    pass_first[ngp] = passes;
    rem_first[ngp] = rest;
}

// Index lo with first[lo] <= x < first[lo + 1] (empty ranges skipped).
__host__ __device__ inline int range_of(const unsigned long long* first, int n, unsigned long long x) {
    int lo = 0, hi = n;
    while (hi - lo > 1) {
        const int mid = (lo + hi) >> 1;
        if (first[mid] <= x) lo = mid;
        else hi = mid;
    }
    return lo;
}

__host__ __device__ inline Slot decode_slot(const Schedule& S, unsigned long long s) {
    Slot r;
    unsigned long long k;
    if (s < S.full_slots) {
        unsigned long long rem, ru;
        const uint32_t t = (uint32_t)quotient(s, S.tile_slots, &rem);
        const unsigned long long f = quotient(rem, S.tile_cols, &ru);  // full pass over all g-points
        const uint32_t u = (uint32_t)ru;
        r.gp = range_of(S.pass_first, S.ngp, f);
        const unsigned long long m = f - S.pass_first[r.gp];
        const uint32_t ty = quotient(t, S.ntx), tx = t - ty * S.ntx.d;
        const uint32_t uy = quotient(u, S.tile_x), ux = u - uy * S.tile_x.d;
        r.i = tx * S.tile_x.d + ux;
        r.j = ty * S.tile_y + uy;
        r.col = r.j * S.nx.d + r.i;
        uint32_t o = (uint32_t)S.col_offset[r.gp] + S.po_mod;
        if (o >= S.ncol) o -= S.ncol;
        const uint32_t j = r.col >= o ? r.col - o : r.col + (S.ncol - o);
        k = (unsigned long long)j + m * S.ncol;
    } else {
        const unsigned long long q = s - S.full_slots;
        r.gp = range_of(S.rem_first, S.ngp, q);
        const uint32_t j = (uint32_t)(q - S.rem_first[r.gp]);
        k = (S.pass_first[r.gp + 1] - S.pass_first[r.gp]) * S.ncol + j;
        uint32_t o = (uint32_t)S.col_offset[r.gp] + S.po_mod;
        if (o >= S.ncol) o -= S.ncol;
        r.col = j + o;
        if (r.col >= S.ncol) r.col -= S.ncol;
        r.j = quotient(r.col, S.nx);
        r.i = r.col - r.j * S.nx.d;
    }
    r.id = S.photon_offset + k;
    return r;
}

// ---------------------------------------------------------------------------
// Deposit buffer.  A 64-bit atomic to a heating tally is performed beyond the
// L2, at most 2.37e10 times a second (random words of 32 KB to 256 MB; 1.8e10 on
// 2 GB), and the tracer makes some 30 per photon: 2^26 photons on 256x256x128
// cells 2.2e9, 93 of the 101 ms that they take.  Where the caller's workspace
// has room, deposits are written to memory instead, 8 bytes each in the order
// they come up, and added to the tallies from there:
//   trace_kernel         waves append deposits (cell and direct/diffuse bit,
//                        amount) to chunks of kChunk that they take from the
//                        buffer (wave w the w mod kTileChunks'th chunk of the
//                        next tile: one counter for all would be asked for
//                        more often than the 13 ns an atomic to one address
//                        takes); when it is full, every wave stores its
//                        lanes' photons and ends;
//   deposit_sort_kernel  orders each tile of kTileDeposits by bin (kBinCells
//                        consecutive cells) in place, and writes where each
//                        bin starts in the tile;
//   deposit_add_kernel   one workgroup per bin reads the bin's run of every
//                        tile, sums it in LDS and adds the sums to the tallies.
// Rounds of the three follow until no photon is left; the number launched is
// an upper estimate (a round with nothing to do ends at once), and the last
// one adds what does not fit by atomics.  The sums are of integers: the
// tallies are those of the atomics, bit for bit.
// ---------------------------------------------------------------------------
constexpr uint32_t kChunk = 256;                         // deposits a wave takes room for at a time
constexpr uint32_t kTileChunks = 64;                     // chunks of a tile
constexpr uint32_t kTileDeposits = kChunk * kTileChunks; // 128 KiB, sorted in LDS
constexpr int kBinShift = 13;                            // a bin's 2 x 2^13 sums (64 bits) are 128 KiB of LDS
constexpr uint32_t kBinCells = 1u << kBinShift;
constexpr uint32_t kMaxBins = 2048;
constexpr uint32_t kMaxRounds = 8192;
constexpr int kLaneWords = 24;  // a lane's photon and pending deposits, stored between rounds

struct Deposits {
    uint32_t* used;         // [2][kTileChunks] 128 bytes apart: chunks taken of each column (past ntiles: full)
    unsigned long long* waves;  // [3][nwaves] queue ids left (next, end), finished
    uint32_t* lanes;        // [kLaneWords][nlanes]
    uint32_t* count;        // [ntiles][kTileChunks] deposits in each chunk
    uint16_t* start;        // [ntiles][nbins + 1] first deposit of each bin in a sorted tile
    uint2* item;            // [ntiles][kTileChunks][kChunk] (cell | diffuse << 31, amount)
    uint32_t ntiles, nbins, nwaves, nlanes;

    // Where the addition reads the run [first, last) of the lane'th tile of a
    // group, counted from the group's first tile.  Its loads are not
    // predicated, so a run without deposits (the tile may then lie past the
    // last one, and `first` at the end of the tile) reads the group's first.
    __device__ __host__ static uint32_t run_at(uint32_t lane, uint32_t first, uint32_t last) {
        return last != first ? lane * kTileDeposits + first : 0u;
    }

    // column q's counter in round r (its set is cleared during round r - 1)
    __device__ uint32_t* used_in(int r, uint32_t q) const { return used + 32 * (kTileChunks * (r & 1) + q); }
};

struct TraceParams {
    // medium: kFactored = false: cells = (k_ext, ssa, k_ext_cloud, g) per cell;
    //         kFactored = true:  cells = (k_ext_cloud, cloud k_abs, g, 0) per cell,
    //                            gas = (k_gas, gas k_abs) per g-point and level
    const float4* __restrict__ cells;
    const float2* __restrict__ gas;
    const float* __restrict__ albedo;
    const float* __restrict__ majorant;                    // [ngp][nmaj]
    // factored only (null: not used): per acceleration cell, one bit per fine
    // cell (1 = some cloud extinction), mask_words words per acceleration
    // cell, the bits in x-fastest order of the cell's bx * by * bz fine cells
    const uint32_t* __restrict__ cell_mask;
    int mask_words;
    Schedule sched;
    unsigned long long* abs_dir;
    unsigned long long* abs_dif;
    unsigned long long* sfc_dir;
    unsigned long long* sfc_dif;
    unsigned long long* sfc_abs;
    unsigned long long* toa_up;
    unsigned long long* ledger;
    unsigned long long* stats;
    unsigned long long* queue;
    int ngp, nmaj, max_walk;
    uint32_t pool;   // photon ids a wave takes from the queue at a time
    uint32_t refill; // a wave refills once this many of its lanes are idle
    int merge;       // merge consecutive deposits of a lane into one cell
    int nx, ny, nz, bx, by, bz, mx, my, mz;
    FastDiv div_bx, div_by;
    float dx, dy, dz, inv_dx, inv_dy, inv_dz;
    float cx, cy, cz;  // acceleration-grid cell size in metres
    float H;
    float sun_x, sun_y, sun_z;
    float diffuse_fraction;
    const float* gp_diffuse;  // per-g-point diffuse fraction (batched), or null
    int sobol;                // scrambled Sobol entry positions
    uint32_t rr_below;
    uint32_t max_iters;
    unsigned long long seed;  // g-point n draws with Philox key seed + n
    unsigned long long photons, photon_offset, ncol;
    Deposits dep;             // kBinned only
    int round, last_round;
};

enum { L_IN, L_TOA, L_ATM_DIR, L_ATM_DIF, L_SFC, L_RR_GAIN, L_RR_LOSS, L_LOST, L_N };
enum { S_PHOT, S_COLL, S_NULL, S_GAS, S_CLOUD, S_SFC, S_ESC, S_RR_KILL, S_RR_SURV,
       S_CROSS, S_ABSORBED, S_CAPPED, S_N };

// Tally update.  kAgg false: one atomic per lane.  kAgg true (wave-aggregated):
// the lanes that update the same address in this instruction add their
// values first and one of them issues the atomic; the loop visits each
// distinct address of the active lanes once (scalar, wave-uniform).
template <bool kAgg>
__device__ __forceinline__ void tally_add(unsigned long long* p, unsigned long long v) {
    if (!kAgg) {
        atomicAdd(p, v);
        return;
    }
    uint64_t todo = __ballot(1);
    const uint64_t a = (uint64_t)(uintptr_t)p;
    while (todo) {
        const int l = __ffsll((unsigned long long)todo) - 1;
        const uint64_t al = ((uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(a >> 32), l) << 32) |
                            (uint64_t)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)a, l);
        const uint64_t m = __ballot(a == al);
        unsigned long long sum = 0;
        for (uint64_t mm = m; mm; mm &= mm - 1) {
            const int j = __ffsll((unsigned long long)mm) - 1;
            sum += ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)(v >> 32), j) << 32) |
                   (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)(uint32_t)v, j);
        }
        if ((int)__lane_id() == l) atomicAdd(p, sum);
        todo &= ~m;
    }
}

__device__ __forceinline__ uint64_t lane_mask_lt() {
    const uint32_t lane = __lane_id();
    return lane ? (~0ull >> (64 - lane)) : 0ull;
}

// Local optical properties at a tentative collision: extinction, absorption,
// scattering and cloud extinction coefficients, cloud asymmetry.
struct Local {
    float ke, ka, ks, kc, g;
};

// Factored: `clear` marks a brick without cloud, whose cell records are all
// zero in the fields used here, so the gather is skipped.
template <bool kFactored>
__device__ __forceinline__ Local local_props(const TraceParams& P, int gp, uint32_t cell, int k, bool clear) {
    float4 c = make_float4(0.f, 0.f, 0.f, 0.f);
    if (!kFactored || !clear) c = P.cells[cell];
    Local L;
    if (!kFactored) {
        L.ke = c.x;
        L.ka = c.x * (1.0f - c.y);
        L.ks = c.x * c.y;
        L.kc = c.z;
        L.g = c.w;
    } else {
        const float2 q = P.gas[gp * P.nz + k];
        L.ke = q.x + c.x;
        L.ka = q.y + c.y;
        L.ks = (q.x - q.y) + (c.x - c.y);
        L.kc = c.x;
        L.g = c.z;
    }
    return L;
}

// a * b rounded to FP32 on its own.  The library is built with FP contraction,
// and the backend then fuses any product with a following addition into one
// FMA; the tallies are integers that depend on every rounding of a photon's
// path, so a product that has to be rounded by itself is written this way: the
// empty asm hides where its operand comes from.  (Not a multiplication in asm:
// the compiler knows no hazards there, and one that follows v_rcp_f32 at once
// reads the register before it is written.)
__device__ __forceinline__ float mul_rounded(float a, float b) {
    float r = a * b;
    asm("" : "+v"(r));
    return r;
}

// State of a lane between loop iterations.  kLive lanes track a photon,
// kDead lanes wait for a new one, every other state is a rare event that
// waits until enough lanes of the wave have one (service block below).
enum LaneState { kLive, kDead, kAtSurface, kEscaped, kCappedOut, kRoulette, kAbsorbedOut, kEnded };

// Event counters of a workgroup: kCntSlots copies of each in LDS, lane l
// updates copy l % kCntSlots.  A counter in one LDS word makes the compiler
// emit a serial loop over the lanes of the wave (one address, different
// values) at every update; copies at lane-dependent addresses are one
// ds_add_u64 each.
enum Counter { C_TOA, C_SFC_W, C_GAIN, C_LOSS, C_LOST, C_COLL, C_GAS, C_CLOUD, C_SFC, C_ESC, C_KILL, C_SURV,
               C_ABSORBED, C_CAPPED, C_PASSES, C_ABS_COLL, C_N };
constexpr int kCntSlots = 32;

// A wave handles pending rare events (surface, escape, roulette, photon ended)
// once one in kServiceShare of its photons has one.  About one comes up per
// loop iteration of a full wave; handled at once it costs the wave the whole
// code path for one lane.  A share, not a count: where few photons are left
// in a wave none should wait for long.
constexpr uint32_t kServiceShare = 8;

// One photon per lane.  Each loop iteration of
// a lane: handle its pending rare event or (re)fill the lane with a new
// photon, once enough lanes of the wave need that, draw the free
// path's four random words, walk acceleration-grid cells (at most
// P.max_walk crossings per iteration) until the tentative collision /
// surface / top, then handle a collision (the other events wait).  kLds:
// majorant grid of the single
// g-point staged in LDS.  kFactored: shared cloud field + per-g-point gas
// profiles (several g-points in one launch).  kTally: heating deposits by
// atomics, by wave-aggregated atomics (so are the surface tallies then), or
// through the deposit buffer.
// Rare events deferred, counters at lane-dependent LDS addresses, no scalar
// spills: 4.24e10 vector instructions on the 256x256x128 field with 2^26
// photons against 6.27e10, 98.7 against 100.1 ms (bound by the tally atomics
// there); 32x32x64 cells with 2^14 photons 1.54 against 2.29 ms; 128^3 cells,
// 112 g-points, 4.2e6 photons 6.5 against 7.0 ms.
// Launch shape: the single-g-point kernel runs workgroups of up to 768 lanes,
// two per CU (which share the 160 KB LDS), at 6 waves per SIMD and 80 vector
// registers (8 waves at 64 registers spill with the deposit buffer: 83.0
// against 81.4 ms on the 256x256x128 field); the factored kernel runs 256-lane
// workgroups at 6 waves.
enum Tally { kDirect, kAggregated, kBinned };

template <bool kFactored>
struct Shape_ {
    static constexpr int threads = kFactored ? 256 : 768;
    static constexpr int waves = 6;
};

// The kernel's parameters for code that runs for a small part of the loop
// iterations.  The pointer is opaque to the compiler, so what is read through
// it is loaded there; read as P.x it is loaded ahead of the loop, and the
// scalar registers that this takes are spilled to vector lanes, a
// v_readlane at every use (629 of them in the kernel before).  The parameters are the kernel's only
// argument, at the start of its argument segment.
__device__ __forceinline__ const TraceParams* cold_params() {
    auto q = __builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(q));
    return (const TraceParams*)q;
}

template <bool kLds, bool kFactored, int kTally>
__global__ void __launch_bounds__(Shape_<kFactored>::threads)
    __attribute__((amdgpu_waves_per_eu(Shape_<kFactored>::waves))) trace_kernel(const TraceParams P) {
    constexpr bool kAgg = kTally == kAggregated;
    extern __shared__ float s_maj[];
    __shared__ unsigned long long s_cnt[C_N][kCntSlots];

    const uint32_t wave = blockIdx.x * (blockDim.x / 64) + threadIdx.x / 64;
    const uint32_t lane_ix = blockIdx.x * blockDim.x + threadIdx.x;
    bool drained = false;
    if (kTally == kBinned && P.round) {
        // nothing left to do for the whole workgroup: end (each wave looks at
        // the flags of all: a workgroup reduction takes LDS that the majorants
        // may fill; none is written before all waves are at the next barrier)
        const uint32_t mine = threadIdx.x / 64, lane = threadIdx.x % 64;
        const uint64_t left = __ballot(lane < blockDim.x / 64 && P.dep.waves[2 * P.dep.nwaves + wave - mine + lane] == 0);
        if (!left) return;
        drained = !((left >> mine) & 1);
    }

    for (int i = threadIdx.x; i < C_N * kCntSlots; i += blockDim.x) s_cnt[i / kCntSlots][i % kCntSlots] = 0;
    if (kLds) {
        for (int i = threadIdx.x; i < P.nmaj; i += blockDim.x) s_maj[i] = P.majorant[i];
    }
    __syncthreads();
    const int slot = threadIdx.x % kCntSlots;
    auto count = [&](int c, unsigned long long v) { atomicAdd(&s_cnt[c][slot], v); };

    // ---- per-lane photon state
    int st = kDead;
    unsigned long long id = 0;
    int gp = 0;
    float px = 0.f, py = 0.f, pz = 0.f, ux = 0.f, uy = 0.f, uz = -1.f;
    int bi = 0, bj = 0, bk = 0;
    float tau = -1.f;  // optical depth left on the current free path; < 0: draw a new one
    // majorant of the current acceleration cell once read (kNoMajorant: not
    // yet); a photon stays in its cell across the null collisions there, so
    // the walk re-reads it only after a crossing or a new emission
    float kmaj = __uint_as_float(kNoMajorant);
    uint32_t w = 0, step = 0, iters = 0;
    // random words of the current free path (id, step): event, cos(theta), phi
    uint32_t r_event = 0, r_cos = 0, r_phi = 0;
    bool direct = false;
    // merged deposit: cell index, bit 31 set for diffuse; and the one before
    // it, which the next loop iteration writes out (amount 0: none)
    uint32_t pend_key = kNoCell, pend_amt = 0, out_key = 0, out_amt = 0;
    // per-photon counters (folded into LDS when the photon ends).  Brick
    // crossings and null collisions are derived when the workgroup ends:
    // crossings = passes - collisions - surface hits - escapes - capped,
    // null = collisions - scatterings - photons absorbed at a collision.
    uint32_t n_coll = 0, n_scat = 0;  // n_scat: gas in the low, cloud in the high 16 bits

    // ---- per-wave photon-id pool (wave-uniform, kept in scalar registers)
    unsigned long long pool_next = 0, pool_end = 0;

    // ---- kBinned: the wave's chunk of the deposit buffer (wave-uniform)
    constexpr uint32_t kNoChunk = 0xffffffffu;
    uint32_t chunk = kNoChunk, chunk_pos = kChunk;
    bool full = false, suspended = false, resumed = false;

    auto uniform = [](unsigned long long v) {
        return ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(v >> 32)) << 32) |
               (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)v);
    };
    // every word of a lane's state that lives from one round to the next
    auto each_word = [&](auto&& f) {
        uint32_t lo = (uint32_t)id, hi = (uint32_t)(id >> 32), fl = (uint32_t)st | (direct ? 256u : 0u);
        auto fw = [&](int n, float& v) {
            uint32_t b = __float_as_uint(v);
            f(n, b);
            v = __uint_as_float(b);
        };
        auto iw = [&](int n, int& v) {
            uint32_t b = (uint32_t)v;
            f(n, b);
            v = (int)b;
        };
        f(0, lo); f(1, hi); f(2, fl); iw(3, gp);
        fw(4, px); fw(5, py); fw(6, pz); fw(7, ux); fw(8, uy); fw(9, uz);
        iw(10, bi); iw(11, bj); iw(12, bk); fw(13, tau); fw(14, kmaj);
        f(15, w); f(16, step); f(17, iters); f(18, pend_key); f(19, pend_amt); f(20, out_key); f(21, out_amt);
        f(22, n_coll); f(23, n_scat);
        static_assert(kLaneWords == 24, "one word per field");
        id = (unsigned long long)lo | ((unsigned long long)hi << 32);
        st = (int)(fl & 255u);
        direct = fl & 256u;
    };
    if (kTally == kBinned && P.round && !drained) {
        const Deposits& D = cold_params()->dep;
        each_word([&](int n, uint32_t& v) { v = D.lanes[(size_t)n * D.nlanes + lane_ix]; });
        pool_next = uniform(D.waves[wave]);
        pool_end = uniform(D.waves[D.nwaves + wave]);
        drained = pool_next >= cold_params()->photons;
        resumed = true;
    }
    auto add_heat = [&](uint32_t key, uint32_t amt) {
        const uint32_t cell = key & 0x7fffffffu;
        tally_add<kAgg>(key & 0x80000000u ? &P.abs_dif[cell] : &P.abs_dir[cell], (unsigned long long)amt);
    };
    auto flush_scat = [&]() {
        count(C_GAS, n_scat & 0xffffu);
        count(C_CLOUD, n_scat >> 16);
        n_scat = 0;
    };
    // the g-point's Philox key (opaque in each use: the round keys are then
    // formed where they are needed, see cold_params)
    auto key = [&]() {
        unsigned long long q = P.seed;
        asm volatile("" : "+s"(q));
        return q + (unsigned long long)(kFactored ? gp : 0);
    };
    auto words = [&](uint32_t at_step) {
        return philox(make_uint4((uint32_t)id, (uint32_t)(id >> 32), at_step, 0u), key());
    };
    auto keep_words = [&](uint4 r) {
        r_event = r.y;
        r_cos = r.z;
        r_phi = r.w;
    };
    if (kTally == kBinned && resumed) keep_words(words(step));
    auto cell_ix = [&](float v, float inv, int b, int n) {
        return min(max((int)floorf(v * inv), b * n), b * n + n - 1);
    };

    for (;;) {
        // ---- the deposits of the last iteration
        if (kTally != kBinned) {
            if (out_amt) add_heat(out_key, out_amt);
            out_amt = 0;
        } else if (const uint64_t depositing = __ballot(out_amt != 0)) {
            const uint32_t n = (uint32_t)__popcll(depositing);
            if (chunk_pos + n > kChunk && !full) {
                const Deposits& D = cold_params()->dep;
                if (chunk != kNoChunk && __lane_id() == 0) D.count[chunk] = chunk_pos;
                // its own column first, then a few others that are not used up
                chunk = kNoChunk;
                chunk_pos = 0;
                for (uint32_t q = 0; q < 8 && chunk == kNoChunk; ++q) {
                    const uint32_t column = (wave + 9 * q) % kTileChunks;
                    uint32_t c = 0;
                    if (__lane_id() == 0) c = atomicAdd(D.used_in(cold_params()->round, column), 1u);
                    c = (uint32_t)__builtin_amdgcn_readfirstlane((int)c);
                    if (c < D.ntiles) chunk = c * kTileChunks + column;
                }
                if (chunk == kNoChunk) {
                    // no room: end here, and go on in the next round; but once
                    // no new photons come, the few deposits left are added by
                    // atomics (the longest photons' time is spent once then)
                    full = true;
                    // (one lane's load for all: read 16 lanes at a time, the
                    // counter may pass the photons in between, and the wave's
                    // lanes must not part here)
                    unsigned long long handed_out = 0;
                    if (__lane_id() == 0)
                        handed_out = __hip_atomic_load(cold_params()->queue, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    handed_out = uniform(handed_out);
                    if (!cold_params()->last_round && handed_out < cold_params()->photons) {
                        suspended = true;
                        break;
                    }
                }
            }
            if (!full) {
                if (out_amt)
                    P.dep.item[(size_t)chunk * kChunk + chunk_pos + (uint32_t)__popcll(depositing & lane_mask_lt())] =
                        make_uint2(out_key, out_amt);
                chunk_pos += n;
            } else if (out_amt) {
                add_heat(out_key, out_amt);
            }
            out_amt = 0;
        }
        // ---- rare events, once enough lanes wait with one or none is live
        const uint64_t waiting = __ballot(st > kDead);
        if (waiting && kServiceShare * (uint32_t)__popcll(waiting) >= (uint32_t)__popcll(__ballot(st != kDead))) {
            const TraceParams& Q = *cold_params();
            if (st == kAtSurface) {
                // ---- Lambertian surface (sec. 2.3)
                const int i = cell_ix(px, Q.inv_dx, bi, Q.bx);
                const int j = cell_ix(py, Q.inv_dy, bj, Q.by);
                const int c2 = j * Q.nx + i;
                tally_add<kAgg>(direct ? &Q.sfc_dir[c2] : &Q.sfc_dif[c2], (unsigned long long)w);
                const uint32_t wn = min(w, (uint32_t)rintf(Q.albedo[c2] * (float)w));
                if (w != wn) {
                    tally_add<kAgg>(&Q.sfc_abs[c2], (unsigned long long)(w - wn));
                    count(C_SFC_W, w - wn);
                }
                count(C_SFC, 1);
                w = wn;
                if (w == 0) {
                    count(C_ABSORBED, 1);
                    st = kEnded;
                } else {
                    const float mu = sqrtf(u01_open(r_cos));
                    float sp, cp;
                    __sincosf(6.28318530717958647f * u01(r_phi), &sp, &cp);
                    const float sn = sqrtf(fmaxf(0.0f, 1.0f - mu * mu));
                    ux = sn * cp;
                    uy = sn * sp;
                    uz = mu;
                    direct = false;
                    if (w < Q.rr_below) {
                        st = kRoulette;
                    } else {
                        ++step;
                        st = kLive;
                    }
                }
            }
            if (st == kRoulette) {
                // Russian roulette (sec. 2.3) with the free path's counter
                // (id, step, 1): survive with probability w, then weight one
                const uint4 q = philox(make_uint4((uint32_t)id, (uint32_t)(id >> 32), step, 1u), key());
                if ((q.x >> 1) < w) {
                    count(C_GAIN, kWOne - w);
                    count(C_SURV, 1);
                    w = kWOne;
                    ++step;
                    st = kLive;
                } else {
                    count(C_LOSS, w);
                    count(C_KILL, 1);
                    st = kEnded;
                }
            }
            if (st == kEscaped) {
                // ---- leaves through the top of the domain
                const int i = cell_ix(px, Q.inv_dx, bi, Q.bx);
                const int j = cell_ix(py, Q.inv_dy, bj, Q.by);
                tally_add<kAgg>(&Q.toa_up[j * Q.nx + i], (unsigned long long)w);
                count(C_TOA, w);
                count(C_ESC, 1);
            }
            if (st == kCappedOut) {
                count(C_LOST, w);
                count(C_CAPPED, 1);
            }
            if (st == kAbsorbedOut) {
                count(C_ABSORBED, 1);
                count(C_ABS_COLL, 1);
            }
            if (st > kDead) {  // the photon has ended
                st = kDead;
                count(C_COLL, n_coll);
                count(C_PASSES, iters);
                flush_scat();
                n_coll = 0;
            }
        }
        // ---- refill finished lanes from the wave's pool of photon ids, once
        // enough of them are idle (the emission code then runs for many
        // lanes at once instead of for one or two) or none is alive
        const uint64_t dead = __ballot(st == kDead);
        if (dead && !drained && ((uint32_t)__popcll(dead) >= P.refill || !__ballot(st != kDead))) {
            const uint32_t need = (uint32_t)__popcll(dead);
            const int leader = __ffsll((unsigned long long)dead) - 1;
            const unsigned long long avail = pool_end - pool_next;
            unsigned long long base = 0;
            if (avail < need) {
                if ((int)__lane_id() == leader) base = atomicAdd(P.queue, (unsigned long long)P.pool);
                base = __shfl(base, leader);
                // readfirstlane returns a signed int: widen through uint32_t
                base = ((unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)(base >> 32)) << 32) |
                       (unsigned long long)(uint32_t)__builtin_amdgcn_readfirstlane((uint32_t)base);
            }
            if (st == kDead) {
                const uint32_t rank = (uint32_t)__popcll(dead & lane_mask_lt());
                const unsigned long long local = rank < avail ? pool_next + rank : base + (rank - avail);
                // (a grab may hold fewer ids than lanes wait: the others try
                // again in the next iteration)
                if (rank < avail + P.pool && local < P.photons) {
                    // queue slot -> g-point, photon id and entry column
                    const TraceParams& Q = *cold_params();
                    const Slot sl = decode_slot(Q.sched, local);
                    gp = kFactored ? sl.gp : 0;
                    id = sl.id;
                    const int ic = (int)sl.i, jc = (int)sl.j;
                    // ---- emission at the top of the domain (sec. 2.3)
                    const uint4 e = philox(make_uint4((uint32_t)id, (uint32_t)(id >> 32), 0xffffffffu, 0u),
                                           key());
                    float fx = u01(e.x), fy = u01(e.y);
                    if (Q.sobol) {
                        // photon id is the (id div ncol)-th to enter its column
                        const uint32_t pass = (uint32_t)(id / Q.ncol);
                        const uint4 sc = philox(make_uint4(sl.col, 0u, 0xfffffffdu, 0u),
                                                key());
                        fx = u01(owen_scramble<24>(__builtin_bitreverse32(pass), sc.x));
                        fy = u01(owen_scramble<24>(sobol_dim2(pass), sc.y));
                    }
                    px = ((float)ic + fx) * Q.dx;
                    py = ((float)jc + fy) * Q.dy;
                    pz = Q.H;
                    const float fd = Q.gp_diffuse ? Q.gp_diffuse[gp] : Q.diffuse_fraction;
                    if (u01(e.z) < fd) {
                        const uint4 q = philox(make_uint4((uint32_t)id, (uint32_t)(id >> 32), 0xffffffffu, 1u),
                                               key());
                        const float mu = sqrtf(u01_open(q.x));
                        float sp, cp;
                        __sincosf(6.28318530717958647f * u01(q.y), &sp, &cp);
                        const float sn = sqrtf(fmaxf(0.0f, 1.0f - mu * mu));
                        ux = sn * cp;
                        uy = sn * sp;
                        uz = -mu;
                        direct = false;
                    } else {
                        ux = Q.sun_x;
                        uy = Q.sun_y;
                        uz = Q.sun_z;
                        direct = true;
                    }
                    bi = (int)quotient((uint32_t)ic, Q.div_bx);
                    bj = (int)quotient((uint32_t)jc, Q.div_by);
                    bk = Q.mz - 1;
                    kmaj = __uint_as_float(kNoMajorant);
                    w = kWOne;
                    step = 0;
                    iters = 0;
                    tau = -1.f;
                    st = kLive;
                }
            }
            if (avail < need) {
                pool_next = base + min((unsigned long long)P.pool, need - avail);
                pool_end = base + P.pool;
            } else {
                pool_next += need;
            }
            // ids only grow (pool first, later grabs above pool_end), so once
            // pool_next passes the photon count no valid id is left
            drained = pool_next >= P.photons;
        }
        if (!__ballot(st == kLive)) {
            if (!__ballot(st > kDead) && drained) break;
            continue;
        }
        if (st != kLive) continue;

        // ---- a free path after an emission or a rare event: its length and
        // random words (after a collision they are formed there)
        if (tau < 0.f) {
            const uint4 r = words(step);
            tau = -__logf(u01_open(r.x));
            asm volatile("" : "+v"(tau));
            keep_words(r);
        }
        const int maj_base = kFactored ? gp * P.nmaj : 0;  // this g-point's majorant grid

        // ---- walk acceleration-grid cells until the path ends
        const float rx = rcp(ux), ry = rcp(uy), rz = rcp(uz);
        bool hit = false;
        for (int walked = 0;; ++walked) {
            if (iters >= P.max_iters) { st = kCappedOut; break; }
            if (walked >= P.max_walk) break;
            ++iters;
            // factored majorants carry the brick's "no cloud" flag in the sign bit
            if (__float_as_uint(kmaj) == kNoMajorant)
                kmaj = kLds ? s_maj[(bk * P.my + bj) * P.mx + bi] : P.majorant[maj_base + (bk * P.my + bj) * P.mx + bi];
            const float Km = fabsf(kmaj);
            // distance to the cell's face ahead in each direction
            auto ahead = [](float p, float u, float ru, int b, float c) {
                const float lo = mul_rounded((float)b, c);
                const float face = u > 0.f ? lo + c : lo;
                return fmaxf(u == 0.f ? INFINITY : (face - p) * ru, 0.f);
            };
            const float tx = ahead(px, ux, rx, bi, P.cx);
            const float ty = ahead(py, uy, ry, bj, P.cy);
            const float tz = ahead(pz, uz, rz, bk, P.cz);
            const float txy = fminf(tx, ty);
            const float s_exit = fminf(txy, tz);
            const float depth = mul_rounded(Km, s_exit);
            hit = depth >= tau;
            const float go = hit ? tau * rcp(Km) : s_exit;
            px = __builtin_fmaf(go, ux, px);
            py = __builtin_fmaf(go, uy, py);
            pz = __builtin_fmaf(go, uz, pz);
            if (hit) break;
            tau -= depth;
            // into the next cell; ties go to x before y before z
            if (tz < txy) {
                const int up = uz < 0.f ? -1 : 1;
                const int nk = bk + up;
                pz = mul_rounded((float)(uz < 0.f ? bk : nk), P.cz);
                if ((unsigned)nk >= (unsigned)P.mz) {
                    st = uz < 0.f ? kAtSurface : kEscaped;
                    break;
                }
                bk = nk;
            } else if (ty < tx) {
                int nb = bj + (uy > 0.f ? 1 : -1);
                nb = nb < 0 ? P.my - 1 : nb == P.my ? 0 : nb;
                bj = nb;
                py = mul_rounded((float)(uy > 0.f ? nb : nb + 1), P.cy);
            } else {
                int nb = bi + (ux > 0.f ? 1 : -1);
                nb = nb < 0 ? P.mx - 1 : nb == P.mx ? 0 : nb;
                bi = nb;
                px = mul_rounded((float)(ux > 0.f ? nb : nb + 1), P.cx);
            }
            kmaj = __uint_as_float(kNoMajorant);  // crossed into another cell
        }
        if (st == kLive && !hit) continue;  // same free path next iteration
        tau = -1.f;
        if (!hit) continue;  // a rare event: waits for the service block

        // ---- tentative collision: local properties from the fine grid
        const int i = cell_ix(px, P.inv_dx, bi, P.bx);
        const int j = cell_ix(py, P.inv_dy, bj, P.by);
        const int k = cell_ix(pz, P.inv_dz, bk, P.bz);
        const uint32_t cell = (uint32_t)((k * P.ny + j) * P.nx + i);
        bool clear = kFactored && __float_as_uint(kmaj) >> 31;
        if (kFactored && !clear && P.cell_mask) {
            // a cloud-free fine cell of a cloudy acceleration cell holds a
            // zero record too: its bit, from a small array that stays in
            // the L2, spares the gather of a whole line of records
            const uint32_t t = (uint32_t)(((k - bk * P.bz) * P.by + (j - bj * P.by)) * P.bx + (i - bi * P.bx));
            const uint32_t b = (uint32_t)((bk * P.my + bj) * P.mx + bi);
            clear = !((P.cell_mask[(size_t)b * P.mask_words + (t >> 5)] >> (t & 31)) & 1u);
        }
        const float K = fabsf(kmaj);
        const Local L = local_props<kFactored>(P, gp, cell, k, clear);
        // the next free path's random words and length, while the cell's
        // record is on its way (16384 photons on 32x32x64, where few waves
        // are live: 620 -> 596 us; none where many hide the latency)
        uint4 rn = words(step + 1);
        float tau_next = -__logf(u01_open(rn.x));
        asm volatile("" : "+v"(tau_next), "+v"(rn.y), "+v"(rn.z), "+v"(rn.w));  // (not put off to their use)
        const float iK = rcp(K);
        ++n_coll;
        if (L.ka > 0.f) {
            const uint32_t dep = min(w, (uint32_t)rintf((float)w * (L.ka * iK)));
            const uint32_t key = cell | (direct ? 0u : 0x80000000u);
            // the merged deposit goes out when the photon deposits elsewhere
            // (or its sum would pass 32 bits)
            if (key != pend_key || pend_amt + dep < dep || !P.merge) {
                out_key = pend_key;
                out_amt = pend_amt;
                pend_key = key;
                pend_amt = 0;
            }
            pend_amt += dep;
            w -= dep;
            if (w == 0) {
                st = kAbsorbedOut;
                continue;
            }
        }
        // scattering with probability k_sca / (K - k_abs), else null
        const float den = K - L.ka;
        const float ps = den > 0.f ? L.ks * rcp(den) : 0.f;
        const float xi = u01(r_event);
        if (xi < ps) {
            float mu;
            if (xi * L.ke < ps * L.kc) {
                mu = hg_cos(L.g, u01(r_cos));
                n_scat += 0x10000u;
            } else {
                mu = rayleigh_cos(u01(r_cos));
                n_scat += 1u;
            }
            turn(ux, uy, uz, mu, u01(r_phi));
            direct = false;
            if ((n_scat & 0x8000u) | (n_scat & 0x80000000u)) flush_scat();
        }
        if (w < P.rr_below) {
            st = kRoulette;
        } else {
            ++step;
            tau = tau_next;
            keep_words(rn);
        }
    }

    const TraceParams& Q = *cold_params();
    if (kTally == kBinned) {
        const Deposits& D = Q.dep;
        if (chunk != kNoChunk && __lane_id() == 0) D.count[chunk] = chunk_pos;
        if (suspended) {
            each_word([&](int n, uint32_t& v) { D.lanes[(size_t)n * D.nlanes + lane_ix] = v; });
            pend_amt = 0;  // (not yet added)
        }
        if (__lane_id() == 0) {
            D.waves[wave] = pool_next;
            D.waves[D.nwaves + wave] = pool_end;
            D.waves[2 * D.nwaves + wave] = suspended ? 0 : 1;
        }
    }
    if (pend_amt) add_heat(pend_key, pend_amt);
    __syncthreads();
    // sums of the counter copies, then the ledger and stats entries
    __shared__ unsigned long long s_sum[C_N];
    if (threadIdx.x < C_N) {
        unsigned long long v = 0;
        for (int q = 0; q < kCntSlots; ++q) v += s_cnt[threadIdx.x][q];
        s_sum[threadIdx.x] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        auto led = [&](int e, unsigned long long v) { if (v) atomicAdd(&Q.ledger[e], v); };
        auto sta = [&](int e, unsigned long long v) { if (v) atomicAdd(&Q.stats[e], v); };
        if (blockIdx.x == 0 && Q.round == 0) {  // every queue slot is traced, each with weight one
            led(L_IN, Q.photons * kWOne);
            sta(S_PHOT, Q.photons);
        }
        led(L_TOA, s_sum[C_TOA]);
        led(L_SFC, s_sum[C_SFC_W]);
        led(L_RR_GAIN, s_sum[C_GAIN]);
        led(L_RR_LOSS, s_sum[C_LOSS]);
        led(L_LOST, s_sum[C_LOST]);
        const unsigned long long coll = s_sum[C_COLL], gas = s_sum[C_GAS], cloud = s_sum[C_CLOUD];
        sta(S_COLL, coll);
        sta(S_NULL, coll - gas - cloud - s_sum[C_ABS_COLL]);
        sta(S_GAS, gas);
        sta(S_CLOUD, cloud);
        sta(S_SFC, s_sum[C_SFC]);
        sta(S_ESC, s_sum[C_ESC]);
        sta(S_RR_KILL, s_sum[C_KILL]);
        sta(S_RR_SURV, s_sum[C_SURV]);
        sta(S_CROSS, s_sum[C_PASSES] - coll - s_sum[C_SFC] - s_sum[C_ESC] - s_sum[C_CAPPED]);
        sta(S_ABSORBED, s_sum[C_ABSORBED]);
        sta(S_CAPPED, s_sum[C_CAPPED]);
    }
}

// The longest column: the maximum over the wave's lanes of their counters.
__device__ __forceinline__ uint32_t tiles_used(uint32_t mine) {
    static_assert(kTileChunks == 64, "one column per lane");
    for (int o = 32; o > 0; o >>= 1) mine = max(mine, (uint32_t)__shfl_xor((int)mine, o));
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)mine);
}

// Sorts each tile of the deposit buffer by bin, in place.  One workgroup per
// tile: its 16384 deposits (16 a lane, in registers) count themselves into LDS
// counters per bin, which also gives each its rank within the bin, the counts
// are scanned to the bins' starts, and the tile is put in order in LDS and
// written back in one piece (scattered 8-byte stores to memory would be
// 32 bytes each).  Bound by its 16 bytes of memory traffic per deposit.
__global__ void __launch_bounds__(1024) deposit_sort_kernel(const Deposits D, int round) {
    __shared__ uint2 s_item[kTileDeposits];
    __shared__ uint32_t s_bin[kMaxBins];
    __shared__ uint32_t s_part[16];
    __shared__ uint32_t s_total;
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    __shared__ uint32_t s_used[kTileChunks];
    if (tid < kTileChunks) {
        s_used[tid] = *D.used_in(round, tid);
        if (blockIdx.x == 0) *D.used_in(round + 1, tid) = 0;
    }
    __syncthreads();
    const uint32_t ntiles = min(tiles_used(s_used[lane]), D.ntiles);
    constexpr int kPer = kTileDeposits / 1024;
    uint2 v[kPer];
    auto load = [&](uint32_t t) {
        const uint2* tile = D.item + (size_t)t * kTileDeposits;
#pragma unroll
        for (int i = 0; i < kPer; ++i) {
            const uint32_t p = i * 1024 + tid, c = p / kChunk;
            v[i] = make_uint2(0u, 0u);
            if (t < s_used[c] && p % kChunk < D.count[t * kTileChunks + c]) v[i] = tile[p];
        }
    };
    if (blockIdx.x < ntiles) load(blockIdx.x);
#pragma unroll 1
    for (uint32_t t = blockIdx.x; t < ntiles; t += gridDim.x) {
        for (uint32_t b = tid; b < D.nbins; b += 1024) s_bin[b] = 0;
        __syncthreads();
        uint2* tile = D.item + (size_t)t * kTileDeposits;
        uint32_t rank[kPer];
#pragma unroll
        for (int i = 0; i < kPer; ++i)  // (a deposit's amount is never 0)
            if (v[i].y) rank[i] = atomicAdd(&s_bin[(v[i].x & 0x7fffffffu) >> kBinShift], 1u);
        __syncthreads();
        // exclusive scan of the counts, two bins a lane
        const uint32_t c0 = 2 * tid < D.nbins ? s_bin[2 * tid] : 0u;
        const uint32_t c1 = 2 * tid + 1 < D.nbins ? s_bin[2 * tid + 1] : 0u;
        uint32_t sum = c0 + c1;
        for (int o = 1; o < 64; o <<= 1) {
            const uint32_t u = __shfl_up(sum, o);
            if ((int)lane >= o) sum += u;
        }
        if (lane == 63) s_part[wave] = sum;
        __syncthreads();
        uint32_t before = sum - c0 - c1;
        for (uint32_t q = 0; q < wave; ++q) before += s_part[q];
        uint16_t* start = D.start + (size_t)t * (D.nbins + 1);
        if (2 * tid < D.nbins) {
            s_bin[2 * tid] = before;
            start[2 * tid] = (uint16_t)before;
        }
        if (2 * tid + 1 < D.nbins) {
            s_bin[2 * tid + 1] = before + c0;
            start[2 * tid + 1] = (uint16_t)(before + c0);
        }
        if (tid == 1023) {
            s_total = before + c0 + c1;
            start[D.nbins] = (uint16_t)(before + c0 + c1);
        }
        __syncthreads();
#pragma unroll
        for (int i = 0; i < kPer; ++i)
            if (v[i].y) s_item[s_bin[(v[i].x & 0x7fffffffu) >> kBinShift] + rank[i]] = v[i];
        __syncthreads();
        const uint32_t total = s_total;
        // the next tile's deposits are on their way while this one is stored
        if (t + gridDim.x < ntiles) load(t + gridDim.x);
        for (uint32_t p = tid; p < total; p += 1024) tile[p] = s_item[p];
        __syncthreads();  // before the next tile clears the counters
    }
}

// Adds the deposits of one bin to the tallies: each half-wave takes the bin's
// run of one sorted tile at a time (the run's place from the table, read for
// 64 tiles at once), 16 tiles in flight per half-wave, and sums it in LDS;
// the sums that are not zero are then added to the tallies, by atomics (other
// calls may accumulate into the same tallies on other streams meanwhile; and a
// load and a store take longer: 2^26 photons on 256x256x128 cells 80.9 against
// 80.2 ms, with a buffer of 1024 tiles 92.5 against 88.2).  Neighbouring bins run on the same XCD, so that the
// 128-byte lines of the table are shared in its L2.
__global__ void __launch_bounds__(1024) deposit_add_kernel(const Deposits D, int round, uint32_t ncell,
                                                           unsigned long long* abs_dir, unsigned long long* abs_dif) {
    __shared__ unsigned long long s_sum[2 * kBinCells];
    const uint32_t tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const uint32_t per_xcd = (D.nbins + 7) / 8;
    const uint32_t bin = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
    const uint32_t ntiles = min(tiles_used(*D.used_in(round, lane)), D.ntiles);
    if (bin >= D.nbins || ntiles == 0) return;
    for (uint32_t i = tid; i < 2 * kBinCells; i += 1024) s_sum[i] = 0;
    __syncthreads();
    const uint32_t hl = lane & 31;
    constexpr int kFlight = 16;
    auto place = [&](uint32_t t, uint32_t& first, uint32_t& last) {
        first = last = 0;
        if (t < ntiles) {
            const uint16_t* start = D.start + (size_t)t * (D.nbins + 1) + bin;
            first = start[0];
            last = start[1];
        }
    };
    uint32_t first_next, last_next;
    place(wave * 64 + lane, first_next, last_next);
    for (uint32_t t0 = wave * 64; t0 < ntiles; t0 += 16 * 64) {
        const uint32_t first = first_next, last = last_next;
        place(t0 + 16 * 64 + lane, first_next, last_next);
        // the run of tile t0 + l: where it starts (counted from tile t0) and its length
        const uint32_t at = Deposits::run_at(lane, first, last), len = last - first;
        const uint2* item = D.item + (size_t)t0 * kTileDeposits;
        auto sum = [&](const uint2& v) {
            atomicAdd(&s_sum[(v.x & (kBinCells - 1)) | ((v.x >> 31) << kBinShift)], (unsigned long long)v.y);
        };
#pragma unroll 1
        for (int q = 0; q < 64; q += 2 * kFlight) {
            uint2 v[kFlight];
            uint32_t n[kFlight];
#pragma unroll
            for (int f = 0; f < kFlight; ++f) {
                const int src = q + 2 * f + (int)(lane >> 5);
                const uint32_t from = __shfl(at, src);
                n[f] = __shfl(len, src);
                // (a lane past the run reads its first deposit again: no branch
                // between the loads, so all of them are in flight)
                v[f] = item[from + (hl < n[f] ? hl : 0u)];
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int f = 0; f < kFlight; ++f)
                if (hl < n[f]) sum(v[f]);
            // runs of more than 32
            bool more = false;
#pragma unroll
            for (int f = 0; f < kFlight; ++f) more |= n[f] > 32;
            if (__ballot(more)) {
                for (int f = 0; f < 2 * kFlight; f += 2) {
                    const int src = q + f + (int)(lane >> 5);
                    const uint32_t from = __shfl(at, src), m = __shfl(len, src);
                    for (uint32_t i = 32 + hl; i < m; i += 32) sum(item[from + i]);
                }
            }
        }
    }
    __syncthreads();
    for (uint32_t i = tid; i < kBinCells; i += 1024) {
        const size_t cell = (size_t)bin * kBinCells + i;
        if (cell >= ncell) break;
        if (s_sum[i]) atomicAdd(&abs_dir[cell], s_sum[i]);
        if (s_sum[kBinCells + i]) atomicAdd(&abs_dif[cell], s_sum[kBinCells + i]);
    }
}

__global__ void clear_atm_kernel(unsigned long long* ledger) {
    if (threadIdx.x == 0) ledger[L_ATM_DIR] = ledger[L_ATM_DIF] = 0;
}

// Heating entries of the energy ledger: ledger[ATM_DIR] = sum(abs_dir),
// ledger[ATM_DIF] = sum(abs_dif), exact uint64 sums (the other entries are
// counted by the tracing kernel, so the identity still checks that no
// deposit was lost).  The two entries hold 0 here; every workgroup adds its
// partial sums.
__global__ void ledger_atm_kernel(const unsigned long long* __restrict__ abs_dir,
                                  const unsigned long long* __restrict__ abs_dif, size_t n,
                                  unsigned long long* __restrict__ ledger) {
    __shared__ unsigned long long part[2][256];
    unsigned long long sd = 0, sf = 0;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        sd += abs_dir[i];
        sf += abs_dif[i];
    }
    part[0][threadIdx.x] = sd;
    part[1][threadIdx.x] = sf;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            part[0][threadIdx.x] += part[0][threadIdx.x + h];
            part[1][threadIdx.x] += part[1][threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        if (part[0][0]) atomicAdd(&ledger[L_ATM_DIR], part[0][0]);
        if (part[1][0]) atomicAdd(&ledger[L_ATM_DIF], part[1][0]);
    }
}

// Row maxima of the acceleration cells, formed while a wave packs 64 cells: a
// row of bx (a power of two, at most a wave) cells is that many lanes next to
// each other, and the first of them merges their maximum into `out` with an
// integer max of the FP32 bits (exact, as every value is >= +0; non-positive
// values and NaN count as 0).  Level k goes to out[k / bz][j / by][bi].  As a
// pass of its own (a lane per row, reading its cells one after the other) the
// levels' maxima of 1024x1024x128 cells took 2.3 ms; packing and maxima here
// take 0.8 together.
struct RowMax {
    uint32_t* out;  // null: none (rows_fit is false)
    FastDiv bx, mx, ny, by, bz;
    int nmx, nmy;   // acceleration cells in x and y

    __device__ __forceinline__ void operator()(uint32_t cell, bool valid, float v) const {
        uint32_t m = valid && v > 0.0f ? __float_as_uint(v) : 0u;
        for (uint32_t o = 1; o < bx.d; o <<= 1) m = max(m, (uint32_t)__shfl_xor((int)m, (int)o));
        if (!valid || (threadIdx.x & (bx.d - 1))) return;
        const uint32_t t = quotient(cell, bx), row = quotient(t, mx), k = quotient(row, ny);
        const uint32_t bi = t - row * mx.d, j = row - k * ny.d;
        atomicMax(&out[((size_t)quotient(k, bz) * nmy + quotient(j, by)) * nmx + bi], m);
    }
};

// Interleave the four SoA property arrays into one 16-byte record per cell,
// so a tentative collision needs a single random 16-byte gather; and the
// majorants of the acceleration cells.
__global__ void pack_cells_kernel(const float* __restrict__ ke, const float* __restrict__ om,
                                  const float* __restrict__ kc, const float* __restrict__ g,
                                  float4* __restrict__ out, size_t n, const RowMax rows) {
    const int lane = threadIdx.x & 63;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i - lane < n; i += (size_t)gridDim.x * blockDim.x) {
        const float k = i < n ? ke[i] : 0.0f;
        if (i < n) out[i] = make_float4(k, om[i], kc[i], g[i]);
        if (rows.out) rows((uint32_t)i, i < n, k);
    }
}

// Factored medium: per cell (k_ext_cloud, cloud k_abs, g, 0), and per level and
// acceleration column the largest cloud extinction; per g-point and level
// (k_gas, gas k_abs).
__global__ void pack_cloud_kernel(const float* __restrict__ kc, const float* __restrict__ om,
                                  const float* __restrict__ g, float4* __restrict__ out, size_t n, const RowMax rows,
                                  const float* __restrict__ kg, const float* __restrict__ og,
                                  float2* __restrict__ gas, size_t ngas) {
    const int lane = threadIdx.x & 63;
    const size_t first = blockIdx.x * (size_t)blockDim.x + threadIdx.x, step = (size_t)gridDim.x * blockDim.x;
    for (size_t i = first; i < ngas; i += step) gas[i] = make_float2(kg[i], kg[i] * (1.0f - og[i]));
    for (size_t i = first; i - lane < n; i += step) {
        const float k = i < n ? kc[i] : 0.0f;
        if (i < n) out[i] = make_float4(k, k * (1.0f - om[i]), g[i], 0.0f);
        if (rows.out) rows((uint32_t)i, i < n, k);
    }
}

// Factored medium: the cloud-cell mask of the tracer, one 32-bit word per
// thread: bit s of word q of acceleration cell b is fine cell t = 32 q + s of
// that cell (x fastest, then y, then z), set where k_ext_cloud != 0 (a cell
// whose bit is clear has the record (0, 0, g, 0), whose g is never used).
__global__ void cell_mask_kernel(const float* __restrict__ kc, uint32_t* __restrict__ mask, int nx, int ny, int bx,
                                 int by, int bz, int mx, int my, int words, size_t n) {
    const int nb = bx * by * bz;
    for (size_t w = blockIdx.x * (size_t)blockDim.x + threadIdx.x; w < n; w += (size_t)gridDim.x * blockDim.x) {
        const size_t b = w / words;
        const int q = (int)(w % words);
        const int bi = (int)(b % mx), bj = (int)((b / mx) % my), bk = (int)(b / ((size_t)mx * my));
        uint32_t m = 0;
        for (int s = 0; s < 32; ++s) {
            const int t = 32 * q + s;
            if (t >= nb) break;
            const int ix = t % bx, jy = (t / bx) % by, kz = t / (bx * by);
            const size_t cell = ((size_t)(bk * bz + kz) * ny + (size_t)(bj * by + jy)) * nx + (size_t)(bi * bx + ix);
            if (kc[cell] != 0.0f) m |= 1u << s;
        }
        mask[w] = m;
    }
}

// Factored majorant, step 1: per level k and acceleration column (bi, bj),
// the largest cloud extinction: layer[k][bj][bi] (FP32 bits, integer max).
// For bricks whose rows RowMax does not take.
__global__ void layer_max_kernel(const float4* __restrict__ cells, uint32_t* __restrict__ layer, int nx, int ny,
                                 int nz, int bx, int by) {
    const int mx = nx / bx, my = ny / by;
    const size_t n = (size_t)mx * ny * nz;
    for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x) {
        const int bi = (int)(t % mx);
        const size_t row = t / mx;  // j + ny * k
        const int j = (int)(row % ny);
        const int k = (int)(row / ny);
        const float4* src = cells + row * nx + (size_t)bi * bx;
        uint32_t m = 0;
        for (int q = 0; q < bx; ++q) {
            const float v = src[q].x;
            const uint32_t bits = v > 0.0f ? __float_as_uint(v) : 0u;
            m = bits > m ? bits : m;
        }
        atomicMax(&layer[((size_t)k * my + j / by) * mx + bi], m);
    }
}

// Factored majorant, step 2: K[n][bk][bj][bi] = max over the levels k of
// brick layer bk of (k_gas[n][k] + layer[k][bj][bi]).  FP32 addition is
// monotonic, so this equals the largest k_gas + k_cloud of the cells.  A
// brick with no cloud extinction in any cell stores -K (sign bit set, -0 for
// K = 0): the tracer reads |K| and skips the cell gather there.
__global__ void gas_majorant_kernel(const uint32_t* __restrict__ layer, const float2* __restrict__ gas,
                                    float* __restrict__ maj, int ngp, int nz, int mx, int my, int bz) {
    const int mz = nz / bz;
    const size_t nmaj = (size_t)mx * my * mz;
    const size_t n = nmaj * ngp;
    for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x) {
        const int gp = (int)(t / nmaj);
        const size_t b = t % nmaj;
        const size_t col = b % ((size_t)mx * my);
        const int bk = (int)(b / ((size_t)mx * my));
        float m = 0.0f;
        uint32_t cloud = 0;
        for (int q = 0; q < bz; ++q) {
            const int k = bk * bz + q;
            const uint32_t lc = layer[(size_t)k * mx * my + col];
            const float v = gas[(size_t)gp * nz + k].x + __uint_as_float(lc);
            m = v > m ? v : m;
            cloud |= lc;
        }
        maj[t] = __uint_as_float(__float_as_uint(m) | (cloud ? 0u : 0x80000000u));
    }
}

// What a trace needs before its kernels, in one launch (a launch costs 2-3 us of
// a small trace; these were 11 of its 16): the control block (photon-id queue,
// validation flag) and the per-g-point schedule by the last workgroup, zeros in
// the tallies and in the majorants to be merged by the others.
// Schedule: prefix sums of the full passes over all columns and of the photons
// left over, and systematic-sampling column offsets (Philox counter
// (0, 0, 0xfffffffe, 0) under the g-point's key, word 0).
constexpr size_t kCtrlBytes = 256;  // queue counter + validation flag
constexpr int kMaxGpoints = 256;
constexpr int kMaxClears = 10;
struct Setup {
    unsigned long long photons[kMaxGpoints];
    unsigned long long seed, ncol;
    unsigned long long *control, *pass_first, *rem_first, *gp_col_offset;  // control null: clears only
    unsigned long long* clear[kMaxClears];
    size_t words[kMaxClears];  // 64-bit words of each
    int ngp, nclear;
};

__global__ void __launch_bounds__(256) setup_kernel(const Setup a) {
    static_assert(kMaxGpoints <= 256, "one g-point a lane");
    __shared__ unsigned long long s_pass[kMaxGpoints], s_rest[kMaxGpoints];
    const int t = threadIdx.x;
    if (a.control && blockIdx.x == gridDim.x - 1) {
        for (int i = t; i < (int)(kCtrlBytes / 8); i += 256) a.control[i] = 0;
        if (t < a.ngp) {
            s_pass[t] = a.photons[t] / a.ncol;
            s_rest[t] = a.photons[t] % a.ncol;
            const unsigned long long key = a.seed + (unsigned long long)t;
            const uint4 r = philox(make_uint4(0u, 0u, 0xfffffffeu, 0u), (uint32_t)key, (uint32_t)(key >> 32));
            a.gp_col_offset[t] = ((unsigned long long)r.x * a.ncol) >> 32;
        }
        __syncthreads();
        for (int n = t; n <= a.ngp; n += 256) {
            unsigned long long passes = 0, rest = 0;
            for (int m = 0; m < n; ++m) {
                passes += s_pass[m];
                rest += s_rest[m];
            }
            a.pass_first[n] = passes;
            a.rem_first[n] = rest;
        }
    }
    for (int q = 0; q < a.nclear; ++q) {
        unsigned long long* const p = a.clear[q];
        const size_t n = a.words[q];
        for (size_t i = blockIdx.x * (size_t)256 + t; i < n; i += (size_t)gridDim.x * 256) p[i] = 0;
    }
}

// ---------------------------------------------------------------------------
// Small kernels
// ---------------------------------------------------------------------------
__global__ void fill_u32_kernel(uint32_t* p, size_t n, uint32_t v) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        p[i] = v;
}

// Row pass of the majorant build: thread (bi, j, k) takes the maximum of
// the bx cells of row (j, k) inside acceleration cell column bi and merges it
// into the acceleration cell with an integer max of the FP32 bits (exact,
// as every value is >= +0; non-positive values and NaN count as 0).
__global__ void majorant_kernel(const float* __restrict__ k_ext, uint32_t* __restrict__ maj, int nx, int ny,
                                int nz, int bx, int by, int bz) {
    const int mx = nx / bx, my = ny / by;
    const size_t n = (size_t)mx * ny * nz;
    for (size_t t = blockIdx.x * (size_t)blockDim.x + threadIdx.x; t < n; t += (size_t)gridDim.x * blockDim.x) {
        const int bi = (int)(t % mx);
        const size_t row = t / mx;  // j + ny * k
        const int j = (int)(row % ny);
        const int k = (int)(row / ny);
        const float* src = k_ext + row * nx + (size_t)bi * bx;
        uint32_t m = 0;
        for (int q = 0; q < bx; ++q) {
            const float v = src[q];
            const uint32_t bits = v > 0.0f ? __float_as_uint(v) : 0u;
            m = bits > m ? bits : m;
        }
        atomicMax(&maj[((size_t)(k / bz) * my + j / by) * mx + bi], m);
    }
}

// Validation of the inputs: sets bit 0 of *flag for any violation.
__global__ void validate_kernel(const float* __restrict__ ke, const float* __restrict__ kc,
                                const float* __restrict__ om, const float* __restrict__ g,
                                const float* __restrict__ alb, size_t ncell, size_t ncol, uint32_t* flag) {
    uint32_t bad = 0;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < ncell; i += (size_t)gridDim.x * blockDim.x) {
        const float a = ke[i], b = kc[i], c = om[i], d = g[i];
        const bool ok = (a >= 0.f) && (a < INFINITY) && (b >= 0.f) && (b <= a) && (c >= 0.f) && (c <= 1.f) &&
                        (d >= -1.f) && (d <= 1.f);
        bad |= ok ? 0u : 1u;
    }
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < ncol; i += (size_t)gridDim.x * blockDim.x) {
        const float a = alb[i];
        bad |= (a >= 0.f && a <= 1.f) ? 0u : 1u;
    }
    if (__ballot(bad) && __lane_id() == 0) atomicOr(flag, 1u);
}

__global__ void validate_batched_kernel(const float* __restrict__ kg, const float* __restrict__ og, size_t ngas,
                                        const float* __restrict__ kc, const float* __restrict__ oc,
                                        const float* __restrict__ g, const float* __restrict__ alb, size_t ncell,
                                        size_t ncol, const float* __restrict__ fd, int ngp, uint32_t* flag) {
    uint32_t bad = 0;
    const size_t s0 = blockIdx.x * (size_t)blockDim.x + threadIdx.x, st = (size_t)gridDim.x * blockDim.x;
    if (fd)
        for (size_t i = s0; i < (size_t)ngp; i += st) bad |= (fd[i] >= 0.f && fd[i] <= 1.f) ? 0u : 1u;
    for (size_t i = s0; i < ngas; i += st) {
        const float a = kg[i], b = og[i];
        bad |= (a >= 0.f && a < INFINITY && b >= 0.f && b <= 1.f) ? 0u : 1u;
    }
    for (size_t i = s0; i < ncell; i += st) {
        const float a = kc[i], b = oc[i], d = g[i];
        bad |= (a >= 0.f && a < INFINITY && b >= 0.f && b <= 1.f && d >= -1.f && d <= 1.f) ? 0u : 1u;
    }
    for (size_t i = s0; i < ncol; i += st) {
        const float a = alb[i];
        bad |= (a >= 0.f && a <= 1.f) ? 0u : 1u;
    }
    if (__ballot(bad) && __lane_id() == 0) atomicOr(flag, 1u);
}

// Tallies to normalised FP32, up to six arrays in one launch: a workgroup
// takes kFinalizeItems elements of one of them, four per lane at a time (two
// 16-byte loads, one 16-byte store where the arrays are aligned).  Bound by
// memory: 512x512x96 cells 5.7 TB/s of 12 bytes an element, 3.9 with one
// element per lane, a 64-bit division for its level and a launch per array.
constexpr unsigned kFinalizeItems = 2048;
struct FinalizeArgs {
    const unsigned long long* src[6];
    float* dst[6];
    const double* level[6];  // scale per level, or null
    double norm[6];
    uint32_t n[6];
    uint32_t first[7];  // first workgroup of each array
    FastDiv plane;
};

__global__ void __launch_bounds__(256) finalize_kernel(const FinalizeArgs a) {
    int t = 0;
    while (blockIdx.x >= a.first[t + 1]) ++t;
    const unsigned long long* const src = a.src[t];
    float* const dst = a.dst[t];
    const double* const level = a.level[t];
    const double norm = a.norm[t];
    const uint32_t n = a.n[t], i0 = (blockIdx.x - a.first[t]) * kFinalizeItems + 4 * threadIdx.x;
    const bool wide = (((uintptr_t)src | (uintptr_t)dst) & 15) == 0;
    auto scale = [&](uint32_t i) { return level ? level[quotient(i, a.plane)] * norm : norm; };
#pragma unroll
    for (uint32_t r = 0; r < kFinalizeItems; r += 1024) {
        const uint32_t i = i0 + r;
        if (wide && i + 4 <= n) {
            const ulonglong2 u = *(const ulonglong2*)(src + i), v = *(const ulonglong2*)(src + i + 2);
            double s[4];
            s[0] = s[1] = s[2] = s[3] = scale(i);
            if (level && quotient(i, a.plane) != quotient(i + 3, a.plane))
                for (int k = 1; k < 4; ++k) s[k] = scale(i + k);
            *(float4*)(dst + i) = make_float4((float)((double)u.x * s[0]), (float)((double)u.y * s[1]),
                                              (float)((double)v.x * s[2]), (float)((double)v.y * s[3]));
        } else {
            for (uint32_t k = i; k < min(i + 4, n); ++k) dst[k] = (float)((double)src[k] * scale(k));
        }
    }
}

__global__ void philox_kernel(const uint4* __restrict__ ctr, uint32_t k0, uint32_t k1, uint4* __restrict__ out,
                              uint32_t n) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = philox(ctr[i], k0, k1);
}

// Entry coordinates of passes first .. first+n-1 of one column, all 32
// digits scrambled (the tracer uses the first 24 of the same values).
__global__ void sobol_entry_kernel(unsigned long long first, uint32_t n, unsigned long long col, uint32_t k0,
                                   uint32_t k1, uint2* __restrict__ out) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    const uint4 sc = philox(make_uint4((uint32_t)col, (uint32_t)(col >> 32), 0xfffffffdu, 0u), k0, k1);
    const uint32_t p = (uint32_t)(first + i);
    out[i] = make_uint2(owen_scramble<32>(__builtin_bitreverse32(p), sc.x), owen_scramble<32>(sobol_dim2(p), sc.y));
}

// The tracer's scattering-angle samplers and direction turn, element-wise,
// for tests: kind 0 = Henyey-Greenstein with g[i], kind 1 = Rayleigh.
__global__ void phase_sample_kernel(int kind, const float* __restrict__ g, const float* __restrict__ xi,
                                    float* __restrict__ mu, uint32_t n) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) mu[i] = kind == 0 ? hg_cos(g[i], xi[i]) : rayleigh_cos(xi[i]);
}

__global__ void turn_kernel(const float* __restrict__ din, const float* __restrict__ mu, const float* __restrict__ t,
                            float* __restrict__ dout, uint32_t n) {
    const uint32_t i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n) return;
    float x = din[3 * i], y = din[3 * i + 1], z = din[3 * i + 2];
    turn(x, y, z, mu[i], t[i]);
    dout[3 * i] = x;
    dout[3 * i + 1] = y;
    dout[3 * i + 2] = z;
}

// ---------------------------------------------------------------------------
// Host side
// ---------------------------------------------------------------------------
thread_local char g_err[256] = "";
thread_local hipEvent_t g_t0 = nullptr, g_t1 = nullptr;
thread_local bool g_timed = false;

rt3d_status dev_fail(hipError_t e, const char* where) {
    snprintf(g_err, sizeof g_err, "%s: %s", where, hipGetErrorString(e));
    return RT3D_EDEVICE;
}

#define HIP_TRY(expr)                                  \
    do {                                               \
        hipError_t e_ = (expr);                        \
        if (e_ != hipSuccess) return dev_fail(e_, #expr); \
    } while (0)

struct Shape {
    int nx, ny, nz, bx, by, bz, mx, my, mz;
    size_t ncell, ncol, nmaj;
};

bool grid_ok(const rt3d_grid* g) {
    if (!g || g->nx <= 0 || g->ny <= 0 || g->nz <= 0) return false;
    if (!(g->dx > 0.f) || !(g->dy > 0.f) || !(g->dz > 0.f)) return false;
    if (!std::isfinite(g->dx) || !std::isfinite(g->dy) || !std::isfinite(g->dz)) return false;
    const long long n = (long long)g->nx * g->ny * g->nz;
    return n < 0x7fffffffLL;
}

void resolve_options(const rt3d_grid* g, const rt3d_options* in, rt3d_options* out) {
    rt3d_default_options(out);
    if (in) *out = *in;
    if (out->brick_x <= 0) out->brick_x = g->nx % 8 == 0 ? 8 : 1;
    if (out->brick_y <= 0) out->brick_y = g->ny % 8 == 0 ? 8 : 1;
    if (out->brick_z <= 0) out->brick_z = g->nz % 8 == 0 ? 8 : 1;
    if (out->max_iters == 0) out->max_iters = 1u << 24;
}

bool shape_of(const rt3d_grid* g, const rt3d_options* o, Shape* s) {
    if (!grid_ok(g)) return false;
    if (o->brick_x <= 0 || o->brick_y <= 0 || o->brick_z <= 0) return false;
    if (g->nx % o->brick_x || g->ny % o->brick_y || g->nz % o->brick_z) return false;
    s->nx = g->nx; s->ny = g->ny; s->nz = g->nz;
    s->bx = o->brick_x; s->by = o->brick_y; s->bz = o->brick_z;
    s->mx = g->nx / o->brick_x; s->my = g->ny / o->brick_y; s->mz = g->nz / o->brick_z;
    s->ncell = (size_t)g->nx * g->ny * g->nz;
    s->ncol = (size_t)g->nx * g->ny;
    s->nmaj = (size_t)s->mx * s->my * s->mz;
    return true;
}

size_t align256(size_t b) { return (b + 255) & ~(size_t)255; }

unsigned grid_for(size_t n, unsigned block = 256, unsigned cap = 8192) {
    size_t g = (n + block - 1) / block;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (unsigned)g;
}

// Workspace layout (every section 256-byte aligned):
//   control  256 B: photon-id queue counter, validation flag
//   meta     schedule tables: full passes [ngp + 1], photons left over
//            [ngp + 1], column offsets [ngp] (uint64)
//   maj      majorants [ngp][nmaj] FP32
//   cells    packed per-cell records [ncell] float4
//   gas      factored only: (k_gas, gas k_abs) [ngp][nz] float2
//   layer    factored only: per-level cloud maxima [nz][my][mx] uint32
//   mask     factored only: cloud-cell bits [nmaj][mask_words] uint32
struct Layout {
    size_t meta, maj, cells, gas, layer, mask, total;
};

int mask_words_of(const Shape& s) { return (s.bx * s.by * s.bz + 31) / 32; }

Layout layout_of(const Shape& s, int ngp, bool factored) {
    Layout l;
    size_t off = kCtrlBytes;
    l.meta = off;
    off += align256(sizeof(unsigned long long) * (3 * (size_t)ngp + 2));
    l.maj = off;
    off += align256(sizeof(float) * s.nmaj * ngp);
    l.cells = off;
    off += align256(sizeof(float4) * s.ncell);
    l.gas = l.layer = l.mask = 0;
    if (factored) {
        l.gas = off;
        off += align256(sizeof(float2) * (size_t)ngp * s.nz);
        l.layer = off;
        off += align256(sizeof(uint32_t) * (size_t)s.nz * s.my * s.mx);
        l.mask = off;
        off += align256(sizeof(uint32_t) * s.nmaj * (size_t)mask_words_of(s));
    }
    l.total = off;
    return l;
}

// Entry tiles of the photon schedule: tile_x x tile_y columns, each edge a
// divisor of the grid's.  Automatic: tiles whose columns hold about
// kTileFootprintBytes of cell records and heating tallies (32 bytes per
// cell), close to square, the whole domain when it holds less.  Measured on
// one MI355X (same photons, bitwise-identical tallies, kernel time against
// one whole-domain tile): 1024x1024x128, 112 g-points, 1024 photons per
// column: 128x128 -11.3 %, 64x64 -10.4 %, 16x16 -9.4 %; 512x512x96: 256x256
// and 128x256 -10.3 %, 64x64 -2.5 %, 16x16 +4.3 %; 256x256x128, one g-point
// (fits the Infinity Cache already): 128x128 +0.8 %, 32x32 +7.2 %.
constexpr size_t kTileFootprintBytes = size_t(128) << 20;

uint32_t largest_divisor_upto(int n, long long cap) {
    for (long long d = cap < n ? cap : n; d > 1; --d)
        if (n % d == 0) return (uint32_t)d;
    return 1u;
}

void tile_shape(const Shape& s, const rt3d_options& o, uint32_t* tx, uint32_t* ty) {
    const long long target = (long long)std::max<size_t>(1, kTileFootprintBytes / ((size_t)s.nz * 32));
    if (o.tile_x > 0 && o.tile_y > 0) {
        *tx = (uint32_t)o.tile_x;
        *ty = (uint32_t)o.tile_y;
    } else if (o.tile_x > 0) {
        *tx = (uint32_t)o.tile_x;
        *ty = largest_divisor_upto(s.ny, std::max<long long>(1, target / o.tile_x));
    } else if (o.tile_y > 0) {
        *ty = (uint32_t)o.tile_y;
        *tx = largest_divisor_upto(s.nx, std::max<long long>(1, target / o.tile_y));
    } else if (target >= (long long)s.ncol) {
        *tx = (uint32_t)s.nx;
        *ty = (uint32_t)s.ny;
    } else {
        *tx = largest_divisor_upto(s.nx, std::max<long long>(1, (long long)std::sqrt((double)target)));
        *ty = largest_divisor_upto(s.ny, std::max<long long>(1, target / *tx));
        if (*ty == (uint32_t)s.ny) *tx = largest_divisor_upto(s.nx, std::max<long long>(1, target / s.ny));
    }
}

void schedule_of(const Shape& s, int ngp, const uint64_t* photons, const rt3d_options& o,
                 const unsigned long long* pass_first, const unsigned long long* rem_first,
                 const unsigned long long* col_offset, Schedule* S) {
    unsigned long long passes = 0;
    for (int n = 0; n < ngp; ++n) passes += photons[n] / s.ncol;
    S->pass_first = pass_first;
    S->rem_first = rem_first;
    S->col_offset = col_offset;
    S->ngp = ngp;
    S->ncol = (uint32_t)s.ncol;
    S->nx = fast_div((uint32_t)s.nx);
    uint32_t tx, ty;
    tile_shape(s, o, &tx, &ty);
    S->tile_x = fast_div(tx);
    S->tile_y = ty;
    S->ntx = fast_div((uint32_t)s.nx / tx);
    S->full_slots = passes * s.ncol;
    // never used as a divisor without full passes (full_slots is 0 then)
    S->tile_cols = fast_div33((unsigned long long)tx * ty);
    S->tile_slots = fast_div33(std::max(1ull, passes * S->tile_cols.d));
    S->photon_offset = o.photon_offset;
    S->po_mod = (uint32_t)(o.photon_offset % s.ncol);
}

// The deposit buffer in the part of the workspace behind the sections above,
// or false where there is no room for it or no use: one g-point, 128 to 2048
// bins, and enough tiles and photons (a round costs its three launches, the
// lanes' states written and read, and a pass over the tallies).  Whole calls in
// ms on a cumulus field, 16-byte records of 256x256x128 cells being 134 MB:
//                             atomics   buffer of 256 tiles  512   1024   2048   4096   8192
//   128x64x128   (128)  2^22     8.36       11.0   8.6    7.4    7.2    7.3    7.3
//                       2^26   110.5       158.6 113.4   90.5   92.1   92.3   92.9
//   128x128x128  (256)  2^22     7.37        8.9   7.4    6.3    6.2    6.3    6.1
//                       2^26    95.8       120.7  90.2   74.4   74.6   72.5   70.9
//   256x128x128  (512)  2^22     7.60       11.5   7.8    6.9    6.8    6.7    6.7
//                       2^23    13.76       18.3  14.6   12.1   12.0   11.9   12.4
//   256x256x128 (1024)  2^22     7.77       10.2   8.3    7.2    7.0    6.8    6.8
//                       2^26   100.7       140.0 103.9   88.2   84.4   81.5   80.2
//   256x256x160 (1280)  2^22     8.20         -     -     7.9    7.6    7.6     -
//                       2^24    27.8          -     -    26.0   25.0   24.4     -
//   256x256x256 (2048)  2^22     8.94       13.2  10.8    9.5    9.4    9.1    9.1
//                       2^23    16.1        24.9  19.4   16.9   16.1   15.9   15.7
//                       2^26   115.4       190.5 141.9  120.0  114.0  109.7  108.4
// Fewer bins (tiles of eight workspaces, before the last changes): 64x64x64 (32
// bins) 8.2 / 8.7 at 2^22 photons, 28.6 / 28.7 at 2^24; 90x66x50 (37), 6e6
// photons 8.6 / 11.3: few workgroups add unlike bins.  Of the 80 ms at 2^26
// photons on 256x256x128 cells the sort takes 13 (2.5 TB/s) and the addition 13.
// The kernel for several g-points, slower itself, gained at most 2 % (128^3
// cells, 112 g-points, 3.4e7 photons: 38.3 / 37.4 ms) and lost up to 4 % below
// 8e6 photons, so it keeps the atomics.
constexpr size_t kMinBins = 128;
constexpr size_t kFewBins = 1280;

unsigned long long min_photons(size_t nbins) { return 1ull << (nbins <= kFewBins ? 22 : 23); }
size_t min_tiles(size_t nbins) { return nbins <= kFewBins ? 1024 : 3072; }

bool deposit_buffer(const Shape& s, unsigned long long photons, char* at, size_t bytes, uint32_t nlanes,
                    Deposits* D) {
    const size_t nbins = (s.ncell + kBinCells - 1) / kBinCells;
    if (nbins < kMinBins || nbins > kMaxBins || photons < min_photons(nbins)) return false;
    D->nbins = (uint32_t)nbins;
    D->nlanes = nlanes;
    D->nwaves = nlanes / 64;
    const size_t fixed = 2 * kTileChunks * 128 + align256(24 * (size_t)D->nwaves) +
                         align256(4 * (size_t)kLaneWords * nlanes);
    const size_t per_tile = 8 * (size_t)kTileDeposits + 4 * kTileChunks + 2 * (nbins + 1);
    if (bytes < fixed + 1024 + min_tiles(nbins) * per_tile) return false;
    D->ntiles = (uint32_t)std::min<size_t>((bytes - fixed - 1024) / per_tile, 1u << 20);
    D->item = (uint2*)at;
    at += 8 * (size_t)kTileDeposits * D->ntiles;
    D->used = (uint32_t*)at;
    at += 2 * kTileChunks * 128;
    D->waves = (unsigned long long*)at;
    at += align256(24 * (size_t)D->nwaves);
    D->lanes = (uint32_t*)at;
    at += align256(4 * (size_t)kLaneWords * nlanes);
    D->count = (uint32_t*)at;
    at += 4 * (size_t)kTileChunks * D->ntiles;
    D->start = (uint16_t*)at;
    return true;
}

// Rounds launched: 64 deposits a photon are more than the fields in use give
// (26 to 31).
int deposit_rounds(const Deposits& D, unsigned long long photons) {
    const unsigned long long room = (unsigned long long)D.ntiles * kTileDeposits;
    return (int)std::min<unsigned long long>(kMaxRounds, 1 + photons / (room / 64 + 1));
}

// One past the last deposit that the addition reads when `ntiles` tiles are in
// use: its groups of 64 tiles, with runs at every edge of a tile.
unsigned long long deposit_reach(uint32_t ntiles) {
    unsigned long long end = 0;
    for (uint32_t t = 0; t < (ntiles + 63) / 64 * 64; ++t) {
        const unsigned long long group = (unsigned long long)(t & ~63u) * kTileDeposits;
        auto run = [&](uint32_t first, uint32_t last) {
            const uint32_t len = last - first;
            end = std::max(end, group + Deposits::run_at(t & 63u, first, last) + (len ? len : 1u));
        };
        run(0, 0);
        if (t >= ntiles) continue;
        run(0, kTileDeposits);
        run(kTileDeposits - 1, kTileDeposits);
        run(kTileDeposits, kTileDeposits);
    }
    return end;
}

struct Launch {
    rt3d_options o;
    Shape s;
    int ngp;
    unsigned long long total;
    char* ws;
    char* spare;         // workspace behind the sections of layout_of
    size_t spare_bytes;
    uint32_t* flag;
    float* maj;
    float4* cells;
    float2* gas;
    uint32_t* layer;
    uint32_t* mask;
    TraceParams P;
    Setup setup;
};

rt3d_status prepare(const rt3d_grid* grid, int ngp, const uint64_t* photons, const float* albedo, double sza_deg,
                    double azimuth_deg, uint64_t seed, const rt3d_options* opt, const rt3d_tallies* out,
                    void* workspace, size_t workspace_bytes, void* stream, bool factored, Launch* L) {
    if (!grid_ok(grid)) return RT3D_EINVAL;
    resolve_options(grid, opt, &L->o);
    const rt3d_options& o = L->o;
    if (!shape_of(grid, &o, &L->s)) return RT3D_EINVAL;
    const Shape& s = L->s;
    if (!albedo || !photons) return RT3D_EINVAL;
    if (!out || !out->abs_dir || !out->abs_dif || !out->sfc_dir || !out->sfc_dif || !out->sfc_abs ||
        !out->toa_up || !out->ledger || !out->stats)
        return RT3D_EINVAL;
    if (!(sza_deg >= 0.0 && sza_deg < 90.0) || !std::isfinite(azimuth_deg)) return RT3D_EINVAL;
    if (!(o.diffuse_fraction >= 0.f && o.diffuse_fraction <= 1.f)) return RT3D_EINVAL;
    if (!(o.rr_threshold >= 0.f && o.rr_threshold <= 1.f)) return RT3D_EINVAL;
    if (o.grid_blocks < 0 || o.block_threads < 0 || o.max_walk < 0 || o.pool_photons < 0) return RT3D_EINVAL;
    // a refill hands out up to one id per lane of the wave from one grab, so
    // a grab must hold at least a wave's 64 ids
    if (o.pool_photons > 0 && o.pool_photons < 64) return RT3D_EINVAL;
    if (o.refill_lanes < 0 || o.refill_lanes > 64) return RT3D_EINVAL;
    if (o.tile_x < 0 || o.tile_y < 0 || (o.tile_x && s.nx % o.tile_x) || (o.tile_y && s.ny % o.tile_y))
        return RT3D_EINVAL;
    // the one size that each kernel takes (1024: the kernel's largest, fewer lanes)
    if (o.block_threads && o.block_threads != (factored ? 256 : 1024)) return RT3D_EINVAL;
    unsigned long long total = 0;
    for (int n = 0; n < ngp; ++n) {
        if (total + photons[n] < total) return RT3D_EINVAL;
        total += photons[n];
    }
    // the ledger holds photons * 2^31 in uint64
    if (total == 0 || total >= (1ull << 33)) return RT3D_EINVAL;
    if (o.photon_offset + total < o.photon_offset) return RT3D_EINVAL;
    const Layout lay = layout_of(s, ngp, factored);
    if (!workspace || workspace_bytes < lay.total || ((uintptr_t)workspace & 255)) return RT3D_EINVAL;

    L->ngp = ngp;
    L->total = total;
    L->ws = (char*)workspace;
    L->spare = L->ws + lay.total;
    L->spare_bytes = workspace_bytes - lay.total;
    L->flag = (uint32_t*)(L->ws + 128);
    L->maj = (float*)(L->ws + lay.maj);
    L->cells = (float4*)(L->ws + lay.cells);
    L->gas = factored ? (float2*)(L->ws + lay.gas) : nullptr;
    L->layer = factored ? (uint32_t*)(L->ws + lay.layer) : nullptr;
    L->mask = factored ? (uint32_t*)(L->ws + lay.mask) : nullptr;
    unsigned long long* pass_first = (unsigned long long*)(L->ws + lay.meta);
    unsigned long long* rem_first = pass_first + ngp + 1;
    unsigned long long* gp_col = rem_first + ngp + 1;

    Setup& b = L->setup;
    memset(&b, 0, sizeof b);
    for (int n = 0; n < ngp; ++n) b.photons[n] = photons[n];
    b.seed = seed;
    b.ncol = s.ncol;
    b.ngp = ngp;
    b.control = (unsigned long long*)L->ws;
    b.pass_first = pass_first;
    b.rem_first = rem_first;
    b.gp_col_offset = gp_col;

    TraceParams& P = L->P;
    memset(&P, 0, sizeof P);
    P.cells = L->cells;
    P.gas = L->gas;
    P.albedo = albedo;
    P.majorant = L->maj;
    P.cell_mask = (o.flags & RT3D_FLAG_CELL_MASK) ? L->mask : nullptr;
    P.mask_words = factored ? mask_words_of(s) : 0;
    schedule_of(s, ngp, photons, o, pass_first, rem_first, gp_col, &P.sched);
    P.abs_dir = (unsigned long long*)out->abs_dir;
    P.abs_dif = (unsigned long long*)out->abs_dif;
    P.sfc_dir = (unsigned long long*)out->sfc_dir;
    P.sfc_dif = (unsigned long long*)out->sfc_dif;
    P.sfc_abs = (unsigned long long*)out->sfc_abs;
    P.toa_up = (unsigned long long*)out->toa_up;
    P.ledger = (unsigned long long*)out->ledger;
    P.stats = (unsigned long long*)out->stats;
    P.queue = (unsigned long long*)L->ws;
    P.ngp = ngp;
    P.nmaj = (int)s.nmaj;
    P.nx = s.nx; P.ny = s.ny; P.nz = s.nz;
    P.bx = s.bx; P.by = s.by; P.bz = s.bz;
    P.mx = s.mx; P.my = s.my; P.mz = s.mz;
    P.div_bx = fast_div((uint32_t)s.bx);
    P.div_by = fast_div((uint32_t)s.by);
    P.dx = grid->dx; P.dy = grid->dy; P.dz = grid->dz;
    P.inv_dx = 1.0f / grid->dx; P.inv_dy = 1.0f / grid->dy; P.inv_dz = 1.0f / grid->dz;
    P.cx = (float)s.bx * grid->dx; P.cy = (float)s.by * grid->dy; P.cz = (float)s.bz * grid->dz;
    P.H = (float)s.nz * grid->dz;
    const double th = sza_deg * M_PI / 180.0, ph = azimuth_deg * M_PI / 180.0;
    P.sun_x = (float)(-sin(th) * sin(ph));
    P.sun_y = (float)(-sin(th) * cos(ph));
    P.sun_z = (float)(-cos(th));
    P.diffuse_fraction = o.diffuse_fraction;
    P.rr_below = (uint32_t)std::nearbyint((double)o.rr_threshold * 2147483648.0);
    P.max_iters = o.max_iters;
    P.pool = o.pool_photons > 0 ? (uint32_t)o.pool_photons : 256u;
    P.refill = o.refill_lanes > 0 ? (uint32_t)o.refill_lanes : 16u;
    P.merge = (o.flags & RT3D_FLAG_NO_MERGE) ? 0 : 1;
    P.sobol = (o.flags & RT3D_FLAG_SOBOL_ENTRY) ? 1 : 0;
    P.seed = seed;
    P.photons = total;
    P.photon_offset = o.photon_offset;
    P.ncol = s.ncol;
    return RT3D_OK;
}

rt3d_status run_setup(const Setup& b, hipStream_t st) {
    size_t most = 1;
    for (int q = 0; q < b.nclear; ++q) most = std::max(most, b.words[q]);
    hipLaunchKernelGGL(setup_kernel, dim3(grid_for(most)), dim3(256), 0, st, b);
    HIP_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status validated(const Launch& L, hipStream_t st) {
    HIP_TRY(hipGetLastError());
    uint32_t h = 0;
    HIP_TRY(hipMemcpyAsync(&h, L.flag, sizeof h, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    return h ? RT3D_EDOMAIN : RT3D_OK;
}

// The setup launch; with RT3D_FLAG_VALIDATE the control block is set up and
// `validate` run before anything is cleared.  merged: the maxima that the
// packing kernel merges (nmerged 32-bit words of a 256-byte aligned section).
template <typename Validate>
rt3d_status begin(Launch& L, const rt3d_tallies* out, uint32_t* merged, size_t nmerged, hipStream_t st,
                  Validate&& validate) {
    Setup& b = L.setup;
    if (L.o.flags & RT3D_FLAG_VALIDATE) {
        rt3d_status r = run_setup(b, st);
        if (r != RT3D_OK) return r;
        validate();
        if ((r = validated(L, st)) != RT3D_OK) return r;
        b.control = nullptr;
    }
    auto clear = [&](void* p, size_t words) {
        b.clear[b.nclear] = (unsigned long long*)p;
        b.words[b.nclear++] = words;
    };
    clear(merged, (nmerged + 1) / 2);
    if (!(L.o.flags & RT3D_FLAG_ACCUMULATE)) {
        clear(out->abs_dir, L.s.ncell);
        clear(out->abs_dif, L.s.ncell);
        clear(out->sfc_dir, L.s.ncol);
        clear(out->sfc_dif, L.s.ncol);
        clear(out->sfc_abs, L.s.ncol);
        clear(out->toa_up, L.s.ncol);
        clear(out->ledger, RT3D_LEDGER_N);
        clear(out->stats, RT3D_STATS_N);
    }
    return run_setup(b, st);
}

// Row maxima with bricks of bz levels into out, by the packing kernel where a
// brick's row is a power of two of at most 64 cells (then rows begin at
// multiples of bx in the cell index, and in the wave).
RowMax row_max(const Shape& s, int bz, uint32_t* out) {
    RowMax r;
    r.out = s.bx <= 64 && (s.bx & (s.bx - 1)) == 0 ? out : nullptr;
    r.bx = fast_div((uint32_t)s.bx);
    r.mx = fast_div((uint32_t)s.mx);
    r.ny = fast_div((uint32_t)s.ny);
    r.by = fast_div((uint32_t)s.by);
    r.bz = fast_div((uint32_t)bz);
    r.nmx = s.mx;
    r.nmy = s.my;
    return r;
}

// The row pass of the majorant build as a launch of its own.
rt3d_status merge_majorants(const Shape& s, const float* k_ext, uint32_t* majorant, hipStream_t st) {
    const size_t n = (size_t)s.mx * s.ny * s.nz;
    hipLaunchKernelGGL(majorant_kernel, dim3(grid_for(n, 256, 16384)), dim3(256), 0, st, k_ext, majorant, s.nx, s.ny,
                       s.nz, s.bx, s.by, s.bz);
    HIP_TRY(hipGetLastError());
    return RT3D_OK;
}

constexpr unsigned kWavePhotons = 16;  // photons a wave has at least, where there are few
constexpr size_t kStagedPerLane = 32;  // majorants that a lane of a smaller workgroup stages in LDS, unless told to
constexpr unsigned kGrabs = 2048;      // grabs of fewer than 64 photons in a launch

rt3d_status launch_trace(Launch& L, bool factored, hipStream_t st) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    int max_lds = 0;
    HIP_TRY(hipDeviceGetAttribute(&max_lds, hipDeviceAttributeMaxSharedMemoryPerBlock, dev));
    const size_t maj_bytes = L.s.nmaj * sizeof(float);
    const size_t own_lds = 8 * (C_N * kCntSlots + C_N);  // the kernel's static LDS
    const size_t lds_limit = L.o.lds_majorant > 0 ? (size_t)max_lds - own_lds : kLdsMajorantBytes;
    int ncu = 0;
    HIP_TRY(hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, dev));
    const int most = factored ? Shape_<true>::threads : Shape_<false>::threads;
    int threads = most;
    // Few photons: a wave per kWavePhotons of them, spread over the CUs in
    // smaller workgroups (a launch then lasts as long as its longest photon,
    // and an iteration is shorter the fewer lanes and waves share it), and
    // the work queue handed out in grabs that leave every wave some: a
    // quarter of a wave's share, 16 to 256.  32x32x64 cells, 2^14 photons:
    // 1325 us with 64 waves on 16 CUs (grabs of 256), 754 with 64 photons a
    // wave on all CUs, 716 with 16 (8: 733); 90x66x50 cells, 1.5e6 photons:
    // 3480 with grabs of 256, 3397 with 32, 3271 with 64.
    const unsigned long long few = (L.total + kWavePhotons - 1) / kWavePhotons;
    if (!L.o.grid_blocks && !L.o.block_threads)
        threads = (int)std::min<unsigned long long>(threads, 64 * ((few + ncu - 1) / ncu));
    // What few lanes stage takes longer than it saves: 16384 majorants for one
    // photon, 185 us staged by 64 lanes, 126 from the L2; 2048 majorants, 166 and
    // 160, with 2^14 photons 232 and 233.
    const bool use_lds = L.ngp == 1 && L.o.lds_majorant >= 0 && maj_bytes <= lds_limit &&
                         maj_bytes + own_lds <= (size_t)max_lds &&
                         (L.o.lds_majorant > 0 || threads == most || L.s.nmaj <= kStagedPerLane * (size_t)threads);
    const size_t lds = use_lds ? maj_bytes : 0;
    // crossings per loop iteration: a short walk keeps the lanes of a wave
    // in step (a long clear-sky walk of one lane would hold the others)
    L.P.max_walk = L.o.max_walk > 0 ? L.o.max_walk : (use_lds ? 3 : 2);
    auto pick = [&](auto tally) {
        constexpr int kTally = decltype(tally)::value;
        return factored ? (use_lds ? trace_kernel<true, true, kTally> : trace_kernel<false, true, kTally>)
                        : (use_lds ? trace_kernel<true, false, kTally> : trace_kernel<false, false, kTally>);
    };
    auto kernel = (L.o.flags & RT3D_FLAG_WAVE_AGGREGATE) ? pick(std::integral_constant<int, kAggregated>{})
                                                         : pick(std::integral_constant<int, kDirect>{});
    int per_cu = 0;
    HIP_TRY(hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, lds));
    if (per_cu < 1) per_cu = 1;
    unsigned blocks = L.o.grid_blocks ? (unsigned)L.o.grid_blocks : (unsigned)(ncu * per_cu);
    // never more lanes than photons need
    const unsigned long long per_block = L.o.grid_blocks || L.o.block_threads ? threads : (threads / 64) * kWavePhotons;
    const unsigned long long max_blocks = (L.total + per_block - 1) / per_block;
    if (blocks > max_blocks) blocks = (unsigned)max_blocks;
    if (blocks < 1) blocks = 1;
    if (L.o.pool_photons == 0) {
        const unsigned long long share = L.total / ((unsigned long long)blocks * (threads / 64));
        const unsigned long long least =
            std::min<unsigned long long>(64, std::max<unsigned long long>(16, std::max(share, L.total / kGrabs)));
        L.P.pool = (uint32_t)std::min<unsigned long long>(256, std::max<unsigned long long>(least, share / 64 * 16));
    }
    if (L.o.flags & RT3D_FLAG_TIME) {
        if (!g_t0) HIP_TRY(hipEventCreate(&g_t0));
        if (!g_t1) HIP_TRY(hipEventCreate(&g_t1));
        HIP_TRY(hipEventRecord(g_t0, st));
    }
    Deposits& D = L.P.dep;
    if (!factored && !(L.o.flags & RT3D_FLAG_WAVE_AGGREGATE) &&
        deposit_buffer(L.s, L.total, L.spare, L.spare_bytes, blocks * (unsigned)threads, &D)) {
        kernel = use_lds ? trace_kernel<true, false, kBinned> : trace_kernel<false, false, kBinned>;
        const int rounds = deposit_rounds(D, L.total);
        hipLaunchKernelGGL(fill_u32_kernel, dim3(4), dim3(256), 0, st, D.used, (size_t)2 * kTileChunks * 32, 0u);
        HIP_TRY(hipGetLastError());
        for (int r = 0; r < rounds; ++r) {
            L.P.round = r;
            L.P.last_round = r == rounds - 1;
            hipLaunchKernelGGL(kernel, dim3(blocks), dim3(threads), lds, st, L.P);
            HIP_TRY(hipGetLastError());
            hipLaunchKernelGGL(deposit_sort_kernel, dim3(std::min<unsigned>(D.ntiles, (unsigned)ncu)), dim3(1024), 0, st, D, r);
            HIP_TRY(hipGetLastError());
            hipLaunchKernelGGL(deposit_add_kernel, dim3((D.nbins + 7) / 8 * 8), dim3(1024), 0, st, D, r,
                               (uint32_t)L.s.ncell, L.P.abs_dir, L.P.abs_dif);
            HIP_TRY(hipGetLastError());
        }
    } else {
        hipLaunchKernelGGL(kernel, dim3(blocks), dim3(threads), lds, st, L.P);
        HIP_TRY(hipGetLastError());
    }
    if (L.o.flags & RT3D_FLAG_TIME) {
        HIP_TRY(hipEventRecord(g_t1, st));
        g_timed = true;
    }
    // The two entries that ledger_atm_kernel forms anew, at the end: another
    // call that accumulates into the same tallies may have run meanwhile.
    if (L.o.flags & RT3D_FLAG_ACCUMULATE) {
        hipLaunchKernelGGL(clear_atm_kernel, dim3(1), dim3(64), 0, st, L.P.ledger);
        HIP_TRY(hipGetLastError());
    }
    hipLaunchKernelGGL(ledger_atm_kernel, dim3(grid_for(L.s.ncell, 256, 2048)), dim3(256), 0, st, L.P.abs_dir,
                       L.P.abs_dif, L.s.ncell, L.P.ledger);
    HIP_TRY(hipGetLastError());
    return RT3D_OK;
}

// Scratch of rt3d_trace_noalloc: the workspace of rt3d_trace (control
// block, photon ranges, majorant grid, packed cell records) in a file-scope
// device array instead of a caller buffer.  Every device the library runs on
// holds its own copy for the life of the process.  In host code the array's
// name is not a device address; its address on each device comes from
// hipGetSymbolAddress (scratch_address) and only that address is used.
static __device__ __align__(256) unsigned char scratch[RT3D_NOALLOC_SCRATCH_BYTES];

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on the current device, looked up once per
// device.
rt3d_status scratch_address(void** out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kMaxDevices) {
        snprintf(g_err, sizeof g_err, "rt3d_trace_noalloc: device %d beyond the %d it keeps scratch for", dev,
                 kMaxDevices);
        return RT3D_EDEVICE;
    }
    std::lock_guard<std::mutex> lock(g_scratch_mu);
    if (!g_scratch_ptr[dev]) {
        void* p = nullptr;
        HIP_TRY(hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)));
        if (!p || ((uintptr_t)p & 255)) {
            snprintf(g_err, sizeof g_err, "rt3d_trace_noalloc: bad scratch address on device %d", dev);
            return RT3D_EDEVICE;
        }
        g_scratch_ptr[dev] = p;
    }
    *out = g_scratch_ptr[dev];
    return RT3D_OK;
}

}  // namespace

// ===========================================================================
// C ABI
// ===========================================================================
extern "C" {

int rt3d_abi_version(void) { return RT3D_ABI_VERSION; }

const char* rt3d_status_string(rt3d_status s) {
    switch (s) {
        case RT3D_OK: return "ok";
        case RT3D_EINVAL: return "invalid argument";
        case RT3D_EDOMAIN: return "field value out of range";
        case RT3D_EDEVICE: return "HIP device error";
        case RT3D_ETOOBIG: return "problem larger than the static scratch of rt3d_trace_noalloc";
    }
    return "unknown status";
}

const char* rt3d_last_device_error(void) { return g_err; }

void rt3d_default_options(rt3d_options* opt) {
    if (!opt) return;
    memset(opt, 0, sizeof *opt);
    opt->diffuse_fraction = 0.0f;
    opt->rr_threshold = 0.5f;
    opt->max_iters = 1u << 24;
}

size_t rt3d_workspace_size(const rt3d_grid* grid, const rt3d_options* opt) {
    rt3d_options o;
    if (!grid_ok(grid)) return 0;
    resolve_options(grid, opt, &o);
    Shape s;
    if (!shape_of(grid, &o, &s)) return 0;
    return layout_of(s, 1, false).total;
}

size_t rt3d_workspace_size_batched(const rt3d_grid* grid, int32_t n_gpoints, const rt3d_options* opt) {
    rt3d_options o;
    if (!grid_ok(grid) || n_gpoints < 1 || n_gpoints > kMaxGpoints) return 0;
    resolve_options(grid, opt, &o);
    Shape s;
    if (!shape_of(grid, &o, &s)) return 0;
    return layout_of(s, n_gpoints, true).total;
}

rt3d_status rt3d_deposit_plan(const rt3d_grid* grid, const rt3d_options* opt, uint64_t photons,
                              size_t workspace_bytes, uint32_t lanes, uint64_t* plan) {
    rt3d_options o;
    if (!grid_ok(grid) || !plan || lanes == 0 || lanes % 64) return RT3D_EINVAL;
    resolve_options(grid, opt, &o);
    Shape s;
    if (!shape_of(grid, &o, &s)) return RT3D_EINVAL;
    const size_t need = layout_of(s, 1, false).total;
    if (workspace_bytes < need) return RT3D_EINVAL;
    for (int i = 0; i < RT3D_DEPOSIT_N; ++i) plan[i] = 0;
    char* const base = (char*)(uintptr_t)256;
    Deposits D;
    if ((o.flags & RT3D_FLAG_WAVE_AGGREGATE) ||
        !deposit_buffer(s, photons, base + need, workspace_bytes - need, lanes, &D))
        return RT3D_OK;
    plan[RT3D_DEPOSIT_TILES] = D.ntiles;
    plan[RT3D_DEPOSIT_BINS] = D.nbins;
    plan[RT3D_DEPOSIT_ROUNDS] = (uint64_t)deposit_rounds(D, photons);
    plan[RT3D_DEPOSIT_END] = (uint64_t)((char*)(D.item + (size_t)D.ntiles * kTileDeposits) - base);
    plan[RT3D_DEPOSIT_READ_END] = (uint64_t)((char*)(D.item + deposit_reach(D.ntiles)) - base);
    plan[RT3D_DEPOSIT_USED] = (uint64_t)((char*)(D.start + (size_t)D.ntiles * (D.nbins + 1)) - base);
    return RT3D_OK;
}

rt3d_status rt3d_majorant_build(const rt3d_grid* grid, const float* k_ext, int32_t bx, int32_t by, int32_t bz,
                                float* majorant, void* stream) {
    rt3d_options o;
    rt3d_default_options(&o);
    o.brick_x = bx; o.brick_y = by; o.brick_z = bz;
    Shape s;
    if (!k_ext || !majorant || bx <= 0 || by <= 0 || bz <= 0 || !shape_of(grid, &o, &s)) return RT3D_EINVAL;
    hipStream_t st = (hipStream_t)stream;
    hipLaunchKernelGGL(fill_u32_kernel, dim3(grid_for(s.nmaj)), dim3(256), 0, st, (uint32_t*)majorant, s.nmaj, 0u);
    HIP_TRY(hipGetLastError());
    return merge_majorants(s, k_ext, (uint32_t*)majorant, st);
}

rt3d_status rt3d_trace(const rt3d_grid* grid, const rt3d_optical_props* props, const float* surface_albedo,
                       double sza_deg, double azimuth_deg, uint64_t photons, uint64_t seed,
                       const rt3d_options* opt, const rt3d_tallies* out, void* workspace, size_t workspace_bytes,
                       void* stream) {
    g_timed = false;
    if (!props || !props->k_ext || !props->k_ext_cloud || !props->ssa || !props->g) return RT3D_EINVAL;
    Launch L;
    rt3d_status st = prepare(grid, 1, &photons, surface_albedo, sza_deg, azimuth_deg, seed, opt, out, workspace,
                             workspace_bytes, stream, false, &L);
    if (st != RT3D_OK) return st;
    hipStream_t hs = (hipStream_t)stream;
    st = begin(L, out, (uint32_t*)L.maj, L.s.nmaj, hs, [&] {
        hipLaunchKernelGGL(validate_kernel, dim3(grid_for(L.s.ncell, 256, 4096)), dim3(256), 0, hs, props->k_ext,
                           props->k_ext_cloud, props->ssa, props->g, surface_albedo, L.s.ncell, L.s.ncol, L.flag);
    });
    if (st != RT3D_OK) return st;
    const RowMax rows = row_max(L.s, L.s.bz, (uint32_t*)L.maj);
    if (!rows.out && (st = merge_majorants(L.s, props->k_ext, (uint32_t*)L.maj, hs)) != RT3D_OK) return st;
    hipLaunchKernelGGL(pack_cells_kernel, dim3(grid_for(L.s.ncell, 256, 16384)), dim3(256), 0, hs, props->k_ext,
                       props->ssa, props->k_ext_cloud, props->g, L.cells, L.s.ncell, rows);
    HIP_TRY(hipGetLastError());
    return launch_trace(L, false, hs);
}

rt3d_status rt3d_trace_noalloc(const rt3d_grid* grid, const rt3d_optical_props* props, const float* surface_albedo,
                               double sza_deg, double azimuth_deg, uint64_t photons, uint64_t seed,
                               const rt3d_options* opt, const rt3d_tallies* out, void* stream) {
    g_timed = false;
    // timing would create HIP events on first use
    if (opt && (opt->flags & RT3D_FLAG_TIME)) return RT3D_EINVAL;
    const size_t need = rt3d_workspace_size(grid, opt);
    if (need == 0) return RT3D_EINVAL;
    if (need > RT3D_NOALLOC_SCRATCH_BYTES) {
        snprintf(g_err, sizeof g_err,
                 "rt3d_trace_noalloc: this grid needs %zu bytes of scratch, more than its %zu", need,
                 (size_t)RT3D_NOALLOC_SCRATCH_BYTES);
        return RT3D_ETOOBIG;
    }
    void* ws = nullptr;
    const rt3d_status st = scratch_address(&ws);
    if (st != RT3D_OK) return st;
    return rt3d_trace(grid, props, surface_albedo, sza_deg, azimuth_deg, photons, seed, opt, out, ws, need, stream);
}

rt3d_status rt3d_trace_batched(const rt3d_grid* grid, int32_t n_gpoints, const rt3d_batched_medium* medium,
                               const uint64_t* photons, const float* surface_albedo, double sza_deg,
                               double azimuth_deg, uint64_t seed, const rt3d_options* opt, const rt3d_tallies* out,
                               void* workspace, size_t workspace_bytes, void* stream) {
    g_timed = false;
    if (!medium || !medium->k_gas || !medium->ssa_gas || !medium->k_cloud || !medium->ssa_cloud ||
        !medium->g_cloud || !photons)
        return RT3D_EINVAL;
    if (n_gpoints < 1 || n_gpoints > kMaxGpoints) return RT3D_EINVAL;
    if (opt && opt->photon_offset != 0) return RT3D_EINVAL;
    Launch L;
    rt3d_status st = prepare(grid, n_gpoints, photons, surface_albedo, sza_deg, azimuth_deg, seed, opt, out,
                             workspace, workspace_bytes, stream, true, &L);
    if (st != RT3D_OK) return st;
    L.P.gp_diffuse = medium->diffuse_fraction;
    hipStream_t hs = (hipStream_t)stream;
    const size_t nlayer = (size_t)L.s.nz * L.s.my * L.s.mx;
    st = begin(L, out, L.layer, nlayer, hs, [&] {
        hipLaunchKernelGGL(validate_batched_kernel, dim3(grid_for(L.s.ncell, 256, 4096)), dim3(256), 0, hs,
                           medium->k_gas, medium->ssa_gas, (size_t)n_gpoints * L.s.nz, medium->k_cloud,
                           medium->ssa_cloud, medium->g_cloud, surface_albedo, L.s.ncell, L.s.ncol,
                           medium->diffuse_fraction, n_gpoints, L.flag);
    });
    if (st != RT3D_OK) return st;
    const size_t ngas = (size_t)n_gpoints * L.s.nz;
    const RowMax rows = row_max(L.s, 1, L.layer);
    hipLaunchKernelGGL(pack_cloud_kernel, dim3(grid_for(std::max(L.s.ncell, ngas), 256, 16384)), dim3(256), 0, hs,
                       medium->k_cloud, medium->ssa_cloud, medium->g_cloud, L.cells, L.s.ncell, rows, medium->k_gas,
                       medium->ssa_gas, L.gas, ngas);
    HIP_TRY(hipGetLastError());
    const size_t nmask = L.P.cell_mask ? L.s.nmaj * (size_t)L.P.mask_words : 0;
    if (nmask) hipLaunchKernelGGL(cell_mask_kernel, dim3(grid_for(nmask, 256, 16384)), dim3(256), 0, hs, medium->k_cloud, L.mask,
                       L.s.nx, L.s.ny, L.s.bx, L.s.by, L.s.bz, L.s.mx, L.s.my, L.P.mask_words, nmask);
    HIP_TRY(hipGetLastError());
    if (!rows.out) {
        const size_t nrow = (size_t)L.s.mx * L.s.ny * L.s.nz;
        hipLaunchKernelGGL(layer_max_kernel, dim3(grid_for(nrow, 256, 16384)), dim3(256), 0, hs, L.cells, L.layer,
                           L.s.nx, L.s.ny, L.s.nz, L.s.bx, L.s.by);
        HIP_TRY(hipGetLastError());
    }
    const size_t nm = L.s.nmaj * (size_t)n_gpoints;
    hipLaunchKernelGGL(gas_majorant_kernel, dim3(grid_for(nm, 256, 16384)), dim3(256), 0, hs, L.layer, L.gas,
                       L.maj, n_gpoints, L.s.nz, L.s.mx, L.s.my, L.s.bz);
    HIP_TRY(hipGetLastError());
    return launch_trace(L, true, hs);
}

rt3d_status rt3d_last_trace_ms(float* ms) {
    if (!ms || !g_timed) return RT3D_EINVAL;
    HIP_TRY(hipEventSynchronize(g_t1));
    HIP_TRY(hipEventElapsedTime(ms, g_t0, g_t1));
    return RT3D_OK;
}

rt3d_status rt3d_finalize(const rt3d_grid* grid, const rt3d_tallies* raw, uint64_t photons,
                          const double* layer_scale, double flux_scale, float* abs_dir, float* abs_dif,
                          float* sfc_dir, float* sfc_dif, float* sfc_abs, float* toa_up, void* stream) {
    if (!grid_ok(grid) || !raw || photons == 0 || !std::isfinite(flux_scale)) return RT3D_EINVAL;
    const size_t ncell = (size_t)grid->nx * grid->ny * grid->nz, ncol = (size_t)grid->nx * grid->ny;
    const double norm = (double)ncol / ((double)photons * 2147483648.0);
    hipStream_t st = (hipStream_t)stream;
    struct Item { const uint64_t* src; float* dst; size_t n; bool three; };
    const Item items[6] = {{raw->abs_dir, abs_dir, ncell, true}, {raw->abs_dif, abs_dif, ncell, true},
                           {raw->sfc_dir, sfc_dir, ncol, false}, {raw->sfc_dif, sfc_dif, ncol, false},
                           {raw->sfc_abs, sfc_abs, ncol, false}, {raw->toa_up, toa_up, ncol, false}};
    FinalizeArgs a;
    memset(&a, 0, sizeof a);
    a.plane = fast_div((uint32_t)ncol);
    int m = 0;
    for (const Item& it : items) {
        if (!it.dst) continue;
        if (!it.src) return RT3D_EINVAL;
        a.src[m] = (const unsigned long long*)it.src;
        a.dst[m] = it.dst;
        a.level[m] = it.three ? layer_scale : nullptr;
        a.norm[m] = it.three ? norm : norm * flux_scale;
        a.n[m] = (uint32_t)it.n;
        a.first[m + 1] = a.first[m] + (uint32_t)((it.n + kFinalizeItems - 1) / kFinalizeItems);
        ++m;
    }
    if (m == 0) return RT3D_OK;
    const uint32_t blocks = a.first[m];
    for (; m < 6; ++m) a.first[m + 1] = 0xffffffffu;
    hipLaunchKernelGGL(finalize_kernel, dim3(blocks), dim3(256), 0, st, a);
    HIP_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_philox4x32_10(const uint32_t* ctr, uint64_t seed, uint32_t* out, uint32_t n, void* stream) {
    if (!ctr || !out) return RT3D_EINVAL;
    if (n == 0) return RT3D_OK;
    hipLaunchKernelGGL(philox_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                       (const uint4*)ctr, (uint32_t)seed, (uint32_t)(seed >> 32), (uint4*)out, n);
    HIP_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_sobol_entry(uint64_t first_pass, uint32_t n, uint64_t column, uint64_t seed, uint32_t* out,
                             void* stream) {
    if (!out) return RT3D_EINVAL;
    if (n == 0) return RT3D_OK;
    hipLaunchKernelGGL(sobol_entry_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream,
                       (unsigned long long)first_pass, n, (unsigned long long)column, (uint32_t)seed,
                       (uint32_t)(seed >> 32), (uint2*)out);
    HIP_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_phase_sample(int32_t kind, const float* g, const float* xi, float* mu, uint32_t n, void* stream) {
    if ((kind != 0 && kind != 1) || !xi || !mu || (kind == 0 && !g)) return RT3D_EINVAL;
    if (n == 0) return RT3D_OK;
    hipLaunchKernelGGL(phase_sample_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream, (int)kind, g,
                       xi, mu, n);
    HIP_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_turn(const float* dir_in, const float* mu, const float* t, float* dir_out, uint32_t n, void* stream) {
    if (!dir_in || !mu || !t || !dir_out) return RT3D_EINVAL;
    if (n == 0) return RT3D_OK;
    hipLaunchKernelGGL(turn_kernel, dim3((n + 255) / 256), dim3(256), 0, (hipStream_t)stream, dir_in, mu, t, dir_out,
                       n);
    HIP_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_schedule_slots(const rt3d_grid* grid, int32_t n_gpoints, const uint64_t* photons,
                                const uint64_t* col_offset, const rt3d_options* opt, uint64_t first_slot, uint64_t n,
                                int32_t* gp_out, uint64_t* id_out, uint32_t* col_out) {
    if (!grid_ok(grid) || n_gpoints < 1 || n_gpoints > kMaxGpoints || !photons || !col_offset) return RT3D_EINVAL;
    rt3d_options o;
    resolve_options(grid, opt, &o);
    Shape s;
    if (!shape_of(grid, &o, &s)) return RT3D_EINVAL;
    if (o.tile_x < 0 || o.tile_y < 0 || (o.tile_x && s.nx % o.tile_x) || (o.tile_y && s.ny % o.tile_y))
        return RT3D_EINVAL;
    unsigned long long total = 0;
    for (int i = 0; i < n_gpoints; ++i) {
        if (col_offset[i] >= s.ncol || total + photons[i] < total) return RT3D_EINVAL;
        total += photons[i];
    }
    if (first_slot > total || n > total - first_slot || (n && (!gp_out || !id_out || !col_out))) return RT3D_EINVAL;
    unsigned long long pass_first[kMaxGpoints + 1], rem_first[kMaxGpoints + 1], offs[kMaxGpoints];
    schedule_tables(photons, n_gpoints, s.ncol, pass_first, rem_first);
    for (int i = 0; i < n_gpoints; ++i) offs[i] = col_offset[i];
    Schedule S;
    schedule_of(s, n_gpoints, photons, o, pass_first, rem_first, offs, &S);
    for (uint64_t i = 0; i < n; ++i) {
        const Slot sl = decode_slot(S, first_slot + i);
        gp_out[i] = sl.gp;
        id_out[i] = sl.id;
        col_out[i] = sl.col;
    }
    return RT3D_OK;
}

}  // extern "C"
