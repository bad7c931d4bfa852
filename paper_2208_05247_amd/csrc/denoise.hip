// denoise.hip -- BF16 MFMA kernels of the learned heating-rate denoiser:
// a 3D convolutional encoder-decoder trained on low/high-photon tally pairs
// produced by the tracer.  Declared in include/rt3d_denoise.h.
//
// Conventions: activations are BF16 channels-last [D][H][W][C] (C a multiple
// of 16, or 4 for the first layer's input); weights BF16 [Cout][KS^3][Cin]
// with FP32 master copies; all products accumulate in FP32 on the matrix
// cores.
//
// Convolution = implicit GEMM on v_mfma_f32_32x32x16_bf16: GEMM rows are 32
// consecutive voxels along x, columns 32 output channels, and the reduction
// runs over the KS^3 taps and 16-channel chunks.  A lane feeds the A operand
// with 8 channels of one voxel (zero outside the domain) and the B operand
// with 8 input channels of one output channel's weights.  The accumulator of
// lane l, element r holds row 8*(r/4) + 4*(l/32) + r%4, column l%32.
// 3x3x3 layers run from an input halo staged in LDS (conv3_kernel,
// conv3_c4_kernel); the 1x1x1 head uses conv_fwd_kernel,
// one wave per 32 x 32 output tile with its operands read directly, or in
// inference runs inside conv3_kernel after the last 3x3x3 layer.
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <string.h>

#include <algorithm>

#include "rt3d.h"
#include "rt3d_denoise.h"

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

thread_local char d_err[256] = "";

rt3d_status dfail(hipError_t e, const char* where) {
    snprintf(d_err, sizeof d_err, "%s: %s", where, hipGetErrorString(e));
    return RT3D_EDEVICE;
}

#define DN_TRY(expr)                                   \
    do {                                               \
        hipError_t e_ = (expr);                        \
        if (e_ != hipSuccess) return dfail(e_, #expr); \
    } while (0)

// 16 zero bytes in global memory (read in place of voxels outside the domain)
__device__ __align__(16) const uint32_t dn_zero16[4] = {0u, 0u, 0u, 0u};

__device__ __forceinline__ float bf2f(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

// FP32 -> BF16, round to nearest even (inputs are finite).
__device__ __forceinline__ uint16_t f2bf(float f) {
    uint32_t u = __float_as_uint(f);
    u += 0x7fffu + ((u >> 16) & 1u);
    return (uint16_t)(u >> 16);
}

__device__ __forceinline__ bf16x8 as_bf16x8(uint4 v) { return __builtin_bit_cast(bf16x8, v); }

unsigned blocks_for(size_t n, unsigned threads = 256, unsigned cap = 65535) {
    size_t g = (n + threads - 1) / threads;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (unsigned)g;
}

// ---------------------------------------------------------------------------
// Convolution forward (also the data gradient, with flipped weights)
// ---------------------------------------------------------------------------
struct ConvArgs {
    const uint16_t* x1;
    const uint16_t* x2;
    int c1, c2;            // input channels from x1 and x2 (multiples of 16)
    const uint16_t* w;     // [cout][taps][c1 + c2], or packed (pack_weights_kernel)
    const float* bias;     // [cout] or null
    uint16_t* y1;          // channels [0, o1)
    uint16_t* y2;          // channels [o1, cout)
    int o1;
    float* yf;             // optional FP32 copy [vox][yf_cols] of channels < yf_cols
    int D, H, W, cout, relu;
    int up1;               // x1 at half resolution, read nearest-upsampled
    // byte steps of the 3x3x3 weights: output channel, 8 inputs, tap, 16 inputs
    // (w_row, conv3_c4_pool_kernel: weights of a tap, 4 used)
    int w_row, w_half, w_tap, w_chunk;
    int yf_cols;
    // optional 1x1x1 head fused after a 32-output 3x3x3 convolution:
    // hy[vox][hcols] = FP32 channels [0, hcols) of conv1(bf16(y), hw) + hb
    const uint16_t* hw;    // [32][32] (head output, input channel)
    const float* hb;       // [32] or null
    float* hy;
    int hcols;
    // conv3_kernel: first output channel and number of channel slabs of this
    // launch; BF16 output only, in 16-byte pieces
    int co_base, slabs, store16;
};

template <int KS>
__global__ void __launch_bounds__(256) conv_fwd_kernel(const ConvArgs a) {
    const int lane = threadIdx.x & 63;
    const long wave = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int ntco = a.cout / 32;
    const int tiles_x = (a.W + 31) / 32;
    const long ntiles = (long)a.D * a.H * tiles_x * ntco;
    if (wave >= ntiles) return;
    const int cot = (int)(wave % ntco);
    long rest = wave / ntco;
    const int tx = (int)(rest % tiles_x);
    rest /= tiles_x;
    const int yy = (int)(rest % a.H);
    const int zz = (int)(rest / a.H);
    const int m = lane & 31, half = lane >> 5;
    const int xv = tx * 32 + m;
    const int co = cot * 32 + m;
    const int cin = a.c1 + a.c2;
    constexpr int taps = KS * KS * KS;
    f32x16 acc;
    for (int r = 0; r < 16; ++r) acc[r] = 0.0f;
    for (int t = 0; t < taps; ++t) {
        const int dz = t / (KS * KS) - KS / 2, dy = (t / KS) % KS - KS / 2, dx = t % KS - KS / 2;
        const int z = zz + dz, y = yy + dy, x = xv + dx;
        const bool inb = z >= 0 && z < a.D && y >= 0 && y < a.H && x >= 0 && x < a.W;
        const long vox = ((long)z * a.H + y) * a.W + x;
        const uint16_t* wrow = a.w + ((long)co * taps + t) * cin + 8 * half;
        for (int c0 = 0; c0 < cin; c0 += 16) {
            uint4 av = make_uint4(0u, 0u, 0u, 0u);
            if (inb) {
                const uint16_t* src = c0 < a.c1 ? a.x1 + vox * a.c1 + c0 : a.x2 + vox * a.c2 + (c0 - a.c1);
                av = *(const uint4*)(src + 8 * half);
            }
            const uint4 bv = *(const uint4*)(wrow + c0);
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(av), as_bf16x8(bv), acc, 0, 0, 0);
        }
    }
    const int n = cot * 32 + m;
    const float b = a.bias ? a.bias[n] : 0.0f;
    for (int r = 0; r < 16; ++r) {
        const int mm = 8 * (r >> 2) + 4 * half + (r & 3);
        const int x = tx * 32 + mm;
        if (x >= a.W) continue;
        float v = acc[r] + b;
        if (a.relu) v = fmaxf(v, 0.0f);
        const long vox = ((long)zz * a.H + yy) * a.W + x;
        if (a.yf && n < a.yf_cols) a.yf[vox * a.yf_cols + n] = v;
        if (n < a.o1) {
            if (a.y1) a.y1[vox * a.o1 + n] = f2bf(v);
        } else if (a.y2) {
            a.y2[vox * (a.cout - a.o1) + (n - a.o1)] = f2bf(v);
        }
    }
}

// Loads from memory that may be the 16-byte zero block.  The compiler loses the
// address space where a pointer is selected, and a flat load in its place also
// counts as a read of LDS: it waits for every load into LDS in flight.
typedef uint32_t uint2v __attribute__((ext_vector_type(2)));
typedef uint32_t uint4v __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint2 load_global8(const void* p) {
    return __builtin_bit_cast(uint2, *(const __attribute__((address_space(1))) uint2v*)p);
}
__device__ __forceinline__ uint4 load_global16(const void* p) {
    return __builtin_bit_cast(uint4, *(const __attribute__((address_space(1))) uint4v*)p);
}

constexpr int kTX = 32;           // voxels of an output row: the rows of an MFMA
constexpr int kHaloX = kTX + 2;
constexpr int kTY32 = 16;         // output rows of the first layer's workgroups
constexpr int kHaloY32 = kTY32 + 2;

constexpr int tile_slots_of(int pieces) { return (pieces + 63) / 64 * 64; }
constexpr int tile_slots(int halo_vox) { return tile_slots_of(halo_vox * 2); }

__device__ __forceinline__ void wait_loads() { __asm__ volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Stages the input halo of one 16-channel chunk, planes z0-1 .. z0+NZ-2 and
// rows y0-1 .. y0+HY-2 of columns x0-1 .. x0+kTX, into LDS as two 16-byte
// halves per voxel (slot 2 v + part).  The 32 inner voxels of a row are one
// load straight to LDS (global_load_lds_dwordx4: lane l of a wave writes its
// 16 bytes at the wave's LDS base + 16 l, checked on the device): the row's
// place is the same for the whole wave, so an address is a scalar plus the
// lane's own offset (decoded per 16-byte piece it was 28 vector instructions
// per load, and staging a fifth of the convolution's time).  The two outer
// voxels of each row go through registers, their loads in flight together with
// the others.  What lies outside the domain reads the 16-byte zero block.  The
// caller's barrier afterwards publishes the tile.
// ALL: every voxel through registers, read (load) while the previous chunk is
// computed; for tiles small enough.
template <int NZ, int HY, bool ALL>
struct Halo16 {
    static constexpr int kRows = NZ * HY;
    static constexpr int kOuter = (4 * kRows + 255) / 256;  // outer pieces a lane moves: i = 4 row + 2 side + half
    const uint16_t* base;
    int cs, hr, h, w;  // channels, 1 at half resolution, extent there
    uint4 outer[kOuter], inner[ALL ? (kRows + 3) / 4 : 1];

    // Before the barrier after which the tile may be overwritten.
    __device__ __forceinline__ void load_outer(const ConvArgs& a, int c0, int x0, int y0, int z0) {
        const bool from1 = c0 < a.c1;
        base = from1 ? a.x1 + c0 : a.x2 + (c0 - a.c1);
        cs = from1 ? a.c1 : a.c2;
        hr = from1 && a.up1 ? 1 : 0;
        h = a.H >> hr;
        w = a.W >> hr;
#pragma unroll
        for (int k = 0; k < kOuter; ++k) {
            const int i = (int)threadIdx.x + 256 * k, row = i >> 2, side = (i >> 1) & 1, part = i & 1;
            const int x = side ? x0 + kTX : x0 - 1, y = y0 + row % HY - 1, z = z0 + row / HY - 1;
            const bool in = row < kRows && x >= 0 && x < a.W && y >= 0 && y < a.H && z >= 0 && z < a.D;
            const uint16_t* src = base + (((long)(z >> hr) * h + (y >> hr)) * w + (x >> hr)) * cs + 8 * part;
            outer[k] = load_global16(in ? src : reinterpret_cast<const uint16_t*>(dn_zero16));
        }
    }
    // After it: the inner voxels, a wait for all loads, the outer voxels.
    __device__ __forceinline__ void stage(uint4* tile, const ConvArgs& a, int x0, int y0, int z0, int wave, int lane) {
        const uint16_t* const zero = reinterpret_cast<const uint16_t*>(dn_zero16);
        const int x = x0 + (lane >> 1);
        const uint32_t lane_at = (uint32_t)((x >> hr) * cs + 8 * (lane & 1));
        for (int row = wave; row < kRows; row += 4) {
            const int y = y0 + row % HY - 1, z = z0 + row / HY - 1;
            const bool in = y >= 0 && y < a.H && z >= 0 && z < a.D && x < a.W;
            const uint16_t* const at = base + ((long)(z >> hr) * h + (y >> hr)) * w * cs;
            __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)(in ? at + lane_at : zero),
                                             (__attribute__((address_space(3))) void*)(tile + (row * kHaloX + 1) * 2), 16,
                                             0, 0);
        }
        wait_loads();
        put_outer(tile);
    }
    __device__ __forceinline__ void load(const ConvArgs& a, int c0, int x0, int y0, int z0, int wave, int lane) {
        load_outer(a, c0, x0, y0, z0);
        const int x = x0 + (lane >> 1);
        const uint32_t lane_at = (uint32_t)((x >> hr) * cs + 8 * (lane & 1));
#pragma unroll
        for (int k = 0; k < (kRows + 3) / 4; ++k) {
            const int row = wave + 4 * k, y = y0 + row % HY - 1, z = z0 + row / HY - 1;
            const bool in = row < kRows && y >= 0 && y < a.H && z >= 0 && z < a.D && x < a.W;
            const uint16_t* const at = base + ((long)(z >> hr) * h + (y >> hr)) * w * cs;
            inner[k] = load_global16(in ? at + lane_at : reinterpret_cast<const uint16_t*>(dn_zero16));
        }
    }
    __device__ __forceinline__ void put(uint4* tile, int wave, int lane) {
#pragma unroll
        for (int k = 0; k < (kRows + 3) / 4; ++k)
            if (wave + 4 * k < kRows) tile[((wave + 4 * k) * kHaloX + 1) * 2 + lane] = inner[k];
        put_outer(tile);
    }
    __device__ __forceinline__ void put_outer(uint4* tile) {
#pragma unroll
        for (int k = 0; k < kOuter; ++k) {
            const int i = (int)threadIdx.x + 256 * k, row = i >> 2, side = (i >> 1) & 1, part = i & 1;
            if (row < kRows) tile[(row * kHaloX + (side ? kHaloX - 1 : 0)) * 2 + part] = outer[k];
        }
    }
};

// Weights through a buffer resource: a 32-bit lane offset and a scalar offset
// per load.  (As 64-bit addresses the 27 taps' take 54 vector registers.)
__device__ __forceinline__ __amdgpu_buffer_rsrc_t weight_resource(const uint16_t* w, long n) {
    const long bytes = 2 * n;
    return __builtin_amdgcn_make_buffer_rsrc((void*)w, 0, (int)(uint32_t)(bytes < 0xffffffffL ? bytes : 0xffffffffL),
                                             0x00027000);
}

__device__ __forceinline__ uint4 load_weights(__amdgpu_buffer_rsrc_t r, uint32_t lane, uint32_t uniform) {
    return __builtin_bit_cast(uint4, __builtin_amdgcn_raw_buffer_load_b128(r, (int)lane, (int)uniform, 0));
}

// Tiled 3x3x3 convolution.  A workgroup (4 waves) owns an output tile of KZ
// z-slices x kRows y-rows x 32 voxels and NCT x 32 output channels; a wave has R
// of the rows and 32 of the channels (NCT 2: two waves share the rows).  For
// each 16-channel input chunk the (KZ+2) x (kRows+2) x 34-voxel halo is loaded
// into LDS: straight, or where a lane's part of it fits beside its accumulators
// through registers, read while the previous chunk is computed.  Per z-slice
// of the kernel a wave keeps its 9 weight fragments in registers (the next
// slice's are loaded meanwhile), walks the R + 2 staged input rows its outputs
// need in each plane that slice reaches, 3 x-shifts each, and feeds every
// fragment it reads from LDS to all (up to 3) of its output rows that use it: at
// R = 4, KZ = 2 half an LDS read and an eighth of a weight load per MFMA.  All
// LDS offsets are constants from one lane address.  An output's products and
// their order are the same in every variant.
// What bounds it (192 -> 64 channels, 44x90x118 voxels, the launch alone, R = 4,
// KZ = 2): 425 us when every wave loaded both channel tiles' weights (8.8 TB/s
// from the L2; 291 with the loads left out), 354 in this split, 337 with
// cheaper staging, 332 with the halo's outer voxels in flight beside its inner
// ones, 290 with packed weights; about 50 of those are staging that the CU's
// other workgroup does not hide.
// The matrix cores themselves sustain 1.6-1.8 PFLOP/s on such operands.
// With a head (ConvArgs::hw, NCT 1) the
// 1x1x1 convolution follows in the epilogue and only its output is stored.
template <int NCT, int R, int KZ>
struct ConvTile {
    static constexpr int kRows = 4 / NCT * R, kHaloY = kRows + 2;
    static constexpr int kHaloVox = (KZ + 2) * kHaloY * kHaloX;
    // the fused head reuses the halo tile: 4 waves x KZ x R rows x 32 x 32 BF16
    // activations, then per wave one output row of 32 voxels x 2 FP32
    static constexpr int kHeadOut = 4 * KZ * R * 32 * 32 * 2;  // bytes
    static_assert(NCT > 1 || kHeadOut + 4 * 32 * 2 * 4 <= kHaloVox * 2 * 16, "head scratch exceeds the halo tile");
};

template <int NCT, int R, int KZ>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) conv3_kernel(const ConvArgs a) {
    using T = ConvTile<NCT, R, KZ>;
    constexpr bool kAhead = KZ * R <= 4;  // room for the next chunk's halo in registers
    __shared__ uint4 tile[tile_slots(T::kHaloVox)];  // 16 channels = two 16-byte halves per voxel
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int m = lane & 31, half = lane >> 5;
    const int nslab = a.slabs;
    const int tiles_x = (a.W + kTX - 1) / kTX, tiles_y = (a.H + T::kRows - 1) / T::kRows;
    long b = blockIdx.x;
    const int slab = (int)(b % nslab);
    b /= nslab;
    const int txi = (int)(b % tiles_x);
    b /= tiles_x;
    const int tyi = (int)(b % tiles_y);
    const int z0 = (int)(b / tiles_y) * KZ;
    const int x0 = txi * kTX, y0 = tyi * T::kRows;
    const int cin = a.c1 + a.c2;
    const int row0 = R * (wave / NCT);
    const int n0 = a.co_base + 32 * (slab * NCT + wave % NCT);  // this wave's 32 output channels
    f32x16 acc[KZ][R];
#pragma unroll
    for (int oz = 0; oz < KZ; ++oz)
#pragma unroll
        for (int o = 0; o < R; ++o)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[oz][o][e] = 0.0f;

    const auto wres = weight_resource(a.w + (long)n0 * 27 * cin, 32L * 27 * cin);
    const uint32_t lane_w = (uint32_t)(m * a.w_row + half * a.w_half);
    // the 9 weight fragments of (chunk c, z-slice dz); past the last chunk the
    // address is clamped and the fragments are never used
    auto load_b = [&](int c, int dz, uint4* out) {
        const int cc = min(c, cin - 16);
#pragma unroll
        for (int t = 0; t < 9; ++t) out[t] = load_weights(wres, lane_w, (uint32_t)((dz * 9 + t) * a.w_tap + (cc >> 4) * a.w_chunk));
    };
    const uint4* const at = tile + (row0 * kHaloX + m) * 2 + half;
    uint4 bnext[9];
    load_b(0, 0, bnext);
    Halo16<KZ + 2, T::kHaloY, kAhead> halo;
    if (kAhead) halo.load(a, 0, x0, y0, z0, wave, lane);
    for (int c0 = 0; c0 < cin; c0 += 16) {
        if (!kAhead) halo.load_outer(a, c0, x0, y0, z0);
        __syncthreads();  // the previous chunk's halo is no longer read
        if (kAhead) halo.put(tile, wave, lane);
        else halo.stage(tile, a, x0, y0, z0, wave, lane);
        __syncthreads();
        if (kAhead && c0 + 16 < cin) halo.load(a, c0 + 16, x0, y0, z0, wave, lane);
#pragma unroll
        for (int dz = 0; dz < 3; ++dz) {
            uint4 bv[9];
#pragma unroll
            for (int t = 0; t < 9; ++t) bv[t] = bnext[t];
            if (dz < 2) load_b(c0, dz + 1, bnext);
            else load_b(c0 + 16, 0, bnext);
            // the fragments of the next row are read before this row's MFMAs
            // run, so the LDS latency hides behind them
            auto row_frags = [&](int step, uint4* av) {
                const int oz = step / (R + 2), r = step % (R + 2);  // output plane oz reads staged plane oz + dz
#pragma unroll
                for (int dx = 0; dx < 3; ++dx) av[dx] = at[(((oz + dz) * T::kHaloY + r) * kHaloX + dx) * 2];
            };
            uint4 av[2][3];
            row_frags(0, av[0]);
#pragma unroll
            for (int step = 0; step < KZ * (R + 2); ++step) {
                const int oz = step / (R + 2), r = step % (R + 2);
                if (step + 1 < KZ * (R + 2)) row_frags(step + 1, av[(step + 1) & 1]);
                // keeps the scheduler from hoisting the reads of later rows
                // ahead of these MFMAs (it would spill at 2 waves/SIMD)
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int dx = 0; dx < 3; ++dx)
#pragma unroll
                    for (int o = 0; o < R; ++o) {
                        const int dy = r - o;  // output row o reads halo row o + dy
                        if (dy >= 0 && dy <= 2)
                            acc[oz][o] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                                as_bf16x8(av[step & 1][dx]), as_bf16x8(bv[dy * 3 + dx]), acc[oz][o], 0, 0, 0);
                    }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    const int n = m;
    const float bias = a.bias ? a.bias[n0 + m] : 0.0f;
    if (NCT == 1 && a.hw) {
        // Fused head.  Each wave writes its BF16 activations, 32 voxels x 32
        // channels per output row, to its own part of the (no longer needed)
        // halo tile, so that a lane can read the 8 consecutive channels of
        // one voxel that the A operand takes; the head then runs the same
        // two MFMAs per row as the 1x1x1 convolution kernel, in the same
        // order, so its output is bitwise that of the unfused pair.
        uint16_t* ht = reinterpret_cast<uint16_t*>(tile) + wave * (KZ * R * 32 * 32);
        __syncthreads();  // every wave is done reading the halo
#pragma unroll
        for (int oz = 0; oz < KZ; ++oz)
#pragma unroll
            for (int o = 0; o < R; ++o)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    float v = acc[oz][o][e] + bias;
                    if (a.relu) v = fmaxf(v, 0.0f);
                    ht[((oz * R + o) * 32 + 8 * (e >> 2) + 4 * half + (e & 3)) * 32 + n] = f2bf(v);
                }
        __syncthreads();
        uint4 hwv[2];
#pragma unroll
        for (int c = 0; c < 2; ++c) hwv[c] = *(const uint4*)(a.hw + m * 32 + 16 * c + 8 * half);
        const float hbias = a.hb ? a.hb[n] : 0.0f;
#pragma unroll
        for (int oz = 0; oz < KZ; ++oz) {
            const int zz = z0 + oz;
            if (zz >= a.D) continue;
#pragma unroll
            for (int o = 0; o < R; ++o) {
                const int y = y0 + row0 + o;
                if (y >= a.H) continue;
                f32x16 h;
#pragma unroll
                for (int e = 0; e < 16; ++e) h[e] = 0.0f;
#pragma unroll
                for (int c = 0; c < 2; ++c) {
                    const uint4 av = *(const uint4*)(ht + ((oz * R + o) * 32 + m) * 32 + 16 * c + 8 * half);
                    h = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(av), as_bf16x8(hwv[c]), h, 0, 0, 0);
                }
                if (a.hcols == 2) {
                    // the two used outputs of the row go through LDS (behind
                    // the activations' part of the tile), so that the row is
                    // stored as one 8-byte piece per voxel by 32 lanes instead
                    // of 16 stores of 4 bytes by 4 lanes each
                    float* hrow = reinterpret_cast<float*>(tile) + T::kHeadOut / 4 + wave * 64;
                    if (n < 2) {
#pragma unroll
                        for (int e = 0; e < 16; ++e) hrow[(8 * (e >> 2) + 4 * half + (e & 3)) * 2 + n] = h[e] + hbias;
                    }
                    // LDS instructions of one wave complete in order; the
                    // barrier keeps the compiler from moving the read across
                    // the writes
                    __builtin_amdgcn_wave_barrier();
                    if (lane < 32) {
                        const float2 v = *reinterpret_cast<const float2*>(hrow + 2 * lane);
                        if (x0 + lane < a.W)
                            *reinterpret_cast<float2*>(a.hy + (((long)zz * a.H + y) * a.W + x0 + lane) * 2) = v;
                    }
                    __builtin_amdgcn_wave_barrier();  // the next row's writes follow this read
                    continue;
                }
                if (n >= a.hcols) continue;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    const int x = x0 + 8 * (e >> 2) + 4 * half + (e & 3);
                    if (x >= a.W) continue;
                    a.hy[(((long)zz * a.H + y) * a.W + x) * a.hcols + n] = h[e] + hbias;
                }
            }
        }
        return;
    }
    if (a.store16) {
        // BF16 output through LDS: a lane holds one channel of 16 voxels, so
        // direct stores would be 2 bytes each; each wave instead writes one
        // output row (32 voxels x 32 channels, 2 KiB) to its own slice of the
        // halo tile and stores it as 16-byte pieces (8 channels of one voxel),
        // 2 per lane.  The 32 channels lie in y1 or in y2 (o1 is a multiple
        // of 32).
        static_assert(4 * 32 * 32 * 2 <= tile_slots(T::kHaloVox) * 16, "row scratch exceeds the halo tile");
        __syncthreads();  // every wave is done reading the halo
        uint16_t* row = reinterpret_cast<uint16_t*>(tile) + wave * (32 * 32);
        uint16_t* const dst = n0 < a.o1 ? a.y1 + n0 : a.y2 + (n0 - a.o1);
        const int stride = n0 < a.o1 ? a.o1 : a.cout - a.o1;
#pragma unroll
        for (int oz = 0; oz < KZ; ++oz) {
            const int zz = z0 + oz;
#pragma unroll
            for (int o = 0; o < R; ++o) {
                const int y = y0 + row0 + o;
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    float v = acc[oz][o][e] + bias;
                    if (a.relu) v = fmaxf(v, 0.0f);
                    row[(8 * (e >> 2) + 4 * half + (e & 3)) * 32 + m] = f2bf(v);
                }
                // LDS instructions of one wave complete in order; the barrier
                // keeps the compiler from moving the reads across the writes
                __builtin_amdgcn_wave_barrier();
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const int q = it * 64 + lane;  // voxel q / 4, channels 8 (q % 4) ..
                    const int x = x0 + (q >> 2);
                    const uint4 v = *reinterpret_cast<const uint4*>(row + (q >> 2) * 32 + 8 * (q & 3));
                    if (zz < a.D && y < a.H && x < a.W)
                        *reinterpret_cast<uint4*>(dst + (((long)zz * a.H + y) * a.W + x) * stride + 8 * (q & 3)) = v;
                }
                __builtin_amdgcn_wave_barrier();  // the next row's writes follow these reads
            }
        }
        return;
    }
#pragma unroll
    for (int oz = 0; oz < KZ; ++oz) {
        const int zz = z0 + oz;
        if (zz >= a.D) continue;
#pragma unroll
        for (int o = 0; o < R; ++o) {
            const int y = y0 + row0 + o;
            if (y >= a.H) continue;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int x = x0 + 8 * (e >> 2) + 4 * half + (e & 3);
                if (x >= a.W) continue;
                float v = acc[oz][o][e] + bias;
                if (a.relu) v = fmaxf(v, 0.0f);
                const long vox = ((long)zz * a.H + y) * a.W + x;
                const int c = n0 + m;
                if (a.yf && c < a.yf_cols) a.yf[vox * a.yf_cols + c] = v;
                if (c < a.o1) {
                    if (a.y1) a.y1[vox * a.o1 + c] = f2bf(v);
                } else if (a.y2) {
                    a.y2[vox * (a.cout - a.o1) + (c - a.o1)] = f2bf(v);
                }
            }
        }
    }
}

// First layer: 3x3x3 convolution of 4 input channels to 32 outputs, input
// [vox][4] (8 bytes per voxel), weights [32][27][4].  One MFMA K-chunk of 16
// holds the three x-taps of one (z, y) tap pair: A = channels 0-3 of voxels
// x-1, x, x+1 and four zeros, B = the matching 12 weights and four zeros, so
// a row takes 9 MFMAs instead of 27 of 16 mostly-zero channels.  Tile and
// reuse as in conv3_kernel (16 rows x 32 voxels, 4 rows per wave, every
// staged input row fed to all output rows that use it).
constexpr int kHaloVoxC4 = 3 * kHaloY32 * kHaloX;

__global__ void __launch_bounds__(256) conv3_c4_kernel(const ConvArgs a) {
    __shared__ uint2 tile[kHaloVoxC4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int m = lane & 31, half = lane >> 5;
    const int tiles_x = (a.W + kTX - 1) / kTX, tiles_y = (a.H + kTY32 - 1) / kTY32;
    long b = blockIdx.x;
    const int txi = (int)(b % tiles_x);
    b /= tiles_x;
    const int tyi = (int)(b % tiles_y);
    const int zz = (int)(b / tiles_y);
    const int x0 = txi * kTX, y0 = tyi * kTY32;
    const int row0 = 4 * wave;
    {
        // straight-line staging in batches of four loads per thread in
        // flight
        constexpr int kPer = (kHaloVoxC4 + 255) / 256, SB = 4;
#pragma unroll 1
        for (int j0 = 0; j0 < kPer; j0 += SB) {
            uint2 vv[SB];
#pragma unroll
            for (int j = 0; j < SB; ++j) {
                const int v = threadIdx.x + 256 * (j0 + j);
                const int hx = v % kHaloX, hy = (v / kHaloX) % kHaloY32, hz = v / (kHaloX * kHaloY32);
                const int x = x0 + hx - 1, y = y0 + hy - 1, z = zz + hz - 1;
                const bool in = x >= 0 && x < a.W && y >= 0 && y < a.H && z >= 0 && z < a.D;
                const int xc = min(max(x, 0), a.W - 1), yc = min(max(y, 0), a.H - 1), zc = min(max(z, 0), a.D - 1);
                // a voxel outside the domain reads zeros from dn_zero16: the
                // address is selected, so the load cannot sink into a branch
                // (which would wait for it before the next one is issued)
                vv[j] = load_global8(in ? a.x1 + (((long)zc * a.H + yc) * a.W + xc) * 4
                                        : reinterpret_cast<const uint16_t*>(dn_zero16));
            }
#pragma unroll
            for (int j = 0; j < SB; ++j) {
                const int v = threadIdx.x + 256 * (j0 + j);
                if (j0 + j < kPer && v < kHaloVoxC4) tile[v] = vv[j];
            }
        }
    }
    // B fragments of the 9 (z, y) tap pairs: lane half 0 holds taps dx = 0, 1,
    // half 1 tap dx = 2 and zeros
    uint4 bv[9];
    const uint16_t* wrow = a.w + (long)m * 27 * 4;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const uint2 lo = *(const uint2*)(wrow + (q * 3 + 2 * half) * 4);
        const uint2 hi = half ? make_uint2(0u, 0u) : *(const uint2*)(wrow + (q * 3 + 1) * 4);
        bv[q] = make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
    __syncthreads();
    f32x16 acc[4];
#pragma unroll
    for (int o = 0; o < 4; ++o)
#pragma unroll
        for (int e = 0; e < 16; ++e) acc[o][e] = 0.0f;
#pragma unroll
    for (int dz = 0; dz < 3; ++dz)
#pragma unroll
        for (int r = 0; r < 6; ++r) {
            const int i = (dz * kHaloY32 + row0 + r) * kHaloX + m;  // voxel x-1 of output column m
            const uint2 lo = tile[i + 2 * half];
            const uint2 hi = half ? make_uint2(0u, 0u) : tile[i + 1];
            const uint4 av = make_uint4(lo.x, lo.y, hi.x, hi.y);
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                const int dy = r - o;
                if (dy >= 0 && dy <= 2)
                    acc[o] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(av), as_bf16x8(bv[dz * 3 + dy]), acc[o],
                                                                     0, 0, 0);
            }
        }
    const int n = m;
    const float bias = a.bias ? a.bias[n] : 0.0f;
    if (!a.yf && a.y1 && a.o1 == 32) {
        // BF16 output through LDS: a lane holds one channel of 16 voxels, so
        // direct stores would be 2 bytes each; each wave instead writes one
        // output row (32 voxels x 32 channels, 2 KiB) to its own slice of the
        // halo tile (every wave is done reading it) and stores it back as
        // 16-byte pieces (8 channels of one voxel), 2 per lane
        static_assert(4 * 32 * 32 * 2 <= kHaloVoxC4 * 8, "row scratch exceeds the halo tile");
        __syncthreads();
        uint16_t* row = reinterpret_cast<uint16_t*>(tile) + wave * (32 * 32);
#pragma unroll
        for (int o = 0; o < 4; ++o) {
            const int y = y0 + row0 + o;
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                float v = acc[o][e] + bias;
                if (a.relu) v = fmaxf(v, 0.0f);
                row[(8 * (e >> 2) + 4 * half + (e & 3)) * 32 + n] = f2bf(v);
            }
            // LDS instructions of one wave complete in order: the reads below
            // see this row; the barrier only keeps the compiler from moving
            // them across the writes
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int it = 0; it < 2; ++it) {
                const int q = it * 64 + lane;  // 16-byte piece: voxel q / 4, channels 8 (q % 4) ..
                const int x = x0 + (q >> 2);
                const uint4 v = *reinterpret_cast<const uint4*>(row + (q >> 2) * 32 + 8 * (q & 3));
                if (y < a.H && x < a.W)
                    *reinterpret_cast<uint4*>(a.y1 + (((long)zz * a.H + y) * a.W + x) * 32 + 8 * (q & 3)) = v;
            }
            __builtin_amdgcn_wave_barrier();  // the next row's writes follow these reads
        }
        return;
    }
#pragma unroll
    for (int o = 0; o < 4; ++o) {
        const int y = y0 + row0 + o;
        if (y >= a.H) continue;
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const int x = x0 + 8 * (e >> 2) + 4 * half + (e & 3);
            if (x >= a.W) continue;
            float v = acc[o][e] + bias;
            if (a.relu) v = fmaxf(v, 0.0f);
            const long vox = ((long)zz * a.H + y) * a.W + x;
            if (a.yf && n < a.yf_cols) a.yf[vox * a.yf_cols + n] = v;
            if (a.y1) a.y1[vox * a.o1 + n] = f2bf(v);
        }
    }
}

// The first layer and the 2x2x2 average pooling of its output in one launch
// (inference).  A workgroup computes both output planes of one pooled plane
// from four staged input planes (the MFMAs of each output in
// conv3_c4_kernel's order), stores them as conv3_c4_kernel does, and pools
// each wave's pairs of output rows from LDS as they pass, adding in
// pool2_kernel's order (z, then y, then x, in FP32) with the sums of the
// first plane kept in registers: the full-resolution and the pooled output
// are bitwise those of the two separate launches, and the full-resolution
// output is not read back.  D, H, W even.
constexpr int kHaloVoxC4P = 4 * kHaloY32 * kHaloX;

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(3)))
conv3_c4_pool_kernel(const ConvArgs a, uint16_t* __restrict__ yp) {
    __shared__ uint2 tile[kHaloVoxC4P];
    __shared__ uint4 rows[4 * 2 * 32 * 32 * 2 / 16];  // per wave two output rows, 32 voxels x 32 BF16 channels
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int m = lane & 31, half = lane >> 5;
    const int tiles_x = (a.W + kTX - 1) / kTX, tiles_y = (a.H + kTY32 - 1) / kTY32;
    long b = blockIdx.x;
    const int txi = (int)(b % tiles_x);
    b /= tiles_x;
    const int tyi = (int)(b % tiles_y);
    const int zp = (int)(b / tiles_y);  // pooled plane: output planes 2 zp, 2 zp + 1
    const int z0 = 2 * zp;
    const int x0 = txi * kTX, y0 = tyi * kTY32;
    const int row0 = 4 * wave;
    {
        constexpr int kPer = (kHaloVoxC4P + 255) / 256, SB = 4;
#pragma unroll 1
        for (int j0 = 0; j0 < kPer; j0 += SB) {
            uint2 vv[SB];
#pragma unroll
            for (int j = 0; j < SB; ++j) {
                const int v = threadIdx.x + 256 * (j0 + j);
                const int hx = v % kHaloX, hy = (v / kHaloX) % kHaloY32, hz = v / (kHaloX * kHaloY32);
                const int x = x0 + hx - 1, y = y0 + hy - 1, z = z0 + hz - 1;
                const bool in = x >= 0 && x < a.W && y >= 0 && y < a.H && z >= 0 && z < a.D;
                const int xc = min(max(x, 0), a.W - 1), yc = min(max(y, 0), a.H - 1), zc = min(max(z, 0), a.D - 1);
                vv[j] = load_global8(in ? a.x1 + (((long)zc * a.H + yc) * a.W + xc) * 4
                                        : reinterpret_cast<const uint16_t*>(dn_zero16));
            }
#pragma unroll
            for (int j = 0; j < SB; ++j) {
                const int v = threadIdx.x + 256 * (j0 + j);
                if (j0 + j < kPer && v < kHaloVoxC4P) tile[v] = vv[j];
            }
        }
    }
    uint4 bv[9];
    const uint16_t* wrow = a.w + (long)m * 27 * a.w_row;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        const uint2 lo = *(const uint2*)(wrow + (q * 3 + 2 * half) * a.w_row);
        const uint2 hi = half ? make_uint2(0u, 0u) : *(const uint2*)(wrow + (q * 3 + 1) * a.w_row);
        bv[q] = make_uint4(lo.x, lo.y, hi.x, hi.y);
    }
    __syncthreads();
    const float bias = a.bias ? a.bias[m] : 0.0f;
    uint16_t* scr = reinterpret_cast<uint16_t*>(rows) + wave * (2 * 32 * 32);
    const int pv = lane >> 2, cg = lane & 3;  // this lane's pooled voxel of a pooled row and 8-channel group
    float s[2][8];
#pragma unroll
    for (int pr = 0; pr < 2; ++pr)
#pragma unroll
        for (int k = 0; k < 8; ++k) s[pr][k] = 0.0f;
#pragma unroll 1
    for (int oz = 0; oz < 2; ++oz) {
        f32x16 acc[4];
#pragma unroll
        for (int o = 0; o < 4; ++o)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[o][e] = 0.0f;
#pragma unroll
        for (int dz = 0; dz < 3; ++dz)
#pragma unroll
            for (int r = 0; r < 6; ++r) {
                const int i = ((oz + dz) * kHaloY32 + row0 + r) * kHaloX + m;  // voxel x-1 of output column m
                const uint2 lo = tile[i + 2 * half];
                const uint2 hi = half ? make_uint2(0u, 0u) : tile[i + 1];
                const uint4 av = make_uint4(lo.x, lo.y, hi.x, hi.y);
#pragma unroll
                for (int o = 0; o < 4; ++o) {
                    const int dy = r - o;
                    if (dy >= 0 && dy <= 2)
                        acc[o] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(av), as_bf16x8(bv[dz * 3 + dy]),
                                                                         acc[o], 0, 0, 0);
                }
            }
        const int zz = z0 + oz;
#pragma unroll
        for (int pr = 0; pr < 2; ++pr) {
#pragma unroll
            for (int oo = 0; oo < 2; ++oo)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    float v = acc[2 * pr + oo][e] + bias;
                    if (a.relu) v = fmaxf(v, 0.0f);
                    scr[(oo * 32 + 8 * (e >> 2) + 4 * half + (e & 3)) * 32 + m] = f2bf(v);
                }
            // LDS instructions of one wave complete in order; the barrier
            // keeps the compiler from moving the reads across the writes
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int oo = 0; oo < 2; ++oo) {
                const int y = y0 + row0 + 2 * pr + oo;
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const int q = it * 64 + lane;  // voxel q / 4, channels 8 (q % 4) ..
                    const int x = x0 + (q >> 2);
                    const uint4 v = *reinterpret_cast<const uint4*>(scr + (oo * 32 + (q >> 2)) * 32 + 8 * (q & 3));
                    if (y < a.H && x < a.W)
                        *reinterpret_cast<uint4*>(a.y1 + (((long)zz * a.H + y) * a.W + x) * 32 + 8 * (q & 3)) = v;
                }
            }
#pragma unroll
            for (int yy = 0; yy < 2; ++yy)
#pragma unroll
                for (int xx = 0; xx < 2; ++xx) {
                    const uint4 u = *reinterpret_cast<const uint4*>(scr + (yy * 32 + 2 * pv + xx) * 32 + 8 * cg);
                    const uint32_t wd[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        s[pr][2 * k] += bf2f((uint16_t)(wd[k] & 0xffffu));
                        s[pr][2 * k + 1] += bf2f((uint16_t)(wd[k] >> 16));
                    }
                }
            __builtin_amdgcn_wave_barrier();  // the next rows' writes follow these reads
        }
    }
    const int hh = a.H / 2, wh = a.W / 2;
#pragma unroll
    for (int pr = 0; pr < 2; ++pr) {
        const int yh = (y0 + row0) / 2 + pr, xh = x0 / 2 + pv;
        if (yh >= hh || xh >= wh) continue;
        uint32_t o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            o[k] = (uint32_t)f2bf(0.125f * s[pr][2 * k]) | ((uint32_t)f2bf(0.125f * s[pr][2 * k + 1]) << 16);
        *reinterpret_cast<uint4*>(yp + (((long)zp * hh + yh) * wh + xh) * 32 + 8 * cg) = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

// The same for a network with the fifth (direct-beam) input: the first
// layer reads 5 input channels stored as 8 per voxel (16 bytes, channels
// 5-7 zero), and one MFMA K-chunk of 16 holds the 15 values of the three
// x-taps of a (z, y) tap pair and one zero: lanes of half 0 take channels
// 0-4 of voxel x-1 and 0-2 of voxel x, lanes of half 1 channels 3-4 of voxel
// x, 0-4 of voxel x+1 and the zero (the B operand the matching weights, taken
// from the 16-channel weight rows w[co][t][16]).  Pooling as in
// conv3_c4_pool_kernel; bitwise equal to the unpacked first layer
// (conv3_kernel on 16-channel features) only up to the order of the
// products within a K-chunk, as the packed 4-channel layer is.
constexpr int kHaloVoxC5P = 4 * kHaloY32 * kHaloX;

__device__ __forceinline__ uint32_t hi_lo(uint32_t a, uint32_t b) { return (a >> 16) | (b << 16); }

__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2)))
conv3_c5_pool_kernel(const ConvArgs a, uint16_t* __restrict__ yp) {
    __shared__ uint4 tile[kHaloVoxC5P];
    __shared__ uint4 rows[4 * 2 * 32 * 32 * 2 / 16];  // per wave two output rows, 32 voxels x 32 BF16 channels
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const int m = lane & 31, half = lane >> 5;
    const int tiles_x = (a.W + kTX - 1) / kTX, tiles_y = (a.H + kTY32 - 1) / kTY32;
    long b = blockIdx.x;
    const int txi = (int)(b % tiles_x);
    b /= tiles_x;
    const int tyi = (int)(b % tiles_y);
    const int zp = (int)(b / tiles_y);  // pooled plane: output planes 2 zp, 2 zp + 1
    const int z0 = 2 * zp;
    const int x0 = txi * kTX, y0 = tyi * kTY32;
    const int row0 = 4 * wave;
    {
        constexpr int kPer = (kHaloVoxC5P + 255) / 256, SB = 4;
#pragma unroll 1
        for (int j0 = 0; j0 < kPer; j0 += SB) {
            uint4 vv[SB];
#pragma unroll
            for (int j = 0; j < SB; ++j) {
                const int v = threadIdx.x + 256 * (j0 + j);
                const int hx = v % kHaloX, hy = (v / kHaloX) % kHaloY32, hz = v / (kHaloX * kHaloY32);
                const int x = x0 + hx - 1, y = y0 + hy - 1, z = z0 + hz - 1;
                const bool in = x >= 0 && x < a.W && y >= 0 && y < a.H && z >= 0 && z < a.D;
                const int xc = min(max(x, 0), a.W - 1), yc = min(max(y, 0), a.H - 1), zc = min(max(z, 0), a.D - 1);
                vv[j] = load_global16(in ? a.x1 + (((long)zc * a.H + yc) * a.W + xc) * 8
                                         : reinterpret_cast<const uint16_t*>(dn_zero16));
            }
#pragma unroll
            for (int j = 0; j < SB; ++j) {
                const int v = threadIdx.x + 256 * (j0 + j);
                if (j0 + j < kPer && v < kHaloVoxC5P) tile[v] = vv[j];
            }
        }
    }
    // B fragments of the 9 (z, y) tap pairs from the 16-channel weight rows:
    // K 0-4 = tap dx 0 channels 0-4, K 5-9 = dx 1, K 10-14 = dx 2, K 15 = 0
    uint4 bv[9];
    const uint16_t* wrow = a.w + (long)m * 27 * 16;
#pragma unroll
    for (int q = 0; q < 9; ++q) {
        uint32_t wd[4];
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            uint32_t lohi[2];
#pragma unroll
            for (int e = 0; e < 2; ++e) {
                const int k = 8 * half + 2 * p + e;  // K index of this lane's element
                lohi[e] = k < 15 ? (uint32_t)wrow[(q * 3 + k / 5) * 16 + k % 5] : 0u;
            }
            wd[p] = lohi[0] | (lohi[1] << 16);
        }
        bv[q] = make_uint4(wd[0], wd[1], wd[2], wd[3]);
    }
    __syncthreads();
    const float bias = a.bias ? a.bias[m] : 0.0f;
    uint16_t* scr = reinterpret_cast<uint16_t*>(rows) + wave * (2 * 32 * 32);
    const int pv = lane >> 2, cg = lane & 3;
    float s[2][8];
#pragma unroll
    for (int pr = 0; pr < 2; ++pr)
#pragma unroll
        for (int k = 0; k < 8; ++k) s[pr][k] = 0.0f;
#pragma unroll 1
    for (int oz = 0; oz < 2; ++oz) {
        f32x16 acc[4];
#pragma unroll
        for (int o = 0; o < 4; ++o)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[o][e] = 0.0f;
#pragma unroll
        for (int dz = 0; dz < 3; ++dz)
#pragma unroll
            for (int r = 0; r < 6; ++r) {
                const int i = ((oz + dz) * kHaloY32 + row0 + r) * kHaloX + m;  // voxel x-1 of output column m
                // words of a voxel: (c0, c1), (c2, c3), (c4, 0), (0, 0)
                const uint4 u = tile[i + half], v = tile[i + half + 1];
                const uint4 av = half ? make_uint4(hi_lo(u.y, u.z), v.x, v.y, v.z)   // x: c3 c4; x+1: c0-c4, 0
                                      : make_uint4(u.x, u.y, u.z | (v.x << 16), hi_lo(v.x, v.y));  // x-1: c0-c4; x: c0-c2
#pragma unroll
                for (int o = 0; o < 4; ++o) {
                    const int dy = r - o;
                    if (dy >= 0 && dy <= 2)
                        acc[o] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(as_bf16x8(av), as_bf16x8(bv[dz * 3 + dy]),
                                                                         acc[o], 0, 0, 0);
                }
            }
        const int zz = z0 + oz;
#pragma unroll
        for (int pr = 0; pr < 2; ++pr) {
#pragma unroll
            for (int oo = 0; oo < 2; ++oo)
#pragma unroll
                for (int e = 0; e < 16; ++e) {
                    float v = acc[2 * pr + oo][e] + bias;
                    if (a.relu) v = fmaxf(v, 0.0f);
                    scr[(oo * 32 + 8 * (e >> 2) + 4 * half + (e & 3)) * 32 + m] = f2bf(v);
                }
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int oo = 0; oo < 2; ++oo) {
                const int y = y0 + row0 + 2 * pr + oo;
#pragma unroll
                for (int it = 0; it < 2; ++it) {
                    const int q = it * 64 + lane;
                    const int x = x0 + (q >> 2);
                    const uint4 v = *reinterpret_cast<const uint4*>(scr + (oo * 32 + (q >> 2)) * 32 + 8 * (q & 3));
                    if (y < a.H && x < a.W)
                        *reinterpret_cast<uint4*>(a.y1 + (((long)zz * a.H + y) * a.W + x) * 32 + 8 * (q & 3)) = v;
                }
            }
#pragma unroll
            for (int yy = 0; yy < 2; ++yy)
#pragma unroll
                for (int xx = 0; xx < 2; ++xx) {
                    const uint4 u = *reinterpret_cast<const uint4*>(scr + (yy * 32 + 2 * pv + xx) * 32 + 8 * cg);
                    const uint32_t wd[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        s[pr][2 * k] += bf2f((uint16_t)(wd[k] & 0xffffu));
                        s[pr][2 * k + 1] += bf2f((uint16_t)(wd[k] >> 16));
                    }
                }
            __builtin_amdgcn_wave_barrier();
        }
    }
    const int hh = a.H / 2, wh = a.W / 2;
#pragma unroll
    for (int pr = 0; pr < 2; ++pr) {
        const int yh = (y0 + row0) / 2 + pr, xh = x0 / 2 + pv;
        if (yh >= hh || xh >= wh) continue;
        uint32_t o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            o[k] = (uint32_t)f2bf(0.125f * s[pr][2 * k]) | ((uint32_t)f2bf(0.125f * s[pr][2 * k + 1]) << 16);
        *reinterpret_cast<uint4*>(yp + (((long)zp * hh + yh) * wh + xh) * 32 + 8 * cg) = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

// wt[ci][taps-1-t][co] = w[co][t][ci]  (data gradient = convolution of the
// output gradient with the flipped, transposed kernel)
__global__ void flip_weights_kernel(const uint16_t* __restrict__ w, uint16_t* __restrict__ wt, int cout, int cin,
                                    int taps) {
    const size_t n = (size_t)cout * cin * taps;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int ci = (int)(i % cin);
        const int t = (int)((i / cin) % taps);
        const int co = (int)(i / ((size_t)cin * taps));
        wt[((size_t)ci * taps + (taps - 1 - t)) * cout + co] = w[i];
    }
}

// The 3x3x3 weights in the order in which conv3_kernel's waves read them,
// [output channels / 32][input channels / 16][27 taps][64 lanes][8], so that a
// fragment is 1 KB in a row.  In [cout][27][cin] its lanes read 32 bytes each of
// 32 cache lines, whose other 96 bytes are fetched again for each of the next
// three chunks: 192 -> 64 channels on 44x90x118 voxels 348 us that way, 305
// packed; 96 -> 32 on 128x1024x1024 20.9 and 18.9 ms.  flip: the kernel of the data gradient, from
// w [cin][27][cout] (flip_weights_kernel's input).  A thread packs one lane's 8.
__global__ void pack_weights_kernel(const uint16_t* __restrict__ w, uint4* __restrict__ out, int cout, int cin,
                                    int flip) {
    const long n = (long)cout / 32 * (cin / 16) * 27 * 64;
    for (long i = blockIdx.x * (long)blockDim.x + threadIdx.x; i < n; i += (long)gridDim.x * blockDim.x) {
        const int lane = (int)(i & 63), t = (int)(i / 64 % 27);
        const long rest = i / (64 * 27);
        const int c = (int)(rest % (cin / 16)) * 16 + 8 * (lane >> 5);
        const long co = rest / (cin / 16) * 32 + (lane & 31);
        if (flip) {
            const uint16_t* src = w + ((long)c * 27 + 26 - t) * cout + co;
            uint32_t q[4];
#pragma unroll
            for (int k = 0; k < 4; ++k)
                q[k] = src[2 * k * 27L * cout] | (uint32_t)src[(2 * k + 1) * 27L * cout] << 16;
            out[i] = make_uint4(q[0], q[1], q[2], q[3]);
        } else {
            out[i] = *reinterpret_cast<const uint4*>(w + (co * 27 + t) * cin + c);
        }
    }
}

// ---------------------------------------------------------------------------
// Weight gradient: dw[co][t][ci] += sum_v dz[v][co] x[v + off(t)][ci], and the
// bias gradient db[co] += sum_v dz[v][co].
// GEMM rows = output channels, columns = input channels, reduction over 16
// voxels of one x-row per MFMA.
// ---------------------------------------------------------------------------
struct WgradArgs {
    const uint16_t* dz;
    int cout;
    const uint16_t* x1;
    const uint16_t* x2;
    int c1, c2;
    float* dw;
    float* db;       // or null
    float* partial;  // per-chunk partial dw [chunks][cout][taps][cin], or null: atomics into dw
    float* partial_b;  // per-chunk partial db [chunks][cout] (with partial)
    int D, H, W;
    int chunks;        // parts of the voxels, one workgroup each
};

// The 3x3x3 weight gradient.  Both MFMA operands run along voxels, which are
// the slow dimension of channels-last data: ds_read_b64_tr_b16 reads a block
// of 4 voxels x 16 channels from LDS and gives each of 16 lanes one channel's
// four voxels (lane l of the 16 addresses voxel l / 4, channels 4 (l % 4) ..;
// checked on the device), so a fragment is two such reads and a tap's shift is
// an address.
// A workgroup of 8 waves owns NCO x 32 output and NCI x 32 input channels of
// one chunk of the voxels.  Of the nine (z, y) rows of three taps each wave has
// one; the three taps of the ninth, and dz times ones (the bias gradient), go
// to waves 0-3, so that each SIMD has seven.  The chunk is a range of
// (tile of TY x 32 voxels, plane) units, planes innermost: the input planes
// z-1, z, z+1 of a tile stay in LDS, in a ring of four whose fourth plane
// (and the next plane of dz) is loaded while this one is computed.
// What bounds it: the latency of those loads, which the compiler's wait before
// the next LDS read exposes (a third of the time; held in registers instead
// they cost as much in addresses: 473 us against 430 in the first case below).
// Measured on 128^3 voxels: 96 -> 32 channels (NCI = 3) 0.43 ms, 810 TFLOP/s;
// 192 -> 64 at 64^3 (NCO = 2) 0.21 ms, 420 TFLOP/s; 16 -> 32 (NCI = 1, two
// workgroups a CU) 0.14 ms, 0.19 with one.  With 4 waves of seven taps they
// took 0.91, 0.24 and 0.22 ms: at 336 accumulators a lane, more than the 256
// accumulation registers, the compiler moved them around every MFMA.  With
// operands gathered from global memory by 2-byte loads, a wave per (32 x 32
// channels, tap), 3.8 and 1.0 ms (32 -> 64 channels on 64x60x52 voxels, whole
// call: 394 us, then 70, now 56).
template <int NCO, int NCI, int TY>
struct WgradTile {
    static constexpr int kRows = TY + 2;
    static constexpr int kSlab = tile_slots_of(kRows * kHaloX * 4);  // 16-byte pieces of one 32-channel plane
    static constexpr int kPlane = kSlab * NCI;
    static constexpr int kDzSlab = TY * kTX * 4;
    static constexpr int kDzPlane = kDzSlab * NCO;
    static constexpr int kPieces = 4 * kPlane + 2 * kDzPlane;
};

typedef short bf16x4_bits __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) bf16x4_bits lds_bf16x4;

// Four voxels of the lane's channel (two registers of two BF16).  at: the
// lane's byte address for the first voxel (see wgrad_lane_offset).
__device__ __forceinline__ uint2 read_voxels(const char* at) {
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_bf16x4*)at));
}

// One MFMA operand fragment: 16 voxels x 32 channels, voxel 8 (lane / 32) + k
// of channel lane % 32 in element k.
__device__ __forceinline__ bf16x8 read_fragment(const char* at) {
    const uint2 lo = read_voxels(at), hi = read_voxels(at + 4 * 64);
    return as_bf16x8(make_uint4(lo.x, lo.y, hi.x, hi.y));
}

// The fragments of the three taps of a row, from one window of 12 voxels: the
// second is the first moved on by one voxel (16 bits), the third by two (a
// register).  Three reads instead of six.
__device__ __forceinline__ void read_row(const char* at, bf16x8* out) {
    const uint2 a = read_voxels(at), b = read_voxels(at + 4 * 64), c = read_voxels(at + 8 * 64);
    out[0] = as_bf16x8(make_uint4(a.x, a.y, b.x, b.y));
    out[1] = as_bf16x8(make_uint4(__builtin_amdgcn_alignbit(a.y, a.x, 16), __builtin_amdgcn_alignbit(b.x, a.y, 16),
                                  __builtin_amdgcn_alignbit(b.y, b.x, 16), __builtin_amdgcn_alignbit(c.x, b.y, 16)));
    out[2] = as_bf16x8(make_uint4(a.y, b.x, b.y, c.x));
}

// Byte offset of the lane's part of a fragment in [voxel][32 channels] data.
__device__ __forceinline__ int wgrad_lane_offset(int lane) {
    return (8 * (lane >> 5) + ((lane & 15) >> 2)) * 64 + ((lane >> 4) & 1) * 32 + (lane & 3) * 8;
}

// One MFMA operand's element of the gradient by a 2-byte load, 0 outside.
__device__ __forceinline__ __bf16 element(bool in, const uint16_t* p) {
    const uint16_t v = in ? *p : (uint16_t)0;
    return __builtin_bit_cast(__bf16, v);
}

// A workgroup's sums of the kernel below, by 2-byte loads and without any
// product of a place outside the domain: see there.
template <int NCO, int NCI, int TY>
__device__ __forceinline__ void wgrad_by_elements(const WgradArgs& a, long u0, long u1, int ci0, int co0, int chunk) {
    int tid = (int)threadIdx.x;
    asm volatile("" : "+v"(tid));
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), m = tid & 31, half = (tid >> 5) & 1;
    const int cin = a.c1 + a.c2, tiles_x = (a.W + kTX - 1) / kTX;
#pragma unroll 1
    for (int k = wave; k < 27 * NCO * NCI + NCO; k += 8) {  // (tap, output and input channels), then the bias
        const bool ones = k >= 27 * NCO * NCI;
        const int t = ones ? 13 : k / (NCO * NCI), o = ones ? k - 27 * NCO * NCI : k / NCI % NCO, i = ones ? 0 : k % NCI;
        const int dz = t / 9 - 1, dy = t / 3 % 3 - 1, dx = t % 3 - 1;
        const int co = co0 + 32 * o + m, ci = ci0 + 32 * i + m;
        const bool first = ci < a.c1;
        const uint16_t* const xs = first ? a.x1 + ci : a.x2 + (ci - a.c1);
        const int xc = first ? a.c1 : a.c2;
        f32x16 acc;
        for (int e = 0; e < 16; ++e) acc[e] = 0.0f;
#pragma unroll 1
        for (long u = u0; u < u1; ++u) {
            const int zz = (int)(u % a.D), z = zz + dz;
            const long tile = u / a.D;
            const int x0 = (int)(tile % tiles_x) * kTX, y0 = (int)(tile / tiles_x) * TY;
#pragma unroll 1
            for (int r = 0; r < 2 * min(TY, a.H - y0); ++r) {
                const int yy = y0 + r / 2, y = yy + dy;
                const bool row = z >= 0 && z < a.D && y >= 0 && y < a.H && ci < cin;
                bf16x8 av, bv;
                for (int q = 0; q < 8; ++q) {
                    const int xx = x0 + 16 * (r & 1) + 8 * half + q, x = xx + dx;
                    av[q] = element(xx < a.W, a.dz + (((long)zz * a.H + yy) * a.W + xx) * a.cout + co);
                    bv[q] = ones ? (__bf16)1.0f
                                 : element(row && xx < a.W && x >= 0 && x < a.W, xs + (((long)z * a.H + y) * a.W + x) * xc);
                }
                acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc, 0, 0, 0);
            }
        }
        for (int e = 0; e < 16; ++e) {
            const int n = co0 + 32 * o + 8 * (e >> 2) + 4 * half + (e & 3);
            const long at = ((long)n * 27 + t) * cin + ci;
            if (ones) {
                if (!a.db || ci0 || m) continue;
                if (a.partial) a.partial_b[(long)chunk * a.cout + n] = acc[e];
                else atomicAdd(&a.db[n], acc[e]);
            } else if (ci < cin) {
                if (a.partial) a.partial[(long)chunk * a.cout * 27 * cin + at] = acc[e];
                else atomicAdd(&a.dw[at], acc[e]);
            }
        }
    }
}

template <int NCO, int NCI, int TY>
__global__ void __launch_bounds__(512)
    __attribute__((amdgpu_waves_per_eu(NCO * NCI == 1 ? 4 : 2, NCO * NCI == 1 ? 4 : 2)))
    conv3_wgrad_kernel(const WgradArgs a) {
    using T = WgradTile<NCO, NCI, TY>;
    extern __shared__ uint4 s_tile[];
    uint4* const s_x = s_tile;                  // ring of 4 planes
    uint4* const s_dz = s_tile + 4 * T::kPlane; // ring of 2 planes
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int cin = a.c1 + a.c2;
    const int nci = (cin + 32 * NCI - 1) / (32 * NCI), nco = a.cout / (32 * NCO);
    const int task = blockIdx.x % (nci * nco), chunk = blockIdx.x / (nci * nco);
    const int ci0 = (task % nci) * 32 * NCI, co0 = (task / nci) * 32 * NCO;
    const int tiles_x = (a.W + kTX - 1) / kTX, tiles_y = (a.H + TY - 1) / TY;
    const long units = (long)tiles_x * tiles_y * a.D;
    const long u0 = units * chunk / a.chunks, u1 = units * (chunk + 1) / a.chunks;

    f32x16 acc[4][NCO][NCI];
#pragma unroll
    for (int q = 0; q < 4; ++q)
#pragma unroll
        for (int o = 0; o < NCO; ++o)
#pragma unroll
            for (int i = 0; i < NCI; ++i)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[q][o][i][e] = 0.0f;

    // 16-byte pieces straight to LDS, 64 a wave instruction (16 voxels x 32
    // channels, of one row: a scalar address plus the lane's own offset); what
    // lies outside the domain or the channels reads zeros
    const uint16_t* const zero = reinterpret_cast<const uint16_t*>(dn_zero16);
    auto put = [&](uint4* to, const uint16_t* src) {
        __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void*)src,
                                         (__attribute__((address_space(3))) void*)to, 16, 0, 0);
    };
    const int part = lane & 3, vx = lane >> 2;  // of a piece within 16 voxels
    auto load_x = [&](int x0, int y0, int z) {
        uint4* const plane = s_x + (z & 3) * T::kPlane;
        for (int k = wave; k < NCI * T::kRows * 2; k += 8) {
            const int sl = k / (T::kRows * 2), hy = (k / 2) % T::kRows, j = k % 2;
            const int c0 = ci0 + 32 * sl, y = y0 + hy - 1, x = x0 + 16 * j + vx;
            const long row = ((long)z * a.H + y) * a.W + x0 + 16 * j;
            const bool in = z >= 0 && z < a.D && y >= 0 && y < a.H && x < a.W;
            const uint16_t* src;
            if (c0 + 32 <= a.c1) {
                src = a.x1 + row * a.c1 + c0 + (uint32_t)(vx * a.c1 + 8 * part);
            } else if (c0 >= a.c1 && c0 + 32 <= cin) {
                src = a.x2 + row * a.c2 + (c0 - a.c1) + (uint32_t)(vx * a.c2 + 8 * part);
            } else {  // the two inputs meet in this slab, or it is not full
                const int c = c0 + 8 * part;
                src = c < a.c1 ? a.x1 + (row + vx) * a.c1 + c : a.x2 + (row + vx) * a.c2 + (c - a.c1);
                if (c >= cin) src = zero;
            }
            put(plane + sl * T::kSlab + (hy * kHaloX + 1 + 16 * j) * 4, in ? src : zero);
        }
    };
    // the outer voxels of the rows, one piece a lane, through a register: read
    // ahead, written (put_edge) once the plane's place in the ring is free
    constexpr int kEdge = NCI * T::kRows * 8;
    static_assert(kEdge <= 512, "one outer piece a lane");
    const int e_sl = (int)threadIdx.x / (T::kRows * 8), e_hy = ((int)threadIdx.x / 8) % T::kRows;
    const int e_side = ((int)threadIdx.x / 4) & 1, e_c = ci0 + 32 * e_sl + 8 * part;
    auto get_edge = [&](int x0, int y0, int z) {
        const int x = e_side ? x0 + kTX : x0 - 1, y = y0 + e_hy - 1;
        const bool in = (int)threadIdx.x < kEdge && e_c < cin && x >= 0 && x < a.W && y >= 0 && y < a.H && z >= 0 && z < a.D;
        const long vox = ((long)z * a.H + y) * a.W + x;
        const uint16_t* src = e_c < a.c1 ? a.x1 + vox * a.c1 + e_c : a.x2 + vox * a.c2 + (e_c - a.c1);
        return load_global16(in ? src : zero);
    };
    auto put_edge = [&](int z, uint4 v) {
        if ((int)threadIdx.x < kEdge)
            s_x[(z & 3) * T::kPlane + e_sl * T::kSlab + (e_hy * kHaloX + (e_side ? kHaloX - 1 : 0)) * 4 + part] = v;
    };
    auto load_dz = [&](int x0, int y0, int z) {
        uint4* const plane = s_dz + (z & 1) * T::kDzPlane;
        for (int k = wave; k < NCO * TY * 2; k += 8) {
            const int sl = k / (TY * 2), hy = (k / 2) % TY, j = k % 2;
            const int y = y0 + hy, x = x0 + 16 * j + vx;
            const uint16_t* src = a.dz + (((long)z * a.H + y) * a.W + x0 + 16 * j) * a.cout + co0 + 32 * sl +
                                  (uint32_t)(vx * a.cout + 8 * part);
            put(plane + sl * T::kDzSlab + (hy * kTX + 16 * j) * 4, x < a.W && y < a.H ? src : zero);
        }
    };
    const char* const lane_x = (const char*)s_x + wgrad_lane_offset(lane);
    const char* const lane_dz = (const char*)s_dz + wgrad_lane_offset(lane);

    int x0 = 0, y0 = 0;
    uint4 edge = make_uint4(0u, 0u, 0u, 0u);
    bool ahead = false;  // the next plane's outer voxels are in `edge`
    for (long u = u0; u < u1; ++u) {
        const int z = (int)(u % a.D);
        if (u == u0 || z == 0) {  // a new tile: its first planes
            const long tile = u / a.D;
            x0 = (int)(tile % tiles_x) * kTX;
            y0 = (int)(tile / tiles_x) * TY;
            __syncthreads();
            uint4 first[3];  // (all of them in flight at once)
#pragma unroll
            for (int k = 0; k < 3; ++k) first[k] = get_edge(x0, y0, z + k - 1);
#pragma unroll
            for (int k = 0; k < 3; ++k) load_x(x0, y0, z + k - 1);
            load_dz(x0, y0, z);
#pragma unroll
            for (int k = 0; k < 3; ++k) put_edge(z + k - 1, first[k]);
        } else if (ahead) {
            put_edge(z + 1, edge);  // (no wave has read that place since the last barrier)
        }
        wait_loads();
        __syncthreads();  // this unit's planes are there, the last one's are no longer read
        ahead = z + 1 < a.D && u + 1 < u1;
        if (ahead) {
            load_x(x0, y0, z + 2);
            load_dz(x0, y0, z + 1);
            edge = get_edge(x0, y0, z + 2);
        }
        // the wave's row of taps, and its tap of the ninth row
        auto row_at = [&](int g) { return lane_x + ((z + g / 3 - 1) & 3) * (T::kPlane * 16) + g % 3 * (kHaloX * 64); };
        const char* at_row = row_at(wave);
        const char* at_tap = row_at(8) + (wave < 3 ? wave : 0) * 64;
        const char* at_dz = lane_dz + (z & 1) * T::kDzPlane * 16;
#pragma unroll 1
        for (int r = 0; r < TY; ++r) {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                bf16x8 av[NCO];
#pragma unroll
                for (int o = 0; o < NCO; ++o) av[o] = read_fragment(at_dz + o * (T::kDzSlab * 16) + h * (16 * 64));
#pragma unroll
                for (int i = 0; i < NCI; ++i) {
                    bf16x8 bv[3];
                    read_row(at_row + i * (T::kSlab * 16) + h * (16 * 64), bv);
#pragma unroll
                    for (int q = 0; q < 3; ++q)
#pragma unroll
                        for (int o = 0; o < NCO; ++o)
                            acc[q][o][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[o], bv[q], acc[q][o][i], 0, 0, 0);
                }
                if (wave < 4) {
#pragma unroll
                    for (int i = 0; i < NCI; ++i) {
                        bf16x8 bv = read_fragment(at_tap + i * (T::kSlab * 16) + h * (16 * 64));
                        if (wave == 3) {
#pragma unroll
                            for (int k = 0; k < 8; ++k) bv[k] = (__bf16)1.0f;
                        }
#pragma unroll
                        for (int o = 0; o < NCO; ++o)
                            acc[3][o][i] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av[o], bv, acc[3][o][i], 0, 0, 0);
                    }
                }
            }
            at_row += kHaloX * 64;
            at_tap += kHaloX * 64;
            at_dz += kTX * 64;
        }
    }
    if (a.W % kTX || a.H % TY) {
        // Where a tile is cut, dz is 0 past the domain, but taps reach back from
        // there to the last column and row of the input, and 0 times an
        // infinity or a NaN is no zero: sums that are not finite are formed
        // again without those products.  (Left out of the loop above they took
        // 3 to 14 % more time.)
        float nought = 0.0f;
#pragma unroll
        for (int q = 0; q < 4; ++q)
#pragma unroll
            for (int o = 0; o < NCO; ++o)
#pragma unroll
                for (int i = 0; i < NCI; ++i)
#pragma unroll
                    for (int e = 0; e < 16; ++e) nought = __builtin_fmaf(acc[q][o][i][e], 0.0f, nought);
        if (__builtin_expect(__syncthreads_or(nought != 0.0f), 0)) {
            wgrad_by_elements<NCO, NCI, TY>(a, u0, u1, ci0, co0, chunk);
            return;
        }
    }
    // element e of lane l: row (output channel) 8 (e / 4) + 4 (l / 32) + e % 4,
    // column (input channel) l % 32
    const int n = lane & 31, half = lane >> 5;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
        if (q == 3 && wave > 3) break;
        const int t = q < 3 ? 3 * wave + q : 24 + wave;
#pragma unroll
        for (int o = 0; o < NCO; ++o)
#pragma unroll
            for (int e = 0; e < 16; ++e) {
                const int co = co0 + 32 * o + 8 * (e >> 2) + 4 * half + (e & 3);
                if (t == 27) {  // every column holds the sum over the chunk's voxels
                    if (a.db && ci0 == 0 && n == 0) {
                        if (a.partial) a.partial_b[(long)chunk * a.cout + co] = acc[q][o][0][e];
                        else atomicAdd(&a.db[co], acc[q][o][0][e]);
                    }
                    continue;
                }
#pragma unroll
                for (int i = 0; i < NCI; ++i) {
                    const int ci = ci0 + 32 * i + n;
                    if (ci >= cin) continue;
                    const long at = ((long)co * 27 + t) * cin + ci;
                    if (a.partial) a.partial[(long)chunk * a.cout * 27 * cin + at] = acc[q][o][i][e];
                    else atomicAdd(&a.dw[at], acc[q][o][i][e]);
                }
            }
    }
}

// The weight gradient by 2-byte loads: one wave per 32 x 32 channels, tap and
// chunk of rows; the same chunk's bias gradient from the first input tile and
// tap.  For the 1x1x1 head, and for the 3x3x3 gradient of tensors that are not
// 16-byte aligned, which the kernel above cannot load.
template <int KS>
__global__ void __launch_bounds__(256) conv_wgrad_kernel(const WgradArgs a) {
    constexpr int taps = KS * KS * KS;
    const int lane = threadIdx.x & 63;
    const long wave = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int cin = a.c1 + a.c2;
    const int ntco = a.cout / 32, ntci = (cin + 31) / 32;
    const long nrows = (long)a.D * a.H;
    if (wave >= (long)ntco * ntci * taps * a.chunks) return;
    const int cot = (int)(wave % ntco);
    const int cit = (int)((wave / ntco) % ntci);
    const int t = (int)((wave / ((long)ntco * ntci)) % taps);
    const long chunk = wave / ((long)ntco * ntci * taps);
    const int dz = t / (KS * KS) - KS / 2, dy = (t / KS) % KS - KS / 2, dx = t % KS - KS / 2;
    const int m = lane & 31, half = lane >> 5;
    const int co = cot * 32 + m;
    const int ci = cit * 32 + m;
    const bool ci_ok = ci < cin;
    const uint16_t* xs = ci < a.c1 ? a.x1 : a.x2;
    const int xc = ci < a.c1 ? a.c1 : a.c2;
    const int xci = ci < a.c1 ? ci : ci - a.c1;
    f32x16 acc, accb;
    for (int r = 0; r < 16; ++r) acc[r] = accb[r] = 0.0f;
    bf16x8 ones;
    for (int k = 0; k < 8; ++k) ones[k] = (__bf16)1.0f;
    const long r0 = nrows * chunk / a.chunks, r1 = nrows * (chunk + 1) / a.chunks;
    for (long row = r0; row < r1; ++row) {
        const int z = (int)(row / a.H) + dz, y = (int)(row % a.H) + dy;
        const bool row_ok = KS == 1 || (z >= 0 && z < a.D && y >= 0 && y < a.H);
        const long vrow = row * a.W, srow = KS == 1 ? vrow : ((long)z * a.H + y) * a.W;
        for (int x0 = 0; x0 < a.W; x0 += 16) {
            bf16x8 av, bv;
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                const int x = x0 + 8 * half + i, sx = x + dx;
                const bool xin = x < a.W, sin = row_ok && xin && ci_ok && sx >= 0 && sx < a.W;
                const uint16_t g = xin ? a.dz[(vrow + x) * a.cout + co] : (uint16_t)0;
                const uint16_t v = sin ? xs[(srow + sx) * xc + xci] : (uint16_t)0;
                av[i] = __builtin_bit_cast(__bf16, g);
                bv[i] = __builtin_bit_cast(__bf16, v);
            }
            acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, bv, acc, 0, 0, 0);
            accb = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, ones, accb, 0, 0, 0);
        }
    }
    for (int r = 0; r < 16; ++r) {
        const int mm = cot * 32 + 8 * (r >> 2) + 4 * half + (r & 3);  // output channel (row)
        if (a.db && cit == 0 && t == 0 && m == 0) {
            if (a.partial) a.partial_b[chunk * a.cout + mm] = accb[r];
            else atomicAdd(&a.db[mm], accb[r]);
        }
        if (!ci_ok) continue;
        if (a.partial) a.partial[((chunk * a.cout + mm) * taps + t) * cin + ci] = acc[r];
        else atomicAdd(&a.dw[((long)mm * taps + t) * cin + ci], acc[r]);
    }
}

// dw[i] += sum over p = 0 .. chunks-1 of partial[p][i], and the same for db, in
// a fixed order: a workgroup has 4 width elements (one 16-byte load of `width`
// lanes), each group of `width` lanes adds its part of the chunks in order, and
// the parts are added in order.  What bounds it: the partials, read once.  One
// lane per element adding all chunks left few loads in flight: 1024 sums of
// 4096 chunks 107 us, now 16; the eight of a training pass at 128^3 196, now 132.
__global__ void __launch_bounds__(1024) sum_partials_kernel(const float* __restrict__ partial, float* __restrict__ dw,
                                                            size_t nw, const float* __restrict__ partial_b,
                                                            float* __restrict__ db, int nb, int chunks, int width) {
    __shared__ float4 s_part[1024];
    const int part = (int)threadIdx.x / width, parts = 1024 / width, at = (int)threadIdx.x % width;
    const size_t i = ((size_t)blockIdx.x * width + at) * 4;  // (nw and nb are multiples of 4)
    const bool bias = i >= nw, in = i < nw + nb;
    const float* src = bias ? partial_b + (in ? i - nw : 0) : partial + i;
    const size_t stride = bias ? (size_t)nb : nw;
    const int p1 = in ? (int)((long)chunks * (part + 1) / parts) : 0;
    float4 s = make_float4(0.0f, 0.0f, 0.0f, 0.0f);
    auto add = [&](const float4& v) {
        s.x += v.x;
        s.y += v.y;
        s.z += v.z;
        s.w += v.w;
    };
    int p = in ? (int)((long)chunks * part / parts) : 0;
    for (; p + 8 <= p1; p += 8) {
        float4 v[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) v[k] = *reinterpret_cast<const float4*>(src + (size_t)(p + k) * stride);
#pragma unroll
        for (int k = 0; k < 8; ++k) add(v[k]);
    }
    for (; p < p1; ++p) add(*reinterpret_cast<const float4*>(src + (size_t)p * stride));
    s_part[threadIdx.x] = s;
    __syncthreads();
    if (part || !in) return;
    for (int q = 1; q < parts; ++q) add(s_part[q * width + at]);
    float* out = bias ? db + (i - nw) : dw + i;  // (4-byte aligned)
    out[0] += s.x;
    out[1] += s.y;
    out[2] += s.z;
    out[3] += s.w;
}

// ---------------------------------------------------------------------------
// Elementwise and resampling kernels (BF16 storage, FP32 arithmetic)
// ---------------------------------------------------------------------------
// Most of these kernels come in two forms: 8 elements (16 bytes) per lane where
// the tensors are 16-byte aligned and the length or channel count is a multiple
// of 8, one element per lane elsewhere.  One element per lane moves 2 bytes per
// load and spends 30 to 60 instructions on its indexes: 128^3 x 32 channels
// ran at 1.0-2.4 TB/s (ReLU derivative 167 us, upsampling 384, pooling adjoint
// 200 and the sum after it 107); here 57, 45, and 89 for the pooling adjoint with
// the sum and the ReLU derivative in it.
struct Eight {
    float v[8];
};

__device__ __forceinline__ Eight load8(const uint16_t* p) {
    const uint4 u = *reinterpret_cast<const uint4*>(p);
    const uint32_t w[4] = {u.x, u.y, u.z, u.w};
    Eight e;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        e.v[2 * k] = bf2f((uint16_t)(w[k] & 0xffffu));
        e.v[2 * k + 1] = bf2f((uint16_t)(w[k] >> 16));
    }
    return e;
}

__device__ __forceinline__ void store8(uint16_t* p, const Eight& e) {
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) w[k] = (uint32_t)f2bf(e.v[2 * k]) | ((uint32_t)f2bf(e.v[2 * k + 1]) << 16);
    *reinterpret_cast<uint4*>(p) = make_uint4(w[0], w[1], w[2], w[3]);
}

// dy where the activation y is positive, else 0 (bits of two BF16)
__device__ __forceinline__ uint32_t relu_mask2(uint32_t dy, uint32_t y) {
    const uint32_t lo = bf2f((uint16_t)(y & 0xffffu)) > 0.0f ? dy & 0xffffu : 0u;
    const uint32_t hi = bf2f((uint16_t)(y >> 16)) > 0.0f ? dy & 0xffff0000u : 0u;
    return lo | hi;
}

__device__ __forceinline__ uint4 relu_mask8(uint4 dy, uint4 y) {
    return make_uint4(relu_mask2(dy.x, y.x), relu_mask2(dy.y, y.y), relu_mask2(dy.z, y.z), relu_mask2(dy.w, y.w));
}

__global__ void relu_bwd8_kernel(const uint4* __restrict__ dy, const uint4* __restrict__ y, uint4* __restrict__ dz,
                                 size_t n8) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n8; i += (size_t)gridDim.x * blockDim.x)
        dz[i] = relu_mask8(dy[i], y[i]);
}

__global__ void relu_bwd_kernel(const uint16_t* __restrict__ dy, const uint16_t* __restrict__ y,
                                uint16_t* __restrict__ dz, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        dz[i] = bf2f(y[i]) > 0.0f ? dy[i] : (uint16_t)0;
}

__global__ void add_kernel(const uint16_t* __restrict__ a, const uint16_t* __restrict__ b, uint16_t* __restrict__ out,
                           size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        out[i] = f2bf(bf2f(a[i]) + bf2f(b[i]));
}

__global__ void add8_kernel(const uint16_t* __restrict__ a, const uint16_t* __restrict__ b, uint16_t* __restrict__ out,
                            size_t n8) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n8; i += (size_t)gridDim.x * blockDim.x) {
        Eight x = load8(a + 8 * i);
        const Eight y = load8(b + 8 * i);
#pragma unroll
        for (int k = 0; k < 8; ++k) x.v[k] += y.v[k];
        store8(out + 8 * i, x);
    }
}

// 2x2x2 average pooling: out [D/2][H/2][W/2][C]
// One thread per output voxel and 8-channel group: eight 16-byte loads, one
// 16-byte store; every channel sums its 8 inputs in the same order.
__global__ void pool2_kernel(const uint16_t* __restrict__ x, uint16_t* __restrict__ y, int D, int H, int W, int C) {
    const int d = D / 2, h = H / 2, w = W / 2, cg = C / 8;
    const size_t n = (size_t)d * h * w * cg;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int c8 = (int)(i % cg);
        size_t v = i / cg;
        const int xo = (int)(v % w), yo = (int)((v / w) % h), zo = (int)(v / ((size_t)w * h));
        float s[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) s[k] = 0.0f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const int z = 2 * zo + (q >> 2), yy = 2 * yo + ((q >> 1) & 1), xx = 2 * xo + (q & 1);
            const uint4 u = *(const uint4*)(x + (((size_t)z * H + yy) * W + xx) * C + 8 * c8);
            const uint32_t wd[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                s[2 * k] += bf2f((uint16_t)(wd[k] & 0xffffu));
                s[2 * k + 1] += bf2f((uint16_t)(wd[k] >> 16));
            }
        }
        uint32_t o[4];
#pragma unroll
        for (int k = 0; k < 4; ++k)
            o[k] = (uint32_t)f2bf(0.125f * s[2 * k]) | ((uint32_t)f2bf(0.125f * s[2 * k + 1]) << 16);
        *(uint4*)(y + v * C + 8 * c8) = make_uint4(o[0], o[1], o[2], o[3]);
    }
}

__global__ void pool2_bwd_kernel(const uint16_t* __restrict__ dy, uint16_t* __restrict__ dx, int D, int H, int W,
                                 int C) {
    const size_t n = (size_t)D * H * W * C;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % C);
        const size_t v = i / C;
        const int x = (int)(v % W), y = (int)((v / W) % H), z = (int)(v / ((size_t)W * H));
        dx[i] = f2bf(0.125f * bf2f(dy[((((size_t)(z / 2)) * (H / 2) + y / 2) * (W / 2) + x / 2) * C + c]));
    }
}

// The adjoint of pooling by 8-channel groups, one lane per pooled voxel and
// group: one load, eight stores.  With `de` (may be the output) the gradient
// that reaches the pooled layer's input another way is added and the ReLU
// derivative of that layer taken through its output y: bitwise
// pool2_bwd_kernel, add_kernel and relu_bwd_kernel in turn (each sum rounded
// to BF16).
__global__ void pool2_bwd8_kernel(const uint16_t* __restrict__ dy, const uint16_t* de, const uint16_t* __restrict__ y,
                                  uint16_t* dx, int D, int H, int W, int C) {
    const uint32_t cg = C / 8, w = W / 2, h = H / 2;
    const size_t n = (size_t)(D / 2) * h * w * cg;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        size_t v;
        uint32_t c8, xo, yo;
        if (n >> 32) {
            c8 = (uint32_t)(i % cg);
            v = i / cg;
            xo = (uint32_t)(v % w);
            v /= w;
            yo = (uint32_t)(v % h);
            v /= h;
        } else {  // 32-bit divisions
            uint32_t q = (uint32_t)i / cg;
            c8 = (uint32_t)i - q * cg;
            xo = q % w;
            q /= w;
            yo = q % h;
            v = q / h;
        }
        Eight g = load8(dy + 8 * i);
#pragma unroll
        for (int k = 0; k < 8; ++k) g.v[k] = bf2f(f2bf(0.125f * g.v[k]));
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const size_t at = (((2 * v + (q >> 2)) * H + 2 * yo + ((q >> 1) & 1)) * W + 2 * xo + (q & 1)) * C + 8 * c8;
            Eight o = g;
            if (de) {
                const Eight e = load8(de + at);
#pragma unroll
                for (int k = 0; k < 8; ++k) o.v[k] = e.v[k] + g.v[k];
            }
            uint32_t wd[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) wd[k] = (uint32_t)f2bf(o.v[2 * k]) | ((uint32_t)f2bf(o.v[2 * k + 1]) << 16);
            uint4 r = make_uint4(wd[0], wd[1], wd[2], wd[3]);
            if (y) r = relu_mask8(r, *reinterpret_cast<const uint4*>(y + at));
            *reinterpret_cast<uint4*>(dx + at) = r;
        }
    }
}

// nearest-neighbour 2x upsampling: out [2D][2H][2W][C]
// by 8-channel groups, one lane per coarse voxel and group: one load, eight
// stores
__global__ void up2_8_kernel(const uint16_t* __restrict__ x, uint16_t* __restrict__ y, int D, int H, int W, int C) {
    const uint32_t cg = C / 8;
    const size_t n = (size_t)D * H * W * cg;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        size_t v = n >> 32 ? i / cg : (uint32_t)i / cg;
        const uint32_t c8 = (uint32_t)(i - v * cg);
        size_t r = n >> 32 ? v / W : (uint32_t)v / (uint32_t)W;
        const uint32_t xo = (uint32_t)(v - r * W);
        const size_t z = n >> 32 ? r / H : (uint32_t)r / (uint32_t)H;
        const uint32_t yo = (uint32_t)(r - z * H);
        const uint4 u = *reinterpret_cast<const uint4*>(x + 8 * i);
#pragma unroll
        for (int q = 0; q < 8; ++q)
            *reinterpret_cast<uint4*>(y + (((2 * z + (q >> 2)) * (2 * (size_t)H) + 2 * yo + ((q >> 1) & 1)) * (2 * (size_t)W) +
                                           2 * xo + (q & 1)) * C + 8 * c8) = u;
    }
}

// The adjoint of upsampling by 8-channel groups; with y the ReLU derivative
// through the upsampled layer's output y follows: bitwise up2_bwd_kernel and
// relu_bwd_kernel in turn.
__global__ void up2_bwd8_kernel(const uint16_t* __restrict__ dy, const uint16_t* __restrict__ act,
                                uint16_t* __restrict__ dx, int D, int H, int W, int C) {
    const uint32_t cg = C / 8;
    const size_t n = (size_t)D * H * W * cg;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        size_t v = n >> 32 ? i / cg : (uint32_t)i / cg;
        const uint32_t c8 = (uint32_t)(i - v * cg);
        size_t r = n >> 32 ? v / W : (uint32_t)v / (uint32_t)W;
        const uint32_t xo = (uint32_t)(v - r * W);
        const size_t z = n >> 32 ? r / H : (uint32_t)r / (uint32_t)H;
        const uint32_t yo = (uint32_t)(r - z * H);
        Eight s;
#pragma unroll
        for (int k = 0; k < 8; ++k) s.v[k] = 0.0f;
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            const Eight e = load8(dy + (((2 * z + (q >> 2)) * (2 * (size_t)H) + 2 * yo + ((q >> 1) & 1)) * (2 * (size_t)W) +
                                        2 * xo + (q & 1)) * C + 8 * c8);
#pragma unroll
            for (int k = 0; k < 8; ++k) s.v[k] += e.v[k];
        }
        uint32_t wd[4];
#pragma unroll
        for (int k = 0; k < 4; ++k) wd[k] = (uint32_t)f2bf(s.v[2 * k]) | ((uint32_t)f2bf(s.v[2 * k + 1]) << 16);
        uint4 o = make_uint4(wd[0], wd[1], wd[2], wd[3]);
        if (act) o = relu_mask8(o, *reinterpret_cast<const uint4*>(act + 8 * i));
        *reinterpret_cast<uint4*>(dx + 8 * i) = o;
    }
}

// one element per lane
__global__ void up2_kernel(const uint16_t* __restrict__ x, uint16_t* __restrict__ y, int D, int H, int W, int C) {
    const size_t n = (size_t)8 * D * H * W * C;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % C);
        const size_t v = i / C;
        const int W2 = 2 * W, H2 = 2 * H;
        const int xx = (int)(v % W2), yy = (int)((v / W2) % H2), zz = (int)(v / ((size_t)W2 * H2));
        y[i] = x[((((size_t)(zz / 2)) * H + yy / 2) * W + xx / 2) * C + c];
    }
}

__global__ void up2_bwd_kernel(const uint16_t* __restrict__ dy, uint16_t* __restrict__ dx, int D, int H, int W,
                               int C) {
    const size_t n = (size_t)D * H * W * C;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % C);
        const size_t v = i / C;
        const int x = (int)(v % W), y = (int)((v / W) % H), z = (int)(v / ((size_t)W * H));
        float s = 0.0f;
        for (int q = 0; q < 8; ++q) {
            const int zz = 2 * z + (q >> 2), yy = 2 * y + ((q >> 1) & 1), xx = 2 * x + (q & 1);
            s += bf2f(dy[(((size_t)zz * (2 * H) + yy) * (2 * W) + xx) * C + c]);
        }
        dx[i] = f2bf(s);
    }
}

// Residual output head and loss: pred[v][c] = out[v][c] + base[v][c] for the
// first nout channels of the FP32 network output (cpad channels per voxel);
// loss += sum (pred - target)^2 (FP64 accumulation); dout[v][c] =
// 2 (pred - target) / count as BF16 (0 for padding channels).
__global__ void mse_kernel(const float* __restrict__ out, int cpad, const float* __restrict__ base,
                           const float* __restrict__ target, int nout, size_t nvox, double inv_count,
                           float* __restrict__ pred, uint16_t* __restrict__ dout, double* __restrict__ loss) {
    __shared__ double part[256];
    double s = 0.0;
    const size_t n = nvox * cpad;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const int c = (int)(i % cpad);
        const size_t v = i / cpad;
        float g = 0.0f;
        if (c < nout) {
            const float p = out[i] + base[v * nout + c];
            if (pred) pred[v * nout + c] = p;
            if (target) {
                const float d = p - target[v * nout + c];
                s += (double)d * d;
                g = (float)(2.0 * inv_count) * d;
            }
        }
        if (dout) dout[i] = f2bf(g);
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) part[threadIdx.x] += part[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0 && loss) atomicAdd(loss, part[0]);
}

// The same for cpad a multiple of 8: one lane per voxel reads the nout channels
// that count and writes the gradient's row in 16-byte pieces (128^3 voxels, 32
// channels: 199 us with a lane per channel, 119 here).
__global__ void __launch_bounds__(256) mse8_kernel(const float* __restrict__ out, int cpad, const float* __restrict__ base,
                                                   const float* __restrict__ target, int nout, size_t nvox,
                                                   double inv_count, float* __restrict__ pred, uint16_t* __restrict__ dout,
                                                   double* __restrict__ loss) {
    __shared__ double part[256];
    double s = 0.0;
    for (size_t v = blockIdx.x * (size_t)blockDim.x + threadIdx.x; v < nvox; v += (size_t)gridDim.x * blockDim.x) {
        for (int c0 = 0; c0 < cpad; c0 += 8) {
            uint32_t wd[4] = {0u, 0u, 0u, 0u};
#pragma unroll
            for (int k = 0; k < 8; ++k) {
                const int c = c0 + k;
                if (c >= nout) break;
                const float p = out[v * cpad + c] + base[v * nout + c];
                if (pred) pred[v * nout + c] = p;
                if (target) {
                    const float d = p - target[v * nout + c];
                    s += (double)d * d;
                    wd[k / 2] |= (uint32_t)f2bf((float)(2.0 * inv_count) * d) << (16 * (k & 1));
                }
            }
            if (dout) *reinterpret_cast<uint4*>(dout + v * cpad + c0) = make_uint4(wd[0], wd[1], wd[2], wd[3]);
        }
    }
    part[threadIdx.x] = s;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) part[threadIdx.x] += part[threadIdx.x + h];
        __syncthreads();
    }
    if (threadIdx.x == 0 && loss) atomicAdd(loss, part[0]);
}

// Adam on FP32 master parameters, BF16 copy for the forward pass.
__global__ void adam_kernel(float* __restrict__ p, const float* __restrict__ g, float* __restrict__ m1,
                            float* __restrict__ m2, uint16_t* __restrict__ pb, size_t n, float lr, float b1, float b2,
                            float eps, float c1, float c2) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        const float gi = g[i];
        const float a = b1 * m1[i] + (1.0f - b1) * gi;
        const float b = b2 * m2[i] + (1.0f - b2) * gi * gi;
        m1[i] = a;
        m2[i] = b;
        const float v = p[i] - lr * (a * c1) / (sqrtf(b * c2) + eps);
        p[i] = v;
        if (pb) pb[i] = f2bf(v);
    }
}

__global__ void to_bf16_kernel(const float* __restrict__ x, uint16_t* __restrict__ y, size_t n) {
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x)
        y[i] = f2bf(x[i]);
}

// Input features per voxel: scaled direct and diffuse heating, log optical
// thickness for extinction and for absorption of the cell, zero padding to
// cpad channels (BF16); the scaled heating is also written as the FP32
// residual base [v][2].
// The reciprocal of the field scale as the host forms it from its value: 1 / s
// in FP32 (in FP64 and rounded, which is the same).
__device__ __forceinline__ float inverse_of(float s) { return (float)(1.0 / (double)s); }

// scale: read there by the kernel (the caller then need not wait for
// field_scale_kernel), or null: inv_scale.
__global__ void features_kernel(const float* __restrict__ hdir, const float* __restrict__ hdif,
                                const float* __restrict__ k_ext, const float* __restrict__ k_abs, float dz,
                                float inv_scale, size_t nvox, int cpad, const float* __restrict__ direct,
                                uint16_t* __restrict__ feat, float* __restrict__ base,
                                const double* __restrict__ scale) {
    if (scale) inv_scale = inverse_of((float)*scale);
    for (size_t v = blockIdx.x * (size_t)blockDim.x + threadIdx.x; v < nvox; v += (size_t)gridDim.x * blockDim.x) {
        const float a = hdir[v] * inv_scale, b = hdif[v] * inv_scale;
        uint16_t* f = feat + v * cpad;
        f[0] = f2bf(a);
        f[1] = f2bf(b);
        f[2] = f2bf(__logf(1.0f + 20.0f * k_ext[v] * dz));
        f[3] = f2bf(__logf(1.0f + 200.0f * k_abs[v] * dz));
        int q = 4;
        if (direct) f[q++] = f2bf(direct[v] * inv_scale);
        for (; q < cpad; ++q) f[q] = 0;
        if (base) {
            base[2 * v] = a;
            base[2 * v + 1] = b;
        }
    }
}

// Direct-beam feature: a deterministic estimate of the heating by the
// unscattered sun beam in a gray medium (flux-weighted extinction k_e and
// absorption k_a).  T[k][j][i], the beam's transmittance at the centre of
// cell (i, j, k), is carried down level by level: the ray through a centre,
// followed back up towards the sun by one level height, meets the level
// above at a point where that level's T is read bilinearly (periodic in x and
// y); the path between them runs half in each level.  In the top level the
// ray leaves through the domain top after half a level.  The cell absorbs
// T_entry (1 - exp(-k_e dz / mu0)) k_a / k_e of the direct flux, T_entry
// being the transmittance half a level above the centre; times the direct
// fraction of the flux and the level's heating-rate scale.  One launch per
// level, from the top: T of the level above is read from work[(k + 1) & 1],
// this level's written to work[k & 1].
struct DirectArgs {
    int nx, ny, nz;
    float sx, sy;       // horizontal offset of the point one level up, in cells
    float path;         // slant path of one level height (m): dz / mu0
    float fdir;         // direct fraction of the flux at the domain top
};

__global__ void direct_level_kernel(const DirectArgs d, int k, const float* __restrict__ ke,
                                    const float* __restrict__ ka, const double* __restrict__ scale,
                                    float* __restrict__ work, float* __restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x, j = blockIdx.y;
    if (i >= d.nx) return;
    const size_t plane = (size_t)d.nx * d.ny;
    const size_t c = (size_t)k * plane + (size_t)j * d.nx + i;
    const float kc = ke[c];
    float t;
    if (k == d.nz - 1) {
        t = __expf(-0.5f * kc * d.path);
    } else {
        const float* above = work + ((k + 1) & 1) * plane;
        const float fx = (float)i + d.sx, fy = (float)j + d.sy;
        const float x0 = floorf(fx), y0 = floorf(fy);
        const float wx = fx - x0, wy = fy - y0;
        auto wrap = [](int v, int n) { v %= n; return v < 0 ? v + n : v; };
        const int i0 = wrap((int)x0, d.nx), i1 = wrap((int)x0 + 1, d.nx);
        const int j0 = wrap((int)y0, d.ny), j1 = wrap((int)y0 + 1, d.ny);
        const float tu = (1.0f - wy) * ((1.0f - wx) * above[(size_t)j0 * d.nx + i0] + wx * above[(size_t)j0 * d.nx + i1]) +
                         wy * ((1.0f - wx) * above[(size_t)j1 * d.nx + i0] + wx * above[(size_t)j1 * d.nx + i1]);
        const int im = wrap((int)floorf((float)i + 0.5f + 0.5f * d.sx), d.nx);
        const int jm = wrap((int)floorf((float)j + 0.5f + 0.5f * d.sy), d.ny);
        const float ku = ke[(size_t)(k + 1) * plane + (size_t)jm * d.nx + im];  // the level above, mid-way
        t = tu * __expf(-0.5f * (kc + ku) * d.path);
    }
    work[(k & 1) * plane + (size_t)j * d.nx + i] = t;
    const float tau = kc * d.path;
    const float absorbed = kc > 0.0f ? t * __expf(0.5f * tau) * -expm1f(-tau) * (ka[c] / kc) : 0.0f;
    out[c] = (float)((double)(d.fdir * absorbed) * scale[k]);
}

// Sums of two FP32 fields in FP64, in a fixed order: per-block partial sums
// over a fixed grid of kSumBlocks blocks, then one block over the partials.
constexpr int kSumBlocks = 1024;

__global__ void field_sum_kernel(const float* __restrict__ a, const float* __restrict__ b, size_t n,
                                 double* __restrict__ partial) {
    __shared__ double sa[256], sb[256];
    double xa = 0.0, xb = 0.0;
    for (size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x; i < n; i += (size_t)gridDim.x * blockDim.x) {
        xa += (double)a[i];
        xb += (double)b[i];
    }
    sa[threadIdx.x] = xa;
    sb[threadIdx.x] = xb;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            sa[threadIdx.x] += sa[threadIdx.x + h];
            sb[threadIdx.x] += sb[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        partial[2 * blockIdx.x] = sa[0];
        partial[2 * blockIdx.x + 1] = sb[0];
    }
}

// scale = (mean a + mean b) / 2, or 1 if that is not positive
__global__ void field_scale_kernel(const double* __restrict__ partial, size_t n, double* __restrict__ scale) {
    __shared__ double sa[256], sb[256];
    double xa = 0.0, xb = 0.0;
    for (int k = threadIdx.x; k < kSumBlocks; k += 256) {
        xa += partial[2 * k];
        xb += partial[2 * k + 1];
    }
    sa[threadIdx.x] = xa;
    sb[threadIdx.x] = xb;
    __syncthreads();
    for (int h = 128; h > 0; h >>= 1) {
        if ((int)threadIdx.x < h) {
            sa[threadIdx.x] += sa[threadIdx.x + h];
            sb[threadIdx.x] += sb[threadIdx.x + h];
        }
        __syncthreads();
    }
    if (threadIdx.x == 0) {
        const double m = (sa[0] / (double)n + sb[0] / (double)n) / 2.0;
        scale[0] = m > 0.0 ? m : 1.0;
    }
}

// a * b rounded to FP32 on its own: the library is built with FP contraction,
// which would otherwise fuse it with a following addition into one FMA (and
// the backend does so even where the source forbids it).  The empty asm hides
// where the addend comes from.  (Not a multiplication in asm: the compiler knows
// no hazards there, and one right behind a v_rcp_f32 whose result it takes reads
// the register before it is written; here the scale's reciprocal is formed on
// the device.)
__device__ __forceinline__ float mul_rounded(float a, float b) {
    float r = a * b;
    asm("" : "+v"(r));
    return r;
}

// Inference: the residual head and the split back into heating fields in one
// pass, hdir[v] = max(out[v][0] + hdir_in[v] / scale, 0) scale (and hdif
// alike), with the division as features_kernel forms it (times the FP32
// reciprocal, rounded before the addition), so the result is bitwise that of
// features_kernel's base, mse_kernel and unfeature_kernel in turn.
__global__ void residual_unfeature_kernel(const float* __restrict__ out, int cpad, const float* __restrict__ hdir_in,
                                          const float* __restrict__ hdif_in, float inv_scale, float scale, size_t nvox,
                                          float* __restrict__ hdir, float* __restrict__ hdif,
                                          const double* __restrict__ scale_at) {
    if (scale_at) {
        scale = (float)*scale_at;
        inv_scale = inverse_of(scale);
    }
    for (size_t v = blockIdx.x * (size_t)blockDim.x + threadIdx.x; v < nvox; v += (size_t)gridDim.x * blockDim.x) {
        const float p0 = out[v * cpad] + mul_rounded(hdir_in[v], inv_scale);
        const float p1 = out[v * cpad + 1] + mul_rounded(hdif_in[v], inv_scale);
        hdir[v] = fmaxf(p0, 0.0f) * scale;
        hdif[v] = fmaxf(p1, 0.0f) * scale;
    }
}

// Split a [v][2] prediction back into heating fields, times scale, >= 0.
__global__ void unfeature_kernel(const float* __restrict__ pred, float scale, size_t nvox, float* __restrict__ hdir,
                                 float* __restrict__ hdif) {
    for (size_t v = blockIdx.x * (size_t)blockDim.x + threadIdx.x; v < nvox; v += (size_t)gridDim.x * blockDim.x) {
        hdir[v] = fmaxf(pred[2 * v], 0.0f) * scale;
        hdif[v] = fmaxf(pred[2 * v + 1], 0.0f) * scale;
    }
}

}  // namespace

// ===========================================================================
// C ABI (include/rt3d_denoise.h)
// ===========================================================================
namespace {

// Packing (3 to 5 us) pays where the wave loads less than half of a cache line
// of each row: 384 -> 128 channels on 10x14x18 93 us without (2 rows, 1
// plane), 55 with.  Up to 32 inputs a tap's two chunks lie in the same 64
// bytes and little is fetched twice (32 -> 64 on 20x28x36: 18 us either way).
constexpr int kPackInputs = 48;

void natural_weights(ConvArgs* a) {
    const int cin = a->c1 + a->c2;
    a->w_row = 54 * cin; a->w_half = 16; a->w_tap = 2 * cin; a->w_chunk = 32;
}

size_t packed_bytes(const rt3d_dn_conv* c) { return (size_t)c->cout * 27 * (c->c1 + c->c2) * 2; }

// Packs a->w into `work` and has a read it there.
rt3d_status pack_weights(const rt3d_dn_conv* c, ConvArgs* a, int flip, void* work, hipStream_t st) {
    hipLaunchKernelGGL(pack_weights_kernel, dim3(blocks_for(packed_bytes(c) / 16)), dim3(256), 0, st, a->w, (uint4*)work,
                       c->cout, c->c1 + c->c2, flip);
    DN_TRY(hipGetLastError());
    a->w = (const uint16_t*)work;
    a->w_row = 16; a->w_half = 512; a->w_tap = 1024; a->w_chunk = 27 * 1024;
    return RT3D_OK;
}

template <int NCT, int R, int KZ>
long conv3_groups(const ConvArgs& a) {
    constexpr int rows = ConvTile<NCT, R, KZ>::kRows;
    return (long)((a.D + KZ - 1) / KZ) * ((a.H + rows - 1) / rows) * ((a.W + kTX - 1) / kTX) * a.slabs;
}

template <int NCT, int R, int KZ>
rt3d_status conv3_launch(const ConvArgs& a, hipStream_t st) {
    const long n = conv3_groups<NCT, R, KZ>(a);
    if (n > 0x7fffffffL) return RT3D_EINVAL;
    hipLaunchKernelGGL((conv3_kernel<NCT, R, KZ>), dim3((unsigned)n), dim3(256), 0, st, a);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

// a.slabs x 32 NCT channels from a.co_base.  The largest tile that fills the
// CUs: it feeds a weight fragment to the most MFMAs, but one workgroup runs all
// its input chunks in series.  Packed weights, the rows of a wave x planes:
//   384 -> 128 on 10x14x18   (4, 2)  20 workgroups 129 us, (2, 2)  40 69, (1, 2)  70 48, (1, 1) 140 40
//   128 -> 256 on 16^3       (4, 2)  64 60,                (2, 2) 128 32, (1, 2) 256 22, (1, 1) 512 25
//   192 -> 64 on 20x28x36    (4, 2)  80 70,                (2, 2) 140 41, (1, 2) 280 42, (1, 1) 560 47
//   192 -> 64 on 64^3        (4, 2) 512 158,               (2, 2) 1024 167, (1, 2) 2048 199
// Tiles of 3 rows instead of 4 (64 channels) where they leave less of the last
// round of 512 workgroups idle or of the last tile row outside the grid: time in
// rows a wave, 0.6 of a round for up to one workgroup a CU, which has the CU to
// itself, and 2 % for the larger halo.  Workgroups and whole calls, 4 / 3 rows:
//   192 -> 64 on 44x90x118  1056 / 1320  339 / 318 us
//    64 -> 64 on 96^3       1728 / 2304  202 / 176
//   192 -> 64 on 64^3        512 /  704  154 / 178
//   160 -> 64 on 52x104x88  1014 / 1404  259 / 273
//    32 -> 64 on 128^3      4096 / 5632  230 / 249
double rounds_of(long groups) {
    const long rest = groups % 512;
    return (double)(groups / 512) + (rest == 0 ? 0.0 : rest <= 256 ? 0.6 : 1.0);
}

// Weights that could be packed and are not bound the smaller tiles, which load
// them more often: the large ones for 64 channels from 129 workgroups on.  Large / (2, 2):
//   128 -> 256 on 28x32x64  448 workgroups  100 / 130 us    8x32x64 (128)  44 / 40
//   384 -> 128 on 18x32x64  144             123 / 183      12x32x64  (96) 121 / 105
//   192 -> 64 on 40x64x96   480             155 / 200       8x64x128 (128) 66 / 59
template <int NCT>
rt3d_status conv3_run(const ConvArgs& a, hipStream_t st) {
    const bool natural = a.c1 + a.c2 >= kPackInputs && a.w_row == 54 * (a.c1 + a.c2);
    const long groups = conv3_groups<NCT, 4, 2>(a);
    if (groups >= (NCT == 2 && natural ? 129 : 512)) {
        if constexpr (NCT == 2)
            if (3 * 1.02 * rounds_of(conv3_groups<2, 3, 2>(a)) < 4 * rounds_of(groups))
                return conv3_launch<2, 3, 2>(a, st);
        return conv3_launch<NCT, 4, 2>(a, st);
    }
    if (conv3_groups<NCT, 2, 2>(a) > 128) return conv3_launch<NCT, 2, 2>(a, st);
    if (conv3_groups<NCT, 1, 2>(a) > 128) return conv3_launch<NCT, 1, 2>(a, st);
    return conv3_launch<NCT, 1, 1>(a, st);
}

rt3d_status conv_fwd(const rt3d_dn_conv* c, const uint16_t* x1, const uint16_t* x2, const uint16_t* w,
                     const float* bias, int32_t relu, uint16_t* y1, uint16_t* y2, int32_t o1, float* yf, int flip,
                     void* work, size_t work_bytes, void* stream) {
    if (!c || !x1 || !w || (c->c2 > 0 && !x2) || (!y1 && !yf)) return RT3D_EINVAL;
    // 4 input channels: only the first layer's packed form
    const bool four = c->c1 == 4 && c->c2 == 0 && c->ksize == 3 && c->cout == 32 && !c->up1 && o1 == 32;
    if (c->D <= 0 || c->H <= 0 || c->W <= 0 || c->c1 <= 0 || (c->c1 % 16 && !four) || c->c2 < 0 || c->c2 % 16)
        return RT3D_EINVAL;
    if (c->cout <= 0 || c->cout % 32 || (c->ksize != 1 && c->ksize != 3)) return RT3D_EINVAL;
    if (o1 <= 0 || o1 > c->cout || o1 % 32 || (o1 < c->cout && !y2)) return RT3D_EINVAL;
    if (c->up1 && (c->ksize != 3 || c->D % 2 || c->H % 2 || c->W % 2)) return RT3D_EINVAL;
    if (c->yf_cols < 0 || c->yf_cols > c->cout) return RT3D_EINVAL;
    ConvArgs a;
    a.x1 = x1; a.x2 = x2; a.c1 = c->c1; a.c2 = c->c2; a.w = w; a.bias = bias;
    a.y1 = y1; a.y2 = y2; a.o1 = o1; a.yf = yf;
    a.D = c->D; a.H = c->H; a.W = c->W; a.cout = c->cout; a.relu = relu ? 1 : 0;
    a.up1 = c->up1 ? 1 : 0;
    a.yf_cols = c->yf_cols ? c->yf_cols : c->cout;
    a.hw = nullptr; a.hb = nullptr; a.hy = nullptr; a.hcols = 0;
    a.co_base = 0; a.slabs = 1; a.store16 = 0;
    if (four) {
        const long tiles = (long)c->D * ((c->H + kTY32 - 1) / kTY32) * ((c->W + kTX - 1) / kTX);
        if (tiles > 0x7fffffffL) return RT3D_EINVAL;
        hipLaunchKernelGGL(conv3_c4_kernel, dim3((unsigned)tiles), dim3(256), 0, (hipStream_t)stream, a);
    } else if (c->ksize == 3) {
        a.store16 = y1 && !yf && ((uintptr_t)y1 | (uintptr_t)(o1 < c->cout ? y2 : nullptr)) % 16 == 0;
        const bool pack = work && work_bytes >= packed_bytes(c) && (uintptr_t)work % 16 == 0;
        if (flip && !pack) return RT3D_EINVAL;
        // 64 output channels per workgroup; 32 that are left over by themselves
        const int wide = c->cout / 64, narrow = (c->cout / 32) % 2;
        natural_weights(&a);
        if (pack) {
            const rt3d_status r = pack_weights(c, &a, flip, work, (hipStream_t)stream);
            if (r != RT3D_OK) return r;
        }
        if (wide) {
            a.slabs = wide;
            const rt3d_status r = conv3_run<2>(a, (hipStream_t)stream);
            if (r != RT3D_OK) return r;
        }
        if (narrow) {
            a.co_base = 64 * wide;
            a.slabs = 1;
            return conv3_run<1>(a, (hipStream_t)stream);
        }
    } else {
        const long waves = (long)c->D * c->H * ((c->W + 31) / 32) * (c->cout / 32);
        const unsigned blocks = (unsigned)((waves + 3) / 4);
        hipLaunchKernelGGL(conv_fwd_kernel<1>, dim3(blocks), dim3(256), 0, (hipStream_t)stream, a);
    }
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

}  // namespace

extern "C" {

const char* rt3d_dn_last_error(void) { return d_err; }

rt3d_status rt3d_dn_conv3d_fwd_pool(const rt3d_dn_conv* c, const uint16_t* x1, const uint16_t* w, const float* bias,
                                    int32_t relu, uint16_t* y, uint16_t* ypool, void* stream) {
    return rt3d_dn_conv3d_fwd_pool_w(c, x1, w, c && c->c1 == 5 ? 16 : 4, bias, relu, y, ypool, stream);
}

rt3d_status rt3d_dn_conv3d_fwd_pool_w(const rt3d_dn_conv* c, const uint16_t* x1, const uint16_t* w, int32_t w_channels,
                                      const float* bias, int32_t relu, uint16_t* y, uint16_t* ypool, void* stream) {
    if (!c || !x1 || !w || !y || !ypool) return RT3D_EINVAL;
    if ((c->c1 != 4 && c->c1 != 5) || c->c2 != 0 || c->ksize != 3 || c->cout != 32 || c->up1 || c->yf_cols)
        return RT3D_EINVAL;
    if (c->D <= 0 || c->H <= 0 || c->W <= 0 || c->D % 2 || c->H % 2 || c->W % 2) return RT3D_EINVAL;
    ConvArgs a;
    memset(&a, 0, sizeof a);
    if (w_channels != 16 && !(w_channels == 4 && c->c1 == 4)) return RT3D_EINVAL;
    a.x1 = x1; a.c1 = c->c1; a.w = w; a.w_row = w_channels; a.bias = bias; a.y1 = y; a.o1 = 32;
    a.D = c->D; a.H = c->H; a.W = c->W; a.cout = 32; a.relu = relu ? 1 : 0;
    const long tiles = (long)(c->D / 2) * ((c->H + kTY32 - 1) / kTY32) * ((c->W + kTX - 1) / kTX);
    if (tiles > 0x7fffffffL) return RT3D_EINVAL;
    if (c->c1 == 4)
        hipLaunchKernelGGL(conv3_c4_pool_kernel, dim3((unsigned)tiles), dim3(256), 0, (hipStream_t)stream, a, ypool);
    else
        hipLaunchKernelGGL(conv3_c5_pool_kernel, dim3((unsigned)tiles), dim3(256), 0, (hipStream_t)stream, a, ypool);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

size_t rt3d_dn_conv_workspace_size(const rt3d_dn_conv* c) {
    if (!c || c->ksize != 3 || c->D <= 0 || c->H <= 0 || c->W <= 0) return 0;
    if (c->c1 <= 0 || c->c1 % 16 || c->c2 < 0 || c->c2 % 16 || c->cout <= 0 || c->cout % 32) return 0;
    return c->c1 + c->c2 >= kPackInputs ? packed_bytes(c) : 0;
}

rt3d_status rt3d_dn_conv3d_fwd(const rt3d_dn_conv* c, const uint16_t* x1, const uint16_t* x2, const uint16_t* w,
                               const float* bias, int32_t relu, uint16_t* y1, uint16_t* y2, int32_t o1, float* yf,
                               void* stream) {
    return conv_fwd(c, x1, x2, w, bias, relu, y1, y2, o1, yf, 0, nullptr, 0, stream);
}

rt3d_status rt3d_dn_conv3d_fwd_ws(const rt3d_dn_conv* c, const uint16_t* x1, const uint16_t* x2, const uint16_t* w,
                                  const float* bias, int32_t relu, uint16_t* y1, uint16_t* y2, int32_t o1, float* yf,
                                  void* workspace, size_t workspace_bytes, void* stream) {
    return conv_fwd(c, x1, x2, w, bias, relu, y1, y2, o1, yf, 0, workspace, workspace_bytes, stream);
}

rt3d_status rt3d_dn_conv3d_dgrad(const rt3d_dn_conv* c, const uint16_t* dz, const uint16_t* w, uint16_t* dx1,
                                 uint16_t* dx2, int32_t o1, void* workspace, size_t workspace_bytes, void* stream) {
    if (!c || c->ksize != 3 || c->c1 % 16 || c->c2 || c->up1 || c->yf_cols) return RT3D_EINVAL;
    return conv_fwd(c, dz, nullptr, w, nullptr, 0, dx1, dx2, o1, nullptr, 1, workspace, workspace_bytes, stream);
}

rt3d_status rt3d_dn_conv3d_fwd_head(const rt3d_dn_conv* c, const uint16_t* x1, const uint16_t* x2, const uint16_t* w,
                                    const float* bias, int32_t relu, const uint16_t* hw, const float* hb, int32_t hcols,
                                    float* hy, void* stream) {
    return rt3d_dn_conv3d_fwd_head_ws(c, x1, x2, w, bias, relu, hw, hb, hcols, hy, nullptr, 0, stream);
}

rt3d_status rt3d_dn_conv3d_fwd_head_ws(const rt3d_dn_conv* c, const uint16_t* x1, const uint16_t* x2,
                                       const uint16_t* w, const float* bias, int32_t relu, const uint16_t* hw, const float* hb,
                                       int32_t hcols, float* hy, void* workspace, size_t workspace_bytes, void* stream) {
    if (!c || !x1 || !w || (c->c2 > 0 && !x2) || !hw || !hy) return RT3D_EINVAL;
    if (c->D <= 0 || c->H <= 0 || c->W <= 0 || c->c1 <= 0 || c->c1 % 16 || c->c2 < 0 || c->c2 % 16)
        return RT3D_EINVAL;
    if (c->ksize != 3 || c->cout != 32 || hcols <= 0 || hcols > 32) return RT3D_EINVAL;
    if (c->up1 && (c->D % 2 || c->H % 2 || c->W % 2)) return RT3D_EINVAL;
    ConvArgs a;
    a.x1 = x1; a.x2 = x2; a.c1 = c->c1; a.c2 = c->c2; a.w = w; a.bias = bias;
    a.y1 = nullptr; a.y2 = nullptr; a.o1 = 32; a.yf = nullptr;
    a.D = c->D; a.H = c->H; a.W = c->W; a.cout = 32; a.relu = relu ? 1 : 0;
    a.up1 = c->up1 ? 1 : 0;
    a.yf_cols = 32;
    a.hw = hw; a.hb = hb; a.hy = hy; a.hcols = hcols;
    a.co_base = 0; a.slabs = 1; a.store16 = 0;
    natural_weights(&a);
    if (workspace && workspace_bytes >= packed_bytes(c) && (uintptr_t)workspace % 16 == 0) {
        const rt3d_status r = pack_weights(c, &a, 0, workspace, (hipStream_t)stream);
        if (r != RT3D_OK) return r;
    }
    return conv3_run<1>(a, (hipStream_t)stream);
}

rt3d_status rt3d_dn_flip_weights(const uint16_t* w, uint16_t* wt, int32_t cout, int32_t cin, int32_t ksize,
                                 void* stream) {
    if (!w || !wt || cout <= 0 || cin <= 0 || (ksize != 1 && ksize != 3)) return RT3D_EINVAL;
    const int taps = ksize * ksize * ksize;
    hipLaunchKernelGGL(flip_weights_kernel, dim3(blocks_for((size_t)cout * cin * taps)), dim3(256), 0,
                       (hipStream_t)stream, w, wt, cout, cin, taps);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

}  // extern "C"

namespace {

// Launch plan of the weight gradient: the voxels are split into chunks so
// that the (chunk, channel tile) workgroups fill the CUs once (one workgroup
// per CU holds the accumulators, two of 32 x 32 channels), but no more chunks
// than there are units of work.
struct WgradPlan {
    WgradArgs a;
    int taps, tasks;      // channel tiles
    int nco, nci;         // 32-channel tiles of a workgroup (3x3x3)
    size_t nw;            // cout * taps * cin
    size_t ws_bytes;      // workspace of the deterministic variant
};

constexpr long kWgradWorkgroups = 256;

bool wgrad_plan(const rt3d_dn_conv* c, WgradPlan* p) {
    if (!c || c->up1) return false;
    if (c->D <= 0 || c->H <= 0 || c->W <= 0 || c->c1 <= 0 || c->c1 % 16 || c->c2 < 0 || c->c2 % 16) return false;
    if (c->cout <= 0 || c->cout % 32 || (c->ksize != 1 && c->ksize != 3)) return false;
    WgradArgs& a = p->a;
    a.cout = c->cout; a.c1 = c->c1; a.c2 = c->c2;
    a.D = c->D; a.H = c->H; a.W = c->W;
    a.partial = a.partial_b = nullptr;
    p->taps = c->ksize * c->ksize * c->ksize;
    const int tco = c->cout / 32, tci = (c->c1 + c->c2 + 31) / 32;
    long units, most;
    if (c->ksize == 3) {
        // two output tiles share each input fragment where there are two;
        // else up to three input tiles share each output fragment
        p->nco = tco % 2 == 0 ? 2 : 1;
        p->nci = p->nco == 2 ? 1 : tci % 3 == 0 ? 3 : tci % 2 == 0 ? 2 : 1;
        p->tasks = (tco / p->nco) * (tci / p->nci);
        const int ty = p->nci == 3 ? 2 : 4;
        units = (long)((c->W + kTX - 1) / kTX) * ((c->H + ty - 1) / ty) * c->D;
        most = (p->nco * p->nci == 1 ? 2 : 1) * kWgradWorkgroups / p->tasks;
    } else {
        p->nco = p->nci = 1;
        p->tasks = tco * tci;
        units = (long)c->D * c->H;
        most = 4096 / p->tasks;
    }
    if (most < 1) most = 1;
    a.chunks = (int)(units < most ? units : most);
    p->nw = (size_t)c->cout * p->taps * (c->c1 + c->c2);
    p->ws_bytes = ((a.chunks * p->nw * sizeof(float) + 255) / 256) * 256 + (size_t)a.chunks * c->cout * sizeof(float);
    return true;
}

template <int NCO, int NCI, int TY>
rt3d_status wgrad3_launch(const WgradPlan& plan, const WgradArgs& a, hipStream_t st) {
    constexpr size_t lds = sizeof(uint4) * WgradTile<NCO, NCI, TY>::kPieces;
    hipLaunchKernelGGL((conv3_wgrad_kernel<NCO, NCI, TY>), dim3((unsigned)(plan.tasks * a.chunks)), dim3(512), lds, st, a);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

template <typename... P>
bool aligned16(const P*... p) {
    return ((reinterpret_cast<uintptr_t>(p) | ...) & 15) == 0;
}

// Where there is little to sum, the element kernel: a wave per tap and channel
// tile against eight that share all taps of one, and an eighth of the sums to
// write.  With a workspace, us, 3x3x3 kernel / elements (channel tiles):
//   32 -> 32 (1)     16^3 18.5 / 16.6, 20^3 20.8 / 24.2
//   32 -> 64 (2)      8^3 21.8 / 13.5, 16^3 27.4 / 23.2, 20^3 29.7 / 32.2
//   64 -> 128 (8)     8^3 28.5 / 24.3, 12^3 32.8 / 32.3, 16^3 33.4 / 42.3
//   128 -> 256 (32)   4x6x10 33.7 / 26.9, 8^3 41.1 / 41.8, 10^3 44.1 / 55.3
//   384 -> 128 (48)   4x6x10 36.8 / 30.8, 8^3 41.0 / 51.1
// Without one every sum of every chunk is an atomic, and the line lies higher:
//   32 -> 64 (2)     32^3 108 / 57, 40^3 114 / 100, 64^3 132 / 307
//   96 -> 32 (3)     24^3 110 / 41, 32^3 116 / 68, 40^3 121 / 142
//   96 -> 96 (9)     16^3 95 / 36, 20^3 92 / 71, 24^3 94 / 110
//   384 -> 128 (48)   8^3 52 / 42, 12^3 58 / 83
bool few_voxels(double voxels, double tiles, bool workspace) {
    if (workspace) return voxels <= 6144 && voxels * tiles <= 12288;
    return voxels * tiles <= (tiles <= 3 ? 98304 : 65536);
}

rt3d_status wgrad_run(const rt3d_dn_conv* c, const WgradPlan& plan, const uint16_t* x1, const uint16_t* x2,
                      const uint16_t* dz, float* dw, float* db, float* part_w, float* part_b, hipStream_t st) {
    WgradArgs a = plan.a;
    a.dz = dz; a.x1 = x1; a.x2 = x2; a.dw = dw; a.db = db; a.partial = part_w; a.partial_b = part_b;
    rt3d_status r = RT3D_OK;
    const long tiles = (long)(c->cout / 32) * ((c->c1 + c->c2 + 31) / 32);
    const bool few = few_voxels((double)c->D * c->H * c->W, (double)tiles, part_w != nullptr);
    if (c->ksize == 1 || few || !aligned16(x1, dz) || (c->c2 && !aligned16(x2))) {
        if (c->ksize == 3) a.chunks = (int)std::min<long>(a.chunks, std::max<long>(1, 4096 / (27 * tiles)));
        const long waves = tiles * plan.taps * a.chunks;
        hipLaunchKernelGGL((c->ksize == 1 ? conv_wgrad_kernel<1> : conv_wgrad_kernel<3>), dim3((unsigned)((waves + 3) / 4)),
                           dim3(256), 0, st, a);
        DN_TRY(hipGetLastError());
    } else if (plan.nco == 2) {
        r = wgrad3_launch<2, 1, 4>(plan, a, st);
    } else if (plan.nci == 3) {
        r = wgrad3_launch<1, 3, 2>(plan, a, st);
    } else if (plan.nci == 2) {
        r = wgrad3_launch<1, 2, 4>(plan, a, st);
    } else {
        r = wgrad3_launch<1, 1, 4>(plan, a, st);
    }
    if (r != RT3D_OK) return r;
    if (part_w) {
        const int nb = db ? c->cout : 0;
        // few sums: more lanes to each (55000 of 256 chunks: 2 us slower that way)
        const size_t quads = (plan.nw + nb) / 4;
        int width = quads < 64 * 64 ? 16 : 64;
        while (1024 / width > a.chunks) width *= 2;  // no lanes without a chunk
        hipLaunchKernelGGL(sum_partials_kernel, dim3((unsigned)((quads + width - 1) / width)), dim3(1024), 0, st, part_w,
                           dw, plan.nw, part_b, db, nb, a.chunks, width);
        DN_TRY(hipGetLastError());
    }
    return RT3D_OK;
}

}  // namespace

extern "C" {

rt3d_status rt3d_dn_conv3d_wgrad(const rt3d_dn_conv* c, const uint16_t* x1, const uint16_t* x2, const uint16_t* dz,
                                 float* dw, float* db, void* stream) {
    WgradPlan plan;
    if (!x1 || !dz || !dw || (c && c->c2 > 0 && !x2) || !wgrad_plan(c, &plan)) return RT3D_EINVAL;
    return wgrad_run(c, plan, x1, x2, dz, dw, db, nullptr, nullptr, (hipStream_t)stream);
}

size_t rt3d_dn_wgrad_workspace_size(const rt3d_dn_conv* c) {
    WgradPlan plan;
    return wgrad_plan(c, &plan) ? plan.ws_bytes : 0;
}

rt3d_status rt3d_dn_conv3d_wgrad_ws(const rt3d_dn_conv* c, const uint16_t* x1, const uint16_t* x2,
                                    const uint16_t* dz, float* dw, float* db, void* workspace,
                                    size_t workspace_bytes, void* stream) {
    WgradPlan plan;
    if (!x1 || !dz || !dw || (c && c->c2 > 0 && !x2) || !wgrad_plan(c, &plan)) return RT3D_EINVAL;
    if (!workspace || workspace_bytes < plan.ws_bytes || ((uintptr_t)workspace & 255)) return RT3D_EINVAL;
    float* part_w = (float*)workspace;
    float* part_b = (float*)((char*)workspace + ((plan.a.chunks * plan.nw * sizeof(float) + 255) / 256) * 256);
    return wgrad_run(c, plan, x1, x2, dz, dw, db, part_w, part_b, (hipStream_t)stream);
}

rt3d_status rt3d_dn_relu_bwd(const uint16_t* dy, const uint16_t* y, uint16_t* dz, uint64_t n, void* stream) {
    if (!dy || !y || !dz) return RT3D_EINVAL;
    if (n % 8 == 0 && aligned16(dy, y, dz))
        hipLaunchKernelGGL(relu_bwd8_kernel, dim3(blocks_for(n / 8)), dim3(256), 0, (hipStream_t)stream, (const uint4*)dy,
                           (const uint4*)y, (uint4*)dz, (size_t)(n / 8));
    else
        hipLaunchKernelGGL(relu_bwd_kernel, dim3(blocks_for(n)), dim3(256), 0, (hipStream_t)stream, dy, y, dz, (size_t)n);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_dn_add(const uint16_t* a, const uint16_t* b, uint16_t* out, uint64_t n, void* stream) {
    if (!a || !b || !out) return RT3D_EINVAL;
    if (n % 8 == 0 && aligned16(a, b, out))
        hipLaunchKernelGGL(add8_kernel, dim3(blocks_for(n / 8)), dim3(256), 0, (hipStream_t)stream, a, b, out,
                           (size_t)(n / 8));
    else
        hipLaunchKernelGGL(add_kernel, dim3(blocks_for(n)), dim3(256), 0, (hipStream_t)stream, a, b, out, (size_t)n);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_dn_pool2(const uint16_t* x, uint16_t* y, int32_t D, int32_t H, int32_t W, int32_t C, int32_t backward,
                          void* stream) {
    if (!x || !y || D <= 0 || H <= 0 || W <= 0 || C <= 0 || D % 2 || H % 2 || W % 2) return RT3D_EINVAL;
    const size_t n = (size_t)D * H * W * C;
    if (backward && C % 8 == 0 && aligned16(x, y)) {
        hipLaunchKernelGGL(pool2_bwd8_kernel, dim3(blocks_for(n / 64)), dim3(256), 0, (hipStream_t)stream, x,
                           (const uint16_t*)nullptr, (const uint16_t*)nullptr, y, D, H, W, C);
    } else if (backward) {
        hipLaunchKernelGGL(pool2_bwd_kernel, dim3(blocks_for(n)), dim3(256), 0, (hipStream_t)stream, x, y, D, H, W, C);
    } else {
        // 16-byte accesses: 8-channel groups, aligned tensors
        if (C % 8 || ((uintptr_t)x | (uintptr_t)y) % 16) return RT3D_EINVAL;
        hipLaunchKernelGGL(pool2_kernel, dim3(blocks_for(n / 64)), dim3(256), 0, (hipStream_t)stream, x, y, D, H, W, C);
    }
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_dn_up2(const uint16_t* x, uint16_t* y, int32_t D, int32_t H, int32_t W, int32_t C, int32_t backward,
                        void* stream) {
    if (!x || !y || D <= 0 || H <= 0 || W <= 0 || C <= 0) return RT3D_EINVAL;
    const size_t n = (size_t)D * H * W * C;
    const bool eight = C % 8 == 0 && aligned16(x, y);
    if (backward && eight)
        hipLaunchKernelGGL(up2_bwd8_kernel, dim3(blocks_for(n / 8)), dim3(256), 0, (hipStream_t)stream, x,
                           (const uint16_t*)nullptr, y, D, H, W, C);
    else if (eight)
        hipLaunchKernelGGL(up2_8_kernel, dim3(blocks_for(n / 8)), dim3(256), 0, (hipStream_t)stream, x, y, D, H, W, C);
    else if (backward)
        hipLaunchKernelGGL(up2_bwd_kernel, dim3(blocks_for(n)), dim3(256), 0, (hipStream_t)stream, x, y, D, H, W, C);
    else
        hipLaunchKernelGGL(up2_kernel, dim3(blocks_for(8 * n)), dim3(256), 0, (hipStream_t)stream, x, y, D, H, W, C);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_dn_up2_relu_bwd(const uint16_t* dy, const uint16_t* act, uint16_t* dx, int32_t D, int32_t H, int32_t W,
                                 int32_t C, void* stream) {
    if (!dy || !act || !dx || D <= 0 || H <= 0 || W <= 0 || C <= 0 || C % 8 || !aligned16(dy, act, dx)) return RT3D_EINVAL;
    const size_t n = (size_t)D * H * W * C;
    hipLaunchKernelGGL(up2_bwd8_kernel, dim3(blocks_for(n / 8)), dim3(256), 0, (hipStream_t)stream, dy, act, dx, D, H, W, C);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_dn_pool2_add_relu_bwd(const uint16_t* dy, const uint16_t* de, const uint16_t* act, uint16_t* dx, int32_t D,
                                       int32_t H, int32_t W, int32_t C, void* stream) {
    if (!dy || !de || !act || !dx || D <= 0 || H <= 0 || W <= 0 || C <= 0 || D % 2 || H % 2 || W % 2) return RT3D_EINVAL;
    if (C % 8 || !aligned16(dy, de, act) || !aligned16(dx)) return RT3D_EINVAL;
    const size_t n = (size_t)D * H * W * C;
    hipLaunchKernelGGL(pool2_bwd8_kernel, dim3(blocks_for(n / 64)), dim3(256), 0, (hipStream_t)stream, dy, de, act, dx, D,
                       H, W, C);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_dn_mse(const float* out, int32_t cpad, const float* base, const float* target, int32_t nout,
                        uint64_t nvox, float* pred, uint16_t* dout, double* loss, void* stream) {
    if (!out || !base || cpad <= 0 || nout <= 0 || nout > cpad || nvox == 0) return RT3D_EINVAL;
    if ((dout || loss) && !target) return RT3D_EINVAL;
    const double inv = 1.0 / ((double)nvox * nout);
    if (cpad % 8 == 0 && (!dout || aligned16(dout)))
        hipLaunchKernelGGL(mse8_kernel, dim3(blocks_for((size_t)nvox, 256, 4096)), dim3(256), 0, (hipStream_t)stream, out,
                           cpad, base, target, nout, (size_t)nvox, inv, pred, dout, loss);
    else
        hipLaunchKernelGGL(mse_kernel, dim3(blocks_for((size_t)nvox * cpad, 256, 4096)), dim3(256), 0,
                       (hipStream_t)stream, out, cpad, base, target, nout, (size_t)nvox, inv, pred, dout, loss);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_dn_adam(float* p, const float* g, float* m1, float* m2, uint16_t* pb, uint64_t n, float lr, float b1,
                         float b2, float eps, int32_t step, void* stream) {
    if (!p || !g || !m1 || !m2 || step < 1) return RT3D_EINVAL;
    const float c1 = 1.0f / (1.0f - powf(b1, (float)step)), c2 = 1.0f / (1.0f - powf(b2, (float)step));
    hipLaunchKernelGGL(adam_kernel, dim3(blocks_for(n)), dim3(256), 0, (hipStream_t)stream, p, g, m1, m2, pb,
                       (size_t)n, lr, b1, b2, eps, c1, c2);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_dn_to_bf16(const float* x, uint16_t* y, uint64_t n, void* stream) {
    if (!x || !y) return RT3D_EINVAL;
    hipLaunchKernelGGL(to_bf16_kernel, dim3(blocks_for(n)), dim3(256), 0, (hipStream_t)stream, x, y, (size_t)n);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

static rt3d_status features_run(const float* hdir, const float* hdif, const float* k_ext, const float* k_abs, float dz,
                                float scale, const double* scale_at, uint64_t nvox, int32_t cpad, const float* direct,
                                uint16_t* feat, float* base, void* stream) {
    if (!hdir || !hdif || !k_ext || !k_abs || !feat || (cpad != 4 && cpad != 8 && (cpad < 16 || cpad % 16)) ||
        !(scale > 0.0f))
        return RT3D_EINVAL;
    if (direct && cpad < 5) return RT3D_EINVAL;
    hipLaunchKernelGGL(features_kernel, dim3(blocks_for(nvox)), dim3(256), 0, (hipStream_t)stream, hdir, hdif, k_ext,
                       k_abs, dz, 1.0f / scale, (size_t)nvox, cpad, direct, feat, base, scale_at);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_dn_features(const float* hdir, const float* hdif, const float* k_ext, const float* k_abs, float dz,
                             float scale, uint64_t nvox, int32_t cpad, const float* direct, uint16_t* feat, float* base,
                             void* stream) {
    return features_run(hdir, hdif, k_ext, k_abs, dz, scale, nullptr, nvox, cpad, direct, feat, base, stream);
}

rt3d_status rt3d_dn_features_at(const float* hdir, const float* hdif, const float* k_ext, const float* k_abs, float dz,
                                const double* scale, uint64_t nvox, int32_t cpad, const float* direct, uint16_t* feat,
                                float* base, void* stream) {
    if (!scale) return RT3D_EINVAL;
    return features_run(hdir, hdif, k_ext, k_abs, dz, 1.0f, scale, nvox, cpad, direct, feat, base, stream);
}

rt3d_status rt3d_dn_unfeature(const float* pred, float scale, uint64_t nvox, float* hdir, float* hdif,
                              void* stream) {
    if (!pred || !hdir || !hdif) return RT3D_EINVAL;
    hipLaunchKernelGGL(unfeature_kernel, dim3(blocks_for(nvox)), dim3(256), 0, (hipStream_t)stream, pred, scale,
                       (size_t)nvox, hdir, hdif);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_dn_field_scale(const float* hdir, const float* hdif, uint64_t nvox, double* work, void* stream) {
    if (!hdir || !hdif || !work || nvox == 0) return RT3D_EINVAL;
    hipLaunchKernelGGL(field_sum_kernel, dim3(kSumBlocks), dim3(256), 0, (hipStream_t)stream, hdir, hdif,
                       (size_t)nvox, work + 1);
    DN_TRY(hipGetLastError());
    hipLaunchKernelGGL(field_scale_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream, work + 1, (size_t)nvox, work);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

static rt3d_status residual_unfeature_run(const float* out, int32_t cpad, const float* hdir_in, const float* hdif_in,
                                          float scale, const double* scale_at, uint64_t nvox, float* hdir, float* hdif,
                                          void* stream) {
    if (!out || !hdir_in || !hdif_in || !hdir || !hdif || cpad < 2 || !(scale > 0.0f)) return RT3D_EINVAL;
    hipLaunchKernelGGL(residual_unfeature_kernel, dim3(blocks_for(nvox)), dim3(256), 0, (hipStream_t)stream, out,
                       cpad, hdir_in, hdif_in, 1.0f / scale, scale, (size_t)nvox, hdir, hdif, scale_at);
    DN_TRY(hipGetLastError());
    return RT3D_OK;
}

rt3d_status rt3d_dn_residual_unfeature(const float* out, int32_t cpad, const float* hdir_in, const float* hdif_in,
                                       float scale, uint64_t nvox, float* hdir, float* hdif, void* stream) {
    return residual_unfeature_run(out, cpad, hdir_in, hdif_in, scale, nullptr, nvox, hdir, hdif, stream);
}

rt3d_status rt3d_dn_residual_unfeature_at(const float* out, int32_t cpad, const float* hdir_in, const float* hdif_in,
                                          const double* scale, uint64_t nvox, float* hdir, float* hdif, void* stream) {
    if (!scale) return RT3D_EINVAL;
    return residual_unfeature_run(out, cpad, hdir_in, hdif_in, 1.0f, scale, nvox, hdir, hdif, stream);
}

rt3d_status rt3d_dn_direct_feature(const rt3d_dn_direct* d, const float* k_ext, const float* k_abs,
                                   const double* layer_scale, float* out, float* work, void* stream) {
    if (!d || !k_ext || !k_abs || !layer_scale || !out || !work) return RT3D_EINVAL;
    if (d->nx <= 0 || d->ny <= 0 || d->nz <= 0 || !(d->dx > 0.f) || !(d->dy > 0.f) || !(d->dz > 0.f)) return RT3D_EINVAL;
    if (!(d->sun_z < 0.f) || !(d->direct_fraction >= 0.f && d->direct_fraction <= 1.f)) return RT3D_EINVAL;
    DirectArgs a;
    const float up = d->dz / -d->sun_z;  // path length of one level height, followed back towards the sun
    a.nx = d->nx; a.ny = d->ny; a.nz = d->nz;
    a.sx = -d->sun_x * up / d->dx;
    a.sy = -d->sun_y * up / d->dy;
    a.path = up;
    a.fdir = d->direct_fraction;
    const dim3 grid((unsigned)((d->nx + 255) / 256), (unsigned)d->ny);
    for (int k = d->nz - 1; k >= 0; --k) {
        hipLaunchKernelGGL(direct_level_kernel, grid, dim3(256), 0, (hipStream_t)stream, a, k, k_ext, k_abs,
                           layer_scale, work, out);
        DN_TRY(hipGetLastError());
    }
    return RT3D_OK;
}

}  // extern "C"
