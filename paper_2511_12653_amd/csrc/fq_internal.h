// Internal interface between the host-side planner (fq_api.cpp) and the gfx950 kernels
// (fq_kernels.hip).  Not part of the C ABI.
#pragma once
#include <stddef.h>
#include <stdint.h>

namespace fq {

constexpr int kBlock = 256;          // threads per block: four 64-wide wavefronts
constexpr int kVecBytes = 16;        // one 128-bit global load/store per lane
constexpr int kChunkVecs = 1280;     // at most this many 128-bit vectors per block (20 KiB)
constexpr int kWaveChunkVecs = kChunkVecs / (kBlock / 64);   // what one wavefront covers: 320 vectors
constexpr int kComputeUnits = 256;   // MI355X; used by the host to balance blocks over the chip
// Three blocks per compute unit: up to here every launch has all its blocks resident at once, whatever its kernel's
// registers (forward: eight would be; backward: four to eight), and as many on one compute unit as on another.
constexpr unsigned kResidentBlocks = 3 * kComputeUnits;
// Backward launches of so many blocks, all resident at once, of so many vectors or more take the schedule made for one
// burst (burst_pays has the figures).
constexpr unsigned kBurstLeastBlocksF16 = kResidentBlocks + 1, kBurstMostBlocksF16 = 4 * kComputeUnits;
constexpr unsigned kBurstLeastBlocksF32 = 400, kBurstMostBlocksF32 = kResidentBlocks;
constexpr unsigned kBurstLeastVecsF16 = 900, kBurstLeastVecsF32 = 600;
// Channels with more units than this have 16 (32) further 64-bit slots in the workspace.  No kernel uses
// them; they keep fq_workspace_bytes and fq_layout at the values that callers have sized memory by.
constexpr unsigned kReserveUnits = 16;
constexpr unsigned kReserveSlots = 16;
constexpr unsigned kReserveManyUnits = 256;
constexpr unsigned kReserveManySlots = 32;
constexpr unsigned kTreeBlocks = 4;      // up to this many blocks per channel combine by atomic exchange alone

// Scratch memory built into the library for fq_backward_static: [slots][partial sums].
constexpr size_t kStaticScratchBytes = 1u << 20;                 // per GPU
constexpr size_t kStaticSlotBytes = 256u << 10;                  // 32768 64-bit slots
constexpr size_t kStaticPartialBytes = kStaticScratchBytes - kStaticSlotBytes;   // 98304 partial sums

// Division of 32-bit numbers by one d > 0 that the host knows (Granlund and Montgomery 1994, Fig. 4.1), exact for
// all n: s = ceil(log2 d), multiplier = floor(2^32 (2^s - d) / d) + 1, shift1 = min(s, 1), shift2 = max(s - 1, 0);
// t = high half of n * multiplier; n / d = (t + ((n - t) >> shift1)) >> shift2.
struct Divisor {
    unsigned multiplier;
    unsigned short shift1, shift2;
};

inline Divisor divisor(unsigned d)
{
    Divisor r = {0u, 0, 0};
    if (d == 0) return r;                         // an empty tensor: never divided by
    const unsigned s = d > 1 ? 32u - (unsigned)__builtin_clz(d - 1) : 0u;
    r.multiplier = (unsigned)((((1ull << s) - d) << 32) / d + 1ull);
    r.shift1 = (unsigned short)(s < 1 ? s : 1);
    r.shift2 = (unsigned short)(s > 0 ? s - 1 : 0);
    return r;
}

// Bias corrections 1 - beta^t of an Adam step that a launch brings with it (set != 0).
struct AdamBias {
    float bc1, bc2;
    unsigned set;
};

// Device-side view of one tensor.  Built on the host; passed as a kernel argument for
// single-tensor calls, or as an array in device memory for the multi-tensor launch.
struct DevTensor {
    const void *x;
    void *y;
    int8_t *q;
    const float *theta;
    float *s;
    const void *gy;
    void *gx;
    float *gs;
    float *gtheta;
    double *partial;           // [channels][outer * cps] partial sums of gy*t, one per unit; all zero between
                               // calls (backward)
    unsigned long long *slot;  // [channels] exchange slot / state of the gathering, then [channels][sub];
                               // all zero between calls (backward)
    long long inner;           // elements per slab
    unsigned slabs;            // outer * channels
    unsigned channels;
    unsigned outer;
    unsigned cps;              // chunks per slab
    unsigned chunk;            // elements per chunk, a multiple of the vector width
    unsigned block_begin;      // first block of this tensor in the grid
    unsigned chan_begin;       // first channel of this tensor in the finalize grid
    Divisor by_cps, by_channels;
    unsigned char wave_units;  // 1: slabs are short, every wavefront owns one (cps = 1, chunk = the slab);
                               // the tensor's blocks then number ceil(slabs / 4) and partial[] is per slab
    unsigned char grid3;       // 1: launched alone with a grid of (cps, channels, outer) blocks (see own_chunk)
    unsigned char sub;         // extra slots per channel after the [channels] main ones: 0, 2 (pair slots of
                               // the exchange tree, 3 or 4 units per channel) or the unused kReserve...
    unsigned char dtype;       // 0 = FP16, 1 = FP32
    unsigned char rows;        // vectors that a lane has in a whole chunk, 1 to kChunkVecs / kBlock
    float lo, hi;              // (float)qmin, (float)qmax
    float eps, s_min, s_max;
    unsigned flags;
    // fused Adam step on theta (backward); adam_m == nullptr: none
    float *adam_m, *adam_v, *adam_theta_out;
    float adam_lr, adam_beta1, adam_one_minus_beta1, adam_beta2, adam_one_minus_beta2, adam_eps;
    float adam_bc1, adam_bc2;      // 1 - beta1^t, 1 - beta2^t
};

constexpr size_t kTableEntryBytes = sizeof(DevTensor) + sizeof(unsigned);   // descriptor and packed first block

struct KArgs {
    DevTensor one;             // used when table == nullptr
    const DevTensor *table;    // device array of n descriptors, and behind it of their n first blocks
                               // (multi-tensor launch)
    int n;
    unsigned whole;            // forward of a table: most of the blocks have as many rows as a chunk can have
    AdamBias bias;             // backward of a table
};

// Launchers; each returns the hipError_t value as int (0 = success).
int launch_forward(const KArgs &a, unsigned blocks, bool emit_q, void *stream);
int launch_backward(const KArgs &a, unsigned blocks, bool fused_finalize, void *stream);
int launch_finalize(const KArgs &a, unsigned total_channels, void *stream);
int launch_scale_only(const KArgs &a, unsigned total_channels, void *stream);
int launch_fill_zero(void *p, size_t bytes, void *stream);
int copy_table_async(void *dst_device, const void *src_host, size_t bytes, void *stream);
int static_scratch(void **ptr, void *stream);
int launch_probe(int inputs, const void *a, const void *b, void *out, size_t bytes, void *stream);

}  // namespace fq
