// Distillation loss between a student and a teacher feature map and its gradient with respect to
// the student (DPVO-QAT++ Sec. 3.2, Eq. (7): MSE plus lambda times one minus the cosine
// similarity over the channel axis, averaged over positions).  This is the producer of the
// upstream gradient that the fake-quantization backward consumes.
//
// [N, C, M] tensors; a "position" is one (n, m).  The reduction runs ACROSS the channel axis, whose
// stride is M elements, so the layout is read the way it lies in memory, without transposition and
// without atomics.  Two ways, chosen on the host:
//
// One pass (fused kernel; channel counts up to 512): a block owns a tile of all channels x one run of
// positions, 128 bytes of each channel (64 FP16 or 32 FP32 positions; 512 threads) or 256 bytes (1024, 512 or 256
// threads); a lane holds 4 consecutive positions of up to 16 channels IN REGISTERS, adds its three sums
// (a.b, a.a, b.b) per position and its one sum of (a-b)^2, the wavefront adds its rows by lane exchanges,
// the block adds the wavefronts through LDS in a fixed order, forms cos and the two gradient coefficients
// per position, and every lane then writes the gradient of the elements it still holds.  HBM traffic:
// read a, read b, write ga -- the algorithmic 3 bytes-widths per element -- where the rows lie on the
// 4-element grid.  Rows that do not are read at any address, and the lines at a tile's ends come twice;
// neighbouring tiles then go to one XCD, so that its L2 has them.
//   Measured, us, before -> now: 1x384x19200 FP16 15.9 -> 12.6 (the sums over rows went through LDS in two
//   passes of 32 dependent additions, and a second launch added the tiles), 1x128x1200 7.1 -> 5.0,
//   15x128x19200 45.3 -> 43.7, 1x384x19200 FP32 25.9 -> 22.3, 4x128x19200 FP32 29.9 -> 25.5; off the grid,
//   where two kernels used to read the pair: 2x128x4819 FP32 13.1 -> 6.6, 4x256x9601 FP32 55.9 -> 35.3,
//   8x250x5001 FP16 39.7 -> 21.9.  With rows of 256 bytes by smaller blocks in launches of many tiles: 15x128x19200 FP16
//   44.2 -> 42.0, 15x64x19200 28.6 -> 25.5, 16x32x19200 23.0 -> 16.2, 15x64x9600 FP32 25.9 -> 23.0, 16x16x4800 11.9 -> 7.3.
//
// Two reads (more than 512 channels): a wavefront owns 64 lanes x V consecutive positions (one coalesced
// row per channel) and walks over a group of channels, every lane keeping the four sums of its V positions
// in binary64 registers:
//   stats kernel   one block per position tile, one wavefront per channel group (up to 16); the
//                  wavefronts add their sums through LDS in a fixed tree, then the block forms
//                  cos and the two coefficients of the gradient for its positions and leaves
//                  its sums of cos and of the squared error
//   grad kernel    elementwise: ga = k1 (a - b) - cB b + cA a, rounded once to the I/O type
// The last small step adds the per-block sums in a fixed order into the 3 results: in the fused kernel
// itself up to 256 tiles (gather_tiles), in a kernel of its own (distill_finish_kernel) or in the
// gradient kernel otherwise.
// What a call has written to its workspace is zero again when it has completed: the backward's partial sums may
// lie in the same memory, and one that is not zero reads as a unit that has arrived.  That costs the summing kernel
// 0.2 to 0.4 us (15x128x19200 FP16 44.2 -> 44.6).  After the two reads a fill does it, 1.7 to 2.4 us: every wavefront of the gradient kernel reads the coefficients, so none can clear them.
// (1x600x4800 FP16 18.5 -> 20.1, 4x768x4800 FP16 33.8 -> 36.1; a kernel that also adds the sums is no faster.)
// All arithmetic is binary64 (two conversions and five fused multiply-adds per element pair, well
// under the memory time), so results do not depend on how the channels were grouped beyond
// rounding at the 1e-16 level, and are reproducible run to run.
#include <hip/hip_runtime.h>
#include <math.h>
#include <stdint.h>

#include <atomic>
#include <chrono>

#include "../../include/fq.h"
#include "fq_device.h"
#include "fq_internal.h"

namespace fq {

using namespace dev;

namespace {

constexpr int kThreads = 256;             // gradient kernel
constexpr int kWaves = kThreads / 64;
constexpr int kUnrollC = 8;               // channels in flight per wavefront (two loads each)
constexpr unsigned kTargetWaves = 2048;   // eight wavefronts per compute unit
constexpr unsigned kMaxGroups = 16;       // wavefronts of a statistics block (1024 threads)
constexpr unsigned kTreeSlots = 4;        // wavefronts that hand their sums over per round of the LDS tree
constexpr int kMaxVec = 4;                // positions per lane (a 1024-thread block has 128 VGPRs per lane)
constexpr long long kMinTiles = 256;      // prefer this many position tiles before narrowing the loads

struct DistillArgs {
    const void *a, *b;
    void *ga;
    double *coef;       // [positions][2]
    double *blocksum;   // [tiles][2]: per-block sums of cos and of (a-b)^2
    unsigned long long *records;   // [tiles][4] and a flag: the same for a kernel that gathers them itself
    unsigned long long nonce;      // this call's number; 0: a second kernel adds the tiles' sums
    double *out;        // mse, cosim, loss
    long long M, P;     // positions per image, positions in total
    unsigned C, groups, per_group, tiles_per_n, tiles, poll_rounds;
    double k1u, k2u, eps, lambda, inv_ncm, inv_nm;
};

template <typename T, int V> struct Pack {
    typedef T type __attribute__((ext_vector_type(V)));
    static __device__ __forceinline__ T get(const type &v, int i) { return v[i]; }
    static __device__ __forceinline__ void set(type &v, int i, T x) { v[i] = x; }
};
template <typename T> struct Pack<T, 1> {
    typedef T type;
    static __device__ __forceinline__ T get(const type &v, int) { return v; }
    static __device__ __forceinline__ void set(type &v, int, T x) { v = x; }
};

typedef double double2v __attribute__((ext_vector_type(2)));

// Which tile / channel group a wavefront works on, and where its lane's V positions start.
struct Where {
    bool active, valid;
    unsigned c0, c1;
    long long first;   // element offset of (n, c0, m0)
    long long p0;      // position index of the lane's first position
};

template <int V>
__device__ __forceinline__ Where locate(const DistillArgs &k, unsigned groups, unsigned per_group)
{
    Where w;
    const unsigned wid = blockIdx.x * kWaves + (threadIdx.x >> 6);
    w.active = wid < k.tiles * groups;
    const unsigned tile = w.active ? wid / groups : 0u;
    const unsigned g = w.active ? wid % groups : 0u;
    const unsigned n = tile / k.tiles_per_n;
    const unsigned tn = tile - n * k.tiles_per_n;
    long long m0 = ((long long)tn * 64 + (threadIdx.x & 63)) * V;
    w.valid = w.active && m0 < k.M;
    if (m0 >= k.M) m0 = k.M - V;            // lanes past the end re-read the last vector; results dropped
    w.c0 = g * per_group;
    w.c1 = w.c0 + per_group < k.C ? w.c0 + per_group : k.C;
    if (w.c0 > w.c1) w.c0 = w.c1;
    w.first = ((long long)n * k.C + w.c0) * k.M + m0;
    w.p0 = (long long)n * k.M + m0;
    return w;
}

// Sums of `u` and `v` over the block (any number of wavefronts up to 16) in a fixed order; valid
// in thread 0.  red: 32 doubles of LDS.
__device__ __forceinline__ void block_sum2(double &u, double &v, double *red)
{
    u = wave_sum(u);
    v = wave_sum(v);
    if ((threadIdx.x & 63) == kSumLane) {
        red[threadIdx.x >> 6] = u;
        red[16 + (threadIdx.x >> 6)] = v;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const unsigned waves = blockDim.x >> 6;
        u = v = 0.0;
        for (unsigned i = 0; i < waves; ++i) {
            u += red[i];
            v += red[16 + i];
        }
    }
}

// One block = one position tile; wavefront w takes channel group w.  Loads roll: as soon as a
// channel's pair of vectors has been consumed its registers are refilled with the channel
// kUnrollC further on, so 2 x kUnrollC loads stay in flight while the binary64 arithmetic runs.
// Dynamic LDS: min(kTreeSlots, max(1, p/2)) x 4V x 64 doubles, p = the number of wavefronts
// rounded up to a power of two.
template <typename T, int V>
__global__ __launch_bounds__(1024) void distill_stats_kernel(DistillArgs k)
{
    typedef typename Pack<T, V>::type VT;
    constexpr int U = V >= 4 ? kUnrollC : 2 * kUnrollC;   // narrow loads: more of them in flight
    constexpr int ES = V * 4;                         // sums per lane
    extern __shared__ double lds[];                   // [slot][ES][64]
    __shared__ double red[32];

    const unsigned wave = threadIdx.x >> 6, lane = threadIdx.x & 63, waves = blockDim.x >> 6;
    const unsigned tile = blockIdx.x;
    const unsigned n = tile / k.tiles_per_n, tn = tile - n * k.tiles_per_n;
    const long long tile_m = (long long)tn * 64 * V;  // first position of the tile in its image
    long long m0 = tile_m + (long long)lane * V;
    if (m0 >= k.M) m0 = k.M - V;                      // lanes past the end re-read the last vector
    const unsigned c0 = wave * k.per_group < k.C ? wave * k.per_group : k.C;
    const unsigned c1 = c0 + k.per_group < k.C ? c0 + k.per_group : k.C;
    const unsigned nch = c1 - c0;                     // 0 for a wavefront without a group
    const long long first = ((long long)n * k.C + (nch ? c0 : 0u)) * k.M + m0;
    const T *a = (const T *)k.a + first;
    const T *b = (const T *)k.b + first;

    double acc[ES];
#pragma unroll
    for (int i = 0; i < ES; ++i) acc[i] = 0.0;
    auto accumulate = [&](const VT &va, const VT &vb) {
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const double x = (double)(float)Pack<T, V>::get(va, e);
            const double y = (double)(float)Pack<T, V>::get(vb, e);
            const double d = x - y;
            acc[e * 4 + 0] = __builtin_fma(x, y, acc[e * 4 + 0]);
            acc[e * 4 + 1] = __builtin_fma(x, x, acc[e * 4 + 1]);
            acc[e * 4 + 2] = __builtin_fma(y, y, acc[e * 4 + 2]);
            acc[e * 4 + 3] = __builtin_fma(d, d, acc[e * 4 + 3]);
        }
    };

    if (nch) {
        VT ra[U], rb[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const unsigned cu = (unsigned)u < nch ? (unsigned)u : nch - 1;
            ra[u] = ld_global((const VT *)(a + (long long)cu * k.M));
            rb[u] = ld_global((const VT *)(b + (long long)cu * k.M));
        }
        unsigned c = 0;
        for (; c + U < nch; c += U) {                 // a next block exists, at least in part
#pragma unroll
            for (int u = 0; u < U; ++u) {
                accumulate(ra[u], rb[u]);
                unsigned nc = c + U + u;
                if (nc >= nch) nc = nch - 1;          // re-read of the last channel, never used
                ra[u] = ld_global((const VT *)(a + (long long)nc * k.M));
                rb[u] = ld_global((const VT *)(b + (long long)nc * k.M));
            }
        }
#pragma unroll
        for (int u = 0; u < U; ++u)
            if (c + u < nch) accumulate(ra[u], rb[u]);
    }

    // Fixed tree over the wavefronts: w += w + stride for stride = 8, 4, 2, 1, at most kTreeSlots
    // wavefronts handing over per round so that the LDS footprint stays at 4 x 4V x 64 doubles.
    for (unsigned stride = kMaxGroups / 2; stride >= 1; stride >>= 1) {
        if (stride >= waves) continue;                // uniform over the block
        for (unsigned base = 0; base < stride; base += kTreeSlots) {
            const unsigned giver = stride + base;     // first wavefront that hands over in this round
            if (wave >= giver && wave < giver + kTreeSlots && wave < 2 * stride) {
#pragma unroll
                for (int i = 0; i < ES; ++i) lds[((wave - giver) * ES + i) * 64 + lane] = acc[i];
            }
            __syncthreads();
            if (wave >= base && wave < base + kTreeSlots && wave < stride && wave + stride < waves) {
#pragma unroll
                for (int i = 0; i < ES; ++i) acc[i] += lds[((wave - base) * ES + i) * 64 + lane];
            }
            __syncthreads();
        }
    }
    if (wave == 0) {
#pragma unroll
        for (int i = 0; i < ES; ++i) lds[i * 64 + lane] = acc[i];
    }
    __syncthreads();

    // One thread per position of the tile: cos, the coefficients of the gradient, block sums.
    double cos_sum = 0.0, sq_sum = 0.0;
    for (unsigned pp = threadIdx.x; pp < 64u * V; pp += blockDim.x) {
        const unsigned src = pp / V, e = pp % V;
        const long long m = tile_m + pp;
        if (m < k.M) {
            const double dot = lds[(e * 4 + 0) * 64 + src], na = lds[(e * 4 + 1) * 64 + src];
            const double nb = lds[(e * 4 + 2) * 64 + src], sq = lds[(e * 4 + 3) * 64 + src];
            const double ra = sqrt(na), rb = sqrt(nb);
            // a NaN norm stays NaN, so a non-finite input poisons its whole position visibly
            const double ca = ra < k.eps ? k.eps : ra, cb = rb < k.eps ? k.eps : rb;
            const double inv = 1.0 / (ca * cb);
            const double cosp = dot / (ca * cb);
            const double self = ra > k.eps ? cosp / na : 0.0;
            if (k.coef) {
                double2v o = {k.k2u * inv, k.k2u * self};
                st_global((double2v *)k.coef + ((long long)n * k.M + m), o);
            }
            cos_sum += cosp;
            sq_sum += sq;
        }
    }
    block_sum2(cos_sum, sq_sum, red);
    if (threadIdx.x == 0) {
        double2v o = {cos_sum, sq_sum};
        st_global((double2v *)k.blocksum + tile, o);
    }
}

// The three results from the per-block sums, added in a fixed order by one wavefront: lane l takes
// the sums l, l + 64, l + 128, ... (eight loads in flight at a time: thousands of tiles would
// otherwise be as many dependent round trips to memory), then the lanes are added by wave_sum.
__device__ __forceinline__ void finish(const DistillArgs &k)
{
    const unsigned lane = threadIdx.x & 63;
    double sc = 0.0, ss = 0.0;
    constexpr unsigned kBatch = 8;
    for (unsigned i0 = lane; i0 < k.tiles; i0 += 64 * kBatch) {
        double2v v[kBatch];
#pragma unroll
        for (unsigned j = 0; j < kBatch; ++j) {
            const unsigned i = i0 + 64 * j;
            v[j] = double2v{0.0, 0.0};
            if (i < k.tiles) v[j] = ld_global((const double2v *)k.blocksum + i);
        }
#pragma unroll
        for (unsigned j = 0; j < kBatch; ++j) {
            if (i0 + 64 * j < k.tiles) {
                sc += v[j][0];
                ss += v[j][1];
            }
        }
    }
    sc = wave_sum(sc);
    ss = wave_sum(ss);
    if (lane == kSumLane) {
        const double mse = ss * k.inv_ncm, cosim = sc * k.inv_nm;
        st_global(k.out + 0, mse);
        st_global(k.out + 1, cosim);
        st_global(k.out + 2, mse + k.lambda * (1.0 - cosim));
    }
}

// The same as a kernel of its own, by one block of 1024 threads: thread t takes the sums t,
// t + 1024, ..., the wavefronts add their lanes (wave_sum), thread 0 adds the sixteen wavefront
// sums in index order.  The sums' places are zero afterwards.
__global__ __launch_bounds__(1024) void distill_finish_kernel(DistillArgs k)
{
    __shared__ double part[2 * 16];
    double sc = 0.0, ss = 0.0;
    constexpr unsigned kBatch = 4;
    for (unsigned i0 = threadIdx.x; i0 < k.tiles; i0 += 1024 * kBatch) {
        double2v v[kBatch];
#pragma unroll
        for (unsigned j = 0; j < kBatch; ++j) {
            const unsigned i = i0 + 1024 * j;
            v[j] = double2v{0.0, 0.0};
            if (i < k.tiles) v[j] = ld_global((const double2v *)k.blocksum + i);
        }
#pragma unroll
        for (unsigned j = 0; j < kBatch; ++j) {
            if (i0 + 1024 * j < k.tiles) {
                sc += v[j][0];
                ss += v[j][1];
            }
        }
    }
    for (unsigned i = threadIdx.x; i < k.tiles; i += 1024) st_global((double2v *)k.blocksum + i, double2v{0.0, 0.0});
    sc = wave_sum(sc);
    ss = wave_sum(ss);
    if ((threadIdx.x & 63) == kSumLane) {
        part[threadIdx.x >> 6] = sc;
        part[16 + (threadIdx.x >> 6)] = ss;
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        sc = ss = 0.0;
        for (unsigned w = 0; w < 16; ++w) {
            sc += part[w];
            ss += part[16 + w];
        }
        const double mse = ss * k.inv_ncm, cosim = sc * k.inv_nm;
        st_global(k.out + 0, mse);
        st_global(k.out + 1, cosim);
        st_global(k.out + 2, mse + k.lambda * (1.0 - cosim));
    }
}

template <typename T, int V>
__global__ __launch_bounds__(kThreads) void distill_grad_kernel(DistillArgs k, unsigned groups, unsigned per_group)
{
    typedef typename Pack<T, V>::type VT;
    if (blockIdx.x == 0 && threadIdx.x < 64) finish(k);
    const Where w = locate<V>(k, groups, per_group);
    if (!w.active) return;
    const T *a = (const T *)k.a + w.first;
    const T *b = (const T *)k.b + w.first;
    T *ga = (T *)k.ga + w.first;
    double cb[V], ca[V];
#pragma unroll
    for (int e = 0; e < V; ++e) {
        const double2v v = ld_global((const double2v *)k.coef + w.p0 + e);
        cb[e] = v[0];
        ca[e] = v[1];
    }
    auto grad = [&](const VT &va, const VT &vb) {
        VT o;
#pragma unroll
        for (int e = 0; e < V; ++e) {
            const double x = (double)(float)Pack<T, V>::get(va, e);
            const double y = (double)(float)Pack<T, V>::get(vb, e);
            double g = k.k1u * (x - y);
            g = __builtin_fma(-cb[e], y, g);
            g = __builtin_fma(ca[e], x, g);
            Pack<T, V>::set(o, e, (T)(float)g);
        }
        return o;
    };
    constexpr int U = kUnrollC / 2;
    unsigned c = w.c0;
    for (; c + U <= w.c1; c += U) {
        VT ra[U], rb[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            ra[u] = ld_stream((const VT *)(a + (long long)u * k.M));
            rb[u] = ld_stream((const VT *)(b + (long long)u * k.M));
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const VT o = grad(ra[u], rb[u]);
            if (w.valid) st_stream((VT *)(ga + (long long)u * k.M), o);
        }
        a += (long long)U * k.M;
        b += (long long)U * k.M;
        ga += (long long)U * k.M;
    }
    for (; c < w.c1; ++c) {
        const VT o = grad(ld_stream((const VT *)a), ld_stream((const VT *)b));
        if (w.valid) st_stream((VT *)ga, o);
        a += k.M;
        b += k.M;
        ga += k.M;
    }
}

// ---------------------------------------------------------------------------------------------
// One pass over the pair.  A block of THREADS threads = R rows of L lanes; lane l of row r holds
// positions 4l .. 4l+3 of the tile for channels r, r + R, r + 2R, ... (KCH of them at most).
constexpr int kFusedVec = 4;                     // positions per lane
constexpr int kFusedMaxKch = 16;                 // channels per lane the registers hold (FP16; half for FP32)
// The shapes of a tile: threads of its block and bytes of each channel in it.  Which one is taken, and why, stands at
// make_plan.  (Rows of 64 bytes would cut a 1x384x120x160 pair into 600 tiles and spread them more evenly over the
// 256 compute units, but half-line accesses cost more than the balance gains: 24.4 us against 16.9.)
enum TileShape { kNarrow, kWide, kLong, kSmall };
constexpr int kTileThreads[] = {512, 1024, 512, 256};
constexpr int kTileRowBytes[] = {128, 256, 256, 256};
template <typename T, int SHAPE> struct FusedShape {
    static constexpr int THREADS = kTileThreads[SHAPE];
    static constexpr int L = kTileRowBytes[SHAPE] / (kFusedVec * (int)sizeof(T));   // lanes per row
    static constexpr int P = kFusedVec * L;                                         // positions per tile
    static constexpr int R = THREADS / L;                                           // channel rows
    static constexpr bool GATHERS = SHAPE == kNarrow || SHAPE == kWide;             // may be launched without a second kernel
};

// Four positions of one channel.  QUADS: rows lie on the 4-element grid.  Otherwise a row starts at
// any element, and the compiler is told so: the target reads and writes 8 or 16 bytes at any address.
template <typename T, bool QUADS> struct Quad {
    typedef T Regs __attribute__((ext_vector_type(4)));
    typedef T Memory __attribute__((ext_vector_type(4), aligned(QUADS ? 4 * sizeof(T) : sizeof(T))));
    static __device__ __forceinline__ Regs load(const T *p) { return __builtin_nontemporal_load((const FQ_GLOBAL Memory *)p); }
    static __device__ __forceinline__ void store(T *p, Regs v) { __builtin_nontemporal_store(v, (FQ_GLOBAL Memory *)p); }
};

// One step of adding the rows of a wavefront: afterwards a + b is, in the lanes of the even rows, the sum of
// a over two rows, and in those of the odd rows the sum of b (rows of 32 lanes or of 16).  Two values and
// two rows become one value per lane for two instructions per 32 bits and one addition.
__device__ __forceinline__ void swap_halves(double &a, double &b, bool rows_of_32)
{
    unsigned long long ua = __builtin_bit_cast(unsigned long long, a), ub = __builtin_bit_cast(unsigned long long, b);
    unsigned al = (unsigned)ua, ah = (unsigned)(ua >> 32), bl = (unsigned)ub, bh = (unsigned)(ub >> 32);
    if (rows_of_32) {
        const auto l = __builtin_amdgcn_permlane32_swap(al, bl, false, false);
        const auto h = __builtin_amdgcn_permlane32_swap(ah, bh, false, false);
        al = l[0]; bl = l[1]; ah = h[0]; bh = h[1];
    } else {
        const auto l = __builtin_amdgcn_permlane16_swap(al, bl, false, false);
        const auto h = __builtin_amdgcn_permlane16_swap(ah, bh, false, false);
        al = l[0]; bl = l[1]; ah = h[0]; bh = h[1];
    }
    a = __builtin_bit_cast(double, ((unsigned long long)ah << 32) | al);
    b = __builtin_bit_cast(double, ((unsigned long long)bh << 32) | bl);
}

constexpr int kStats = 3 * kFusedVec;            // per lane: a.b, a.a, b.b of four positions

// The three results out of the tiles' sums, by one wavefront, in the kernel that makes them (at most
// kGatherTiles tiles).  A tile's record is {cos, cos ^ N, sq, sq ^ N} with a number N of this call's own: the
// workspace may hold anything, and a pair of words that does not fit together with N has not arrived.
// The protocol is that of the backward's sums (kPollRounds rounds, then a flag, here N, and the tile that
// arrives last finishes; whoever claims the call puts ~N into the flag).  Afterwards all four words are zero,
// which fits no N.  A graph replays N, and the words travel one by one: a pair left as it is would be taken
// for the next replay's where that one's other pair is visible first.
constexpr unsigned kGatherTiles = 256;
constexpr unsigned kPollRounds = 32;

__device__ __forceinline__ unsigned long long bits_of(double v) { return __builtin_bit_cast(unsigned long long, v); }
__device__ __forceinline__ void wait_stores_acknowledged() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

__device__ __forceinline__ bool gather_tiles(const DistillArgs &k, double &sc, double &ss)
{
    const unsigned lane = threadIdx.x & 63;
    constexpr unsigned kEach = kGatherTiles / 64;
    unsigned long long w[kEach][4];
#pragma unroll
    for (unsigned i = 0; i < kEach; ++i) {
        const unsigned tile = lane + 64 * i;
        if (tile < k.tiles) {
#pragma unroll
            for (int j = 0; j < 4; ++j)
                w[i][j] = __hip_atomic_load(k.records + (size_t)tile * 4 + j, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
    }
    bool here = true;
    sc = ss = 0.0;
#pragma unroll
    for (unsigned i = 0; i < kEach; ++i) {
        if (lane + 64 * i < k.tiles) {
            here = here && (w[i][0] ^ w[i][1]) == k.nonce && (w[i][2] ^ w[i][3]) == k.nonce;
            sc += __builtin_bit_cast(double, w[i][0]);
            ss += __builtin_bit_cast(double, w[i][2]);
        }
    }
    sc = wave_sum(sc);
    ss = wave_sum(ss);
    return __builtin_amdgcn_ballot_w64(!here) == 0ull;
}

__device__ __forceinline__ void write_results(const DistillArgs &k, double sc, double ss)
{
    const double mse = ss * k.inv_ncm, cosim = sc * k.inv_nm;
    st_global(k.out + 0, mse);
    st_global(k.out + 1, cosim);
    st_global(k.out + 2, mse + k.lambda * (1.0 - cosim));
}

__device__ __forceinline__ void finish_gathered(const DistillArgs &k, double sc, double ss)
{
    const unsigned lane = threadIdx.x & 63;
    if (lane == kSumLane) write_results(k, sc, ss);
    // (Plain stores, 16 bytes each: nobody else needs to see them within this launch, and written through to the
    // level that all XCDs share, one word each, they add 0.2 to 0.5 us: 2x128x4819 FP32 7.46 / 7.14, 1x128x16384
    // FP16 6.41 / 5.88.)
    for (unsigned i = lane; i < k.tiles * 2; i += 64) st_global((double2v *)k.records + i, double2v{0.0, 0.0});
}

__device__ __forceinline__ void finish_if_complete(const DistillArgs &k, unsigned long long *flag)
{
    double sc, ss;
    if (!gather_tiles(k, sc, ss)) return;
    unsigned won = 0u;
    if ((threadIdx.x & 63) == 0) {
        unsigned long long expected = k.nonce;
        won = __hip_atomic_compare_exchange_strong(flag, &expected, ~k.nonce, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT) ? 1u : 0u;
    }
    if (!__builtin_amdgcn_readfirstlane((int)won)) return;
    finish_gathered(k, sc, ss);
    if ((threadIdx.x & 63) == 0) __hip_atomic_store(flag, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// One wavefront of every block, when its own work is done; the block's record is on its way.
// A look costs about 0.5 us, and one that comes too early costs that for nothing.  Without a gradient the block that looks is done
// as soon as the others are, so with more than 64 tiles its first look waits 0.3 us for their records.  Since the first loads no longer
// wait for the kernel's arguments, the look without the wait came too early for some shapes.  us, loads behind the arguments / loads
// early / and the wait, without a gradient: 13x45x704 FP16 (143 tiles) 5.0 / 5.5 / 4.8; over 2800 pairs of 65 to 256 tiles,
// against the first, 0.09 less early on average, one shape in twenty 1.05 of the time and the worst 1.10; with the wait 0.33 less, one in
// twenty above 1.008, worst 1.05.  (A wait of 0.05 or 0.1 us leaves half of that, 0.24 gains 0.06 less.)  Up to 64 tiles nothing was lost.
// With a gradient, which takes the block longer, a wait of 0.1 us and more only adds to the time of most shapes; there one shape in twenty of
// more than 128 tiles stays 2 to 5 % above the first.
template <bool WANT_GRAD> __device__ __forceinline__ void gather_or_leave(const DistillArgs &k)
{
    unsigned long long *flag = k.records + (size_t)k.tiles * 4;
    if (blockIdx.x + 1u != k.tiles) {
        wait_stores_acknowledged();
        const unsigned long long f = __hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        if (__builtin_expect(f == k.nonce, 0)) finish_if_complete(k, flag);
        return;
    }
    double sc, ss;
    if (!WANT_GRAD && k.tiles > 64u) __builtin_amdgcn_s_sleep(12);
    for (unsigned round = 0; round < k.poll_rounds; ++round) {
        asm volatile("" ::: "memory");
        if (gather_tiles(k, sc, ss)) {
            finish_gathered(k, sc, ss);
            return;
        }
    }
    wait_stores_acknowledged();
    if ((threadIdx.x & 63) == 0) __hip_atomic_store(flag, k.nonce, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wait_stores_acknowledged();
    finish_if_complete(k, flag);
}

// Blocks go to the eight XCDs in turn; this gives each XCD a run of neighbouring tiles.  One to one.
// Only where rows are no whole number of 128-byte lines, so that neighbours share the lines at their ends, us
// without / with: 4x256x9601 FP32 40.2 / 35.3, 8x250x5001 FP16 26.6 / 21.9, 3x134x6588 FP32 14.9 / 12.4, 6x200x3300
// FP32 18.4 / 16.3; otherwise it loses: 15x128x19200 FP16 44.3 / 47.4.
__device__ __forceinline__ unsigned tile_of_block(unsigned block, unsigned tiles)
{
    constexpr unsigned kXcds = 8;
    const unsigned each = tiles / kXcds, more = tiles % kXcds, xcd = block % kXcds;
    return xcd * each + (xcd < more ? xcd : more) + block / kXcds;
}

// The leading arguments, which are what the first loads' addresses are made of, come in registers with the launch (see
// forward_kernel in the other file).  neighbours: 0, or the number of tiles (see tile_of_block).
// (Known loss: FP16 pairs of 257 to 384 channels with a gradient, in at most 256 tiles the last of which has 4 or 8 positions, take
// longer with the same instructions when their loads start earlier: 6x300x132 8.7 / 9.3 us, 12x365x68 10.2 / 10.9; with 12 positions
// 7.9 / 7.8.  Leaving out the loads of absent positions, spreading them, or storing such tiles by plain stores changes nothing or little.)
template <typename T, int SHAPE, int KCH, bool QUADS, bool WANT_GRAD>
__global__ __launch_bounds__(kTileThreads[SHAPE], 4)
void distill_fused_kernel(const void *student, const void *teacher, long long M, unsigned C, unsigned tiles_per_n,
                          unsigned by_multiplier, unsigned by_shifts, unsigned neighbours, const DistillArgs rest)
{
    DistillArgs k = rest;
    k.a = student;
    k.b = teacher;
    k.M = M;
    k.C = C;
    k.tiles_per_n = tiles_per_n;
    const Divisor by_tiles_per_n = {by_multiplier, (unsigned short)by_shifts, (unsigned short)(by_shifts >> 16)};
    typedef FusedShape<T, SHAPE> Shape;
    constexpr int THREADS = Shape::THREADS;
    constexpr int V = kFusedVec, L = Shape::L, P = Shape::P, R = Shape::R, W = THREADS / 64, S = 64 / L;
    constexpr int HELD = S >= 4 ? kStats / 4 : kStats / 2;      // sums a lane is left with
    typedef Quad<T, QUADS> Q;
    typedef typename Q::Regs Regs;
    __shared__ double red[W * 3 * P];             // per wavefront, statistic and position
    __shared__ double red_sq[W];                  // per wavefront: (a-b)^2
    __shared__ double coefs[P * 2];               // per position: the two gradient coefficients
    __shared__ double cosines[P];

    const unsigned lane = threadIdx.x % L, row = threadIdx.x / L, wave = threadIdx.x >> 6;
    const unsigned tile = neighbours ? tile_of_block(blockIdx.x, neighbours) : blockIdx.x;
    const unsigned n = divide(tile, by_tiles_per_n), tn = tile - n * k.tiles_per_n;
    const long long tile_m = (long long)tn * P;
    long long m0 = tile_m + (long long)lane * V;
    // positions of this lane that exist; QUADS: four or none (none: re-read the last quad, results dropped)
    const int valid = m0 >= k.M ? 0 : (m0 + V <= k.M ? V : (int)(k.M - m0));
    if (QUADS && !valid) m0 = k.M - V;
    const bool whole = QUADS || valid == V;
    const long long base = (long long)n * k.C * k.M + m0;
    const T *a = (const T *)k.a + base;
    const T *b = (const T *)k.b + base;

    Regs ra[KCH], rb[KCH];
    if (whole) {
#pragma unroll
        for (int j = 0; j < KCH; ++j) {
            unsigned c = row + (unsigned)j * R;
            c = c < k.C ? c : k.C - 1;            // rows past the last channel re-read it; results dropped
            ra[j] = Q::load(a + (long long)c * k.M);
            rb[j] = Q::load(b + (long long)c * k.M);
        }
    } else {
#pragma unroll
        for (int j = 0; j < KCH; ++j) {
            unsigned c = row + (unsigned)j * R;
            c = c < k.C ? c : k.C - 1;
#pragma unroll
            for (int e = 0; e < V; ++e) {
                ra[j][e] = e < valid ? ld_global(a + (long long)c * k.M + e) : (T)0.0f;
                rb[j][e] = e < valid ? ld_global(b + (long long)c * k.M + e) : (T)0.0f;
            }
        }
    }

    // acc[e * 3 + s]: statistic s of position e
    double acc[kStats], sq = 0.0;
#pragma unroll
    for (int i = 0; i < kStats; ++i) acc[i] = 0.0;
#pragma unroll
    for (int j = 0; j < KCH; ++j) {
        if (row + (unsigned)j * R < k.C) {
#pragma unroll
            for (int e = 0; e < V; ++e) {
                const double x = (double)(float)ra[j][e];
                const double y = (double)(float)rb[j][e];
                const double d = x - y;
                acc[e * 3 + 0] = __builtin_fma(x, y, acc[e * 3 + 0]);
                acc[e * 3 + 1] = __builtin_fma(x, x, acc[e * 3 + 1]);
                acc[e * 3 + 2] = __builtin_fma(y, y, acc[e * 3 + 2]);
                sq = __builtin_fma(d, d, sq);
            }
        }
    }
    if (QUADS && !valid) sq = 0.0;                // (a re-read quad; without QUADS absent positions hold zeros)

    // Over the rows of the wavefront, then over the wavefronts.
#pragma unroll
    for (int i = 0; i < kStats / 2; ++i) {
        swap_halves(acc[i], acc[i + kStats / 2], true);
        acc[i] += acc[i + kStats / 2];
    }
    unsigned e0 = (threadIdx.x & 32) ? 2 : 0;     // the first of the positions whose sums this lane is left with
    if (S >= 4) {
#pragma unroll
        for (int i = 0; i < kStats / 4; ++i) {
            swap_halves(acc[i], acc[i + kStats / 4], false);
            acc[i] += acc[i + kStats / 4];
        }
        e0 += (threadIdx.x & 16) ? 1 : 0;
    }
    if (S == 8) {                                 // rows of eight lanes: add the other one of the sixteen
#pragma unroll
        for (int i = 0; i < kStats / 4; ++i) acc[i] += dpp_move<0x128, 0xf>(acc[i]);      // row_ror:8
    }
    if (S < 8 || (threadIdx.x & 8) == 0) {
#pragma unroll
        for (int i = 0; i < HELD; ++i) red[(wave * 3 + i % 3) * P + lane * V + e0 + i / 3] = acc[i];
    }
    sq = wave_sum(sq);
    if ((threadIdx.x & 63) == kSumLane) red_sq[wave] = sq;
    __syncthreads();

    // One thread per position: cos and the gradient's coefficients.
    if (threadIdx.x < (unsigned)P) {
        const unsigned pp = threadIdx.x;
        double dot = 0.0, na = 0.0, nb = 0.0;
#pragma unroll
        for (int w = 0; w < W; ++w) {
            dot += red[(w * 3 + 0) * P + pp];
            na += red[(w * 3 + 1) * P + pp];
            nb += red[(w * 3 + 2) * P + pp];
        }
        const double ra_ = sqrt(na), rb_ = sqrt(nb);
        // a NaN norm stays NaN, so a non-finite input poisons its whole position visibly
        const double ca = ra_ < k.eps ? k.eps : ra_, cb = rb_ < k.eps ? k.eps : rb_;
        const double inv = 1.0 / (ca * cb);
        const double cosp = dot / (ca * cb);
        const double self = ra_ > k.eps ? cosp / na : 0.0;
        coefs[pp * 2 + 0] = k.k2u * inv;
        coefs[pp * 2 + 1] = k.k2u * self;
        cosines[pp] = tile_m + pp < k.M ? cosp : 0.0;
    }
    __syncthreads();

    if (wave == 0) {                              // the tile's sums of cos and of the squared error
        double cos_sum = threadIdx.x < (unsigned)P ? cosines[threadIdx.x] : 0.0;
        if (P > 64) cos_sum += cosines[64 + threadIdx.x];
        double sq_sum = threadIdx.x < (unsigned)W ? red_sq[threadIdx.x] : 0.0;
        cos_sum = wave_sum(cos_sum);
        sq_sum = wave_sum(sq_sum);
        if (threadIdx.x == kSumLane) {
            if (Shape::GATHERS && k.nonce) {
                unsigned long long *r = k.records + (size_t)tile * 4;
                const unsigned long long w[4] = {bits_of(cos_sum), bits_of(cos_sum) ^ k.nonce, bits_of(sq_sum),
                                                 bits_of(sq_sum) ^ k.nonce};
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    __hip_atomic_store(r + j, w[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                double2v o = {cos_sum, sq_sum};
                st_global((double2v *)k.blocksum + tile, o);
            }
        }
    }

    if (WANT_GRAD && valid) {
        double cb[V], ca[V];
#pragma unroll
        for (int e = 0; e < V; ++e) {
            cb[e] = coefs[(lane * V + e) * 2 + 0];
            ca[e] = coefs[(lane * V + e) * 2 + 1];
        }
        T *ga = (T *)k.ga + base;
#pragma unroll
        for (int j = 0; j < KCH; ++j) {
            const unsigned c = row + (unsigned)j * R;
            if (c < k.C) {
                Regs o;
#pragma unroll
                for (int e = 0; e < V; ++e) {
                    const double x = (double)(float)ra[j][e];
                    const double y = (double)(float)rb[j][e];
                    double g = k.k1u * (x - y);
                    g = __builtin_fma(-cb[e], y, g);
                    g = __builtin_fma(ca[e], x, g);
                    o[e] = (T)(float)g;
                }
                T *to = ga + (long long)c * k.M;
                if (whole) {
                    Q::store(to, o);
                } else {
#pragma unroll
                    for (int e = 0; e < V; ++e)
                        if (e < valid) st_global(to + e, (T)o[e]);
                }
            }
        }
    }
    if (Shape::GATHERS && k.nonce && wave == 0) gather_or_leave<WANT_GRAD>(k);
}

size_t align256(size_t v) { return (v + 255) & ~(size_t)255; }

struct Plan {
    int vec;                 // elements per lane
    int fused_kch;           // > 0: the fused kernel with this many channels per lane; 0: two kernels
    bool quads;              // fused: see Quad
    TileShape shape;         // fused
    bool neighbours;         // fused: see tile_of_block
    bool one_launch;         // fused: the kernel adds its tiles' sums itself
    unsigned tiles_per_n, tiles, groups, per_group, grad_groups, grad_per_group;
    size_t stats_lds, off_blocksum, bytes;
};

template <typename T> constexpr int positions_of(int shape) { return kTileRowBytes[shape] / (int)sizeof(T); }
template <typename T> constexpr int rows_of(int shape) { return kTileThreads[shape] * kFusedVec * (int)sizeof(T) / kTileRowBytes[shape]; }

// Channels per lane that a tile's shape is built for, at most.
template <typename T> constexpr int most_channels_per_lane(int shape)
{
    return shape == kSmall ? 4 : sizeof(T) == 2 ? kFusedMaxKch : kFusedMaxKch / 2;
}

long long tile_positions(const fq_distill *d, TileShape s) { return d->dtype == FQ_F16 ? positions_of<_Float16>(s) : positions_of<float>(s); }

// Channels per lane the fused kernel needs for this pair with tiles of this shape, rounded up to a width it is
// built for; 0 if there are more channels than a lane's registers hold.
int fused_channels_per_lane(const fq_distill *d, TileShape s)
{
    const bool half = d->dtype == FQ_F16;
    const long long rows = half ? rows_of<_Float16>(s) : rows_of<float>(s);
    const long long need = (d->channels + rows - 1) / rows;
    const long long cap = half ? most_channels_per_lane<_Float16>(s) : most_channels_per_lane<float>(s);
    if (need > cap) return 0;
    for (int kch : {2, 4, 6, 8, 12, 16})
        if (kch >= need) return kch;
    return 0;
}

// Whether all rows of the pair lie on the 4-element grid.
bool on_quads(const fq_distill *d)
{
    const size_t esz = d->dtype == FQ_F16 ? 2 : 4;
    const uintptr_t addr_bits = (uintptr_t)d->student | (uintptr_t)d->teacher | (uintptr_t)d->gstudent;
    return d->inner % kFusedVec == 0 && addr_bits % (kFusedVec * esz) == 0;
}

// The shape of the tiles in launches of more than kGatherTiles of them, which a second kernel follows.  Rows of 256
// bytes: longer runs in memory and half the tiles, for as many positions behind the last tile of an image.
//
// Long tiles, 512 threads: a compute unit holds two to four of them, so that some read while others reduce or write.
// Measured, us, before (narrow for FP16, narrow or wide for FP32) / long:
//   FP16  15x128x19200 44.2 / 42.0   8x128x19200 27.2 / 26.0   15x64x19200 28.6 / 25.5   3x256x19200 22.1 / 20.7   60x128x1000
//         16.2 / 14.4   30x64x4800 16.9 / 15.4   20x30x4819 12.4 / 9.4
//   FP32  4x128x19200 26.2 / 25.6   15x64x9600 25.9 / 23.7   16x32x9600 20.7 / 15.8   3x134x6588 13.5 / 12.7   8x256x4800
//         26.7 / 25.0   4x256x9601 35.8 / 32.8
// FP16 loses where the tiles are few and uneven over the compute units (tiles of the launch: 300, 2x128x19200 10.8 / 12.0;
// 304, 8x256x4800 16.5 / 19.6; 600, 4x128x19200 15.8 / 16.5; but 450, 3x128x19200 13.25 / 13.0 and 480, 60x128x1000), less so with
// few channels (608, 16x64x4800 11.1 / 11.0; 600, 4x32x19200 9.3 / 8.4).  Both lose where the last tile of an image is half
// empty and images are short (400x128x129 FP16 20.6 / 26.7, 400x128x96 FP32 15.2 / 16.7), with few channels from shorter images on
// (200x16x400 FP16 9.4 / 7.9, 200x32x200 FP32 10.3 / 8.5).  FP32 off the grid with 65 to 128 channels, whose wide
// tiles go two to a compute unit, stays with those (12x100x4819 20.6 / 22.7), and so do few tiles of the most channels
// (450, 3x256x9600 19.9 / 20.2).
//
// Nor, for FP16 with 193 to 256 channels (or 129 to 192), where rows are whole cache lines and the tiles are more than two to a
// compute unit: against the narrow ones a median of 1.03 (1.06) without a gradient and 0.99 with one over two thousand pairs, worst
// 1.12 (1.17).  Nor without a gradient where images have an odd number of positions, or twice an odd one, and the tiles are few, with 97
// to 128 and 193 to 256 channels (long against narrow, median and worst, tiles of the launch: up to 512 1.035 and 1.12, up to
// 1024 0.99 and 1.12, up to 1536 1.00 and 1.12, beyond 0.95 and 1.03; 4x180x15730, 492, 16.0 / 17.0).  Nor with a gradient in such
// images where the tiles are fewer than two to a compute unit: median and worst with 97 to 128 channels 1.025 and 1.18
// (23x115x2435, 460, 18.7 / 21.4), 129 to 160 1.02 to 1.04 and 1.18, with more channels in images of up to 56 tiles 1.01 to 1.08 and 1.19; longer images of
// more than 160 channels gain, 0.97 (6x243x9999, 474, 35.4 / 38.4, is one that loses).  These look at nothing but the
// extents and the type, so that a workspace serves the pair at any alignment.
bool long_pays(const fq_distill *d, bool quads, long long narrow_tpn, long long wide_tpn, bool grad)
{
    const int kch = fused_channels_per_lane(d, kLong);
    if (!kch || (2 * wide_tpn - narrow_tpn) * (kch <= 2 ? 4 : 16) > narrow_tpn) return false;
    const long long tiles = wide_tpn * d->n, rounds = (tiles + kComputeUnits - 1) / kComputeUnits;
    if (d->dtype == FQ_F32) return (quads || kch != 4) && (kch < 8 || tiles >= 2 * kComputeUnits);
    if (kch >= 12 && d->inner % 64 == 0 && tiles > 2 * kComputeUnits) return false;
    if (!grad && (kch == 8 || kch == 16) && d->inner % kFusedVec != 0 && tiles < 6 * kComputeUnits) return false;
    if (grad && d->inner % kFusedVec != 0 && tiles < 2 * kComputeUnits &&
        (kch == 8 || (kch > 8 && (d->channels <= 160 || wide_tpn <= 56)))) return false;
    return 8 * tiles >= 7 * rounds * kComputeUnits || tiles >= (kch <= 4 ? 2 : kch <= 8 ? 4 : 7) * kComputeUnits;
}

// Where long tiles pay: with few channels the same rows by 256 threads, twice the channels per lane.  us, long / small:
//   FP16  16x32x9600 11.1 / 10.7   60x24x2000 9.3 / 8.9   30x16x19200 22.6 / 18.5   64 channels: no difference
//   FP32  16x16x4800 8.45 / 7.3   60x48x1200 13.5 / 12.8   15x64x9600 23.7 / 23.0
// Off the grid, and in smaller launches, with the fewest channels only (10x64x4819 FP32 11.9 / 12.2, 20x30x4819 FP16 9.4 /
// 10.0, 8x64x4800 FP32 9.5 / 9.9; but 30x30x2411 FP32 11.3 / 10.5).
bool small_pays(const fq_distill *d, bool quads, long long tiles)
{
    const int kch = fused_channels_per_lane(d, kSmall);
    return kch && (kch <= 2 || (quads && tiles >= 2 * kComputeUnits));
}

// Where rows of 256 bytes pay, but by 1024 threads: with half the channels per lane.  long against wide, time over that of the
// tiles that the other rule below would take, median and worst of a few hundred pairs each:
//   without a gradient  FP32 with 193 to 256 channels, any alignment 1.00 to 1.03 and 1.11 / 0.98 to 0.995 and 1.03 (15x249x11944
//     71.0 / 67.0 us); FP16 with 129 to 192 0.95 to 1.05 and 1.14 / 0.92 to 0.96 and 1.05, with 193 to 256 on the grid
//     0.93 to 1.00 and 1.05 / 0.90 to 0.97 and 1.00 (off it 0.95 and 1.1 / 1.08 and 1.19)
//   with one  FP32 on the grid with 65 to 128 or 193 to 256 channels, rows no whole number of 64-byte halves of a line and launches of
//     many tiles 1.02 and 1.09 / 0.99 and 1.01 (smaller ones 0.97 / 0.99); off the grid with 193 to 256, in the largest 0.99 and 1.08 / 0.99
//     and 1.00 (smaller ones 0.93 / 0.99).  14x234x17044 203 / 190 us, 8x81x38440 81 / 77.6, 13x254x19507 229 / 216.  Off the grid with 57
//     to 64, which fill the 64 rows of 1024 threads, and many elements, in millions, median and worst: 14 to 16 1.00 and 1.03 / 0.984 and
//     0.99, 20 to 22 1.02 and 1.06, 28 to 30 1.04 and 1.07 / the same 0.984 and 0.99 (10x60x39795 83.9 / 78.6); fewer channels gain up to 26 million
//     and are level beyond
constexpr long long kManyElements = 6400000, kMostElements = 33000000, kFewChannelsElements = 14000000;
bool by_1024_threads(const fq_distill *d, bool quads, bool grad)
{
    const int kch = fused_channels_per_lane(d, kLong);
    if (d->dtype == FQ_F16) return !grad && (kch == 12 || (kch == 16 && quads));
    if (!grad) return kch == 8;
    const long long elements = d->n * d->channels * d->inner;
    if (quads) return (kch == 4 || kch == 8) && d->inner % 16 != 0 && elements > kManyElements;
    return (kch == 8 && elements > kMostElements) || (kch == 2 && d->channels > 56 && elements > kFewChannelsElements);
}

// Where they don't: wide tiles, 1024 threads, for FP32 (us, narrow / wide: 3x384x19200 61 / 55, 12x100x4819 25.8 /
// 20.6; a wide FP16 tile fills a compute unit by itself, with nothing to stream while it reduces: 15x256x19200 85 / 95).
// Not where the narrow ones are all resident at once and the wide ones need a second round (on the grid; its registers
// let a compute unit hold 4, 3 or 2 narrow tiles, 2 or 1 wide ones; 150x384x96 15.5 / 17.2).
// Nor where the last wide tile of an image is half empty and images are short: on the grid if more than a
// sixteenth of the wide tiles' positions lie behind the image (400x128x96 15.3 / 17.2, 150x384x288 37.6 / 40.6,
// 400x128x224 27.7 / 28.9), off it, where wide rows share fewer lines (400x128x129 29.3 / 24.1), if they are
// as many as the narrow ones (1000x128x9 11.4 / 15.6; on the grid 4000x128x4 22.6 / 36.4, 3000x24x32 13.9 / 21.7).
bool wide_pays(const fq_distill *d, bool quads, long long narrow_tpn, long long wide_tpn, int kch)
{
    const long long held_narrow = kch <= 2 ? 4 : kch <= 4 ? 3 : 2, held_wide = kch <= 2 ? 2 : 1;
    const bool second_round = quads && narrow_tpn * d->n <= held_narrow * kComputeUnits &&
                              wide_tpn * d->n > held_wide * kComputeUnits;
    const bool half_empty = quads ? 16 * (2 * wide_tpn - narrow_tpn) > narrow_tpn : wide_tpn == narrow_tpn;
    return d->dtype == FQ_F32 && !second_round && !half_empty;
}

fq_status make_plan(const fq_distill *d, Plan &pl)
{
    if (!d) return FQ_ERR_NULL;
    if (d->dtype != FQ_F16 && d->dtype != FQ_F32) return FQ_ERR_DTYPE;
    if (d->n < 0 || d->channels < 0 || d->inner < 0) return FQ_ERR_SHAPE;
    const size_t esz = d->dtype == FQ_F16 ? 2 : 4;
    // positions index 32-bit grids of 64-lane tiles; the element count must fit in 62 bits
    if (d->n > 0 && d->inner > (long long)0x7fffffff / d->n) return FQ_ERR_SHAPE;
    const long long P = d->n * d->inner;
    if (d->channels > 0x7fffffff) return FQ_ERR_SHAPE;
    if (P > 0 && d->channels > ((long long)1 << 60) / P) return FQ_ERR_SHAPE;
    if (!(d->lambda == d->lambda) || !(d->upstream == d->upstream) || !(d->eps >= 0.0f)) return FQ_ERR_SCALE_PARAMS;
    if (!d->out) return FQ_ERR_NULL;
    if ((uintptr_t)d->out % sizeof(double)) return FQ_ERR_ALIGN;
    const bool empty = P == 0 || d->channels == 0;
    if (!empty) {
        if (!d->student || !d->teacher) return FQ_ERR_NULL;
        if ((uintptr_t)d->student % esz || (uintptr_t)d->teacher % esz || (uintptr_t)d->gstudent % esz)
            return FQ_ERR_ALIGN;
        if (d->gstudent) {
            // exact in-place over the student is fine (each element is read before it is written
            // by the same lane); any other overlap is not
            const char *g0 = (const char *)d->gstudent, *g1 = g0 + (size_t)P * d->channels * esz;
            const void *ins[2] = {d->student, d->teacher};
            for (const void *in : ins) {
                const char *i0 = (const char *)in, *i1 = i0 + (size_t)P * d->channels * esz;
                if (g0 != i0 && g0 < i1 && i0 < g1) return FQ_ERR_ALIAS;
            }
        }
    }
    pl = Plan{};
    if (empty) {
        pl.vec = 1;
        pl.bytes = 256;
        return FQ_OK;
    }
    pl.fused_kch = fused_channels_per_lane(d, kNarrow);
    if (pl.fused_kch) {
        pl.quads = on_quads(d);
        const long long narrow = tile_positions(d, kNarrow);
        const long long narrow_tpn = (d->inner + narrow - 1) / narrow, wide_tpn = (d->inner + 2 * narrow - 1) / (2 * narrow);
        const long long wide_tiles = wide_tpn * d->n;
        const bool grad = d->gstudent != nullptr;
        pl.shape = kNarrow;
        if (narrow_tpn * d->n > (long long)kGatherTiles) {
            if (wide_tiles <= (long long)kGatherTiles) pl.shape = kWide;     // one launch (1x384x19200 FP16: 15.9 -> 12.6 us)
            else if (long_pays(d, pl.quads, narrow_tpn, wide_tpn, grad))
                pl.shape = small_pays(d, pl.quads, wide_tiles) ? kSmall : by_1024_threads(d, pl.quads, grad) ? kWide : kLong;
            else if (wide_pays(d, pl.quads, narrow_tpn, wide_tpn, pl.fused_kch)) pl.shape = kWide;
        }
        if (pl.shape != kNarrow) pl.fused_kch = fused_channels_per_lane(d, pl.shape);
        const long long tpn = pl.shape != kNarrow ? wide_tpn : narrow_tpn;
        pl.one_launch = tpn * d->n <= (long long)kGatherTiles;
        if (tpn * d->n > 0x3fffffffLL) return FQ_ERR_SHAPE;
        pl.vec = kFusedVec;
        pl.tiles_per_n = (unsigned)tpn;
        pl.tiles = (unsigned)(tpn * d->n);
        pl.groups = pl.per_group = pl.grad_groups = pl.grad_per_group = 0;
        pl.stats_lds = 0;
        pl.off_blocksum = 0;                       // no per-position coefficients leave the block
        // A workspace serves the pair with its gradient and without: where one of the two has narrow tiles, room for those.
        const long long most = d->dtype == FQ_F16 && !pl.one_launch && !long_pays(d, pl.quads, narrow_tpn, wide_tpn, !grad)
                                   ? narrow_tpn * d->n : (long long)pl.tiles;
        pl.bytes = pl.one_launch ? align256(((size_t)pl.tiles * 4 + 1) * sizeof(unsigned long long))
                           : align256((size_t)most * 2 * sizeof(double));
        if (pl.bytes < 256) pl.bytes = 256;
        return FQ_OK;
    }
    const int full = (int)(kVecBytes / esz) < kMaxVec ? (int)(kVecBytes / esz) : kMaxVec;
    // Elements per lane: the widest load whose tiles (64 lanes x vec positions) are still many
    // enough to fill the chip without splitting the channels into many groups; a narrow load
    // still covers whole cache lines (64 lanes x 4 bytes = two lines).
    const uintptr_t addr_bits = (uintptr_t)d->student | (uintptr_t)d->teacher | (uintptr_t)d->gstudent;
    pl.vec = 1;
    for (int v = full; v > 1; v /= 2) {
        if (d->inner % v || addr_bits % (v * esz)) continue;
        pl.vec = v;
        if (d->n * ((d->inner + 64LL * v - 1) / (64LL * v)) >= kMinTiles) break;
    }
    const long long per_tile = 64LL * pl.vec;
    const long long tpn = empty ? 0 : (d->inner + per_tile - 1) / per_tile;
    if (tpn * d->n > 0x3fffffffLL) return FQ_ERR_SHAPE;
    pl.tiles_per_n = (unsigned)tpn;
    pl.tiles = (unsigned)(tpn * d->n);
    auto split = [&](unsigned want_waves, unsigned cap, unsigned &groups, unsigned &per_group) {
        unsigned g = pl.tiles ? (want_waves + pl.tiles - 1) / pl.tiles : 1u;
        if (g > cap) g = cap;
        if (g > (unsigned)d->channels) g = (unsigned)d->channels;
        if (g < 1u) g = 1u;
        per_group = empty ? 0u : ((unsigned)d->channels + g - 1) / g;
        groups = per_group ? ((unsigned)d->channels + per_group - 1) / per_group : 1u;
    };
    split(kTargetWaves, kMaxGroups, pl.groups, pl.per_group);
    split(2 * kTargetWaves, 1024u, pl.grad_groups, pl.grad_per_group);
    if ((unsigned long long)pl.tiles * pl.grad_groups > 0x3fffffffULL) {
        pl.grad_groups = pl.groups;
        pl.grad_per_group = pl.per_group;
    }
    unsigned pow2 = 1;
    while (pow2 < pl.groups) pow2 *= 2;
    unsigned slots = pow2 > 1 ? pow2 / 2 : 1;
    if (slots > kTreeSlots) slots = kTreeSlots;
    pl.stats_lds = (size_t)slots * 4 * pl.vec * 64 * sizeof(double);
    const size_t coef = align256((size_t)P * 2 * sizeof(double));
    const size_t blocksum = align256((size_t)pl.tiles * 2 * sizeof(double));
    pl.off_blocksum = coef;
    pl.bytes = coef + blocksum;
    if (pl.bytes < 256) pl.bytes = 256;
    return FQ_OK;
}

__global__ void distill_empty_kernel(double *out, bool has_positions)
{
    // a mean over no elements is 0/0; positions without channels have cos = 0 / eps^2 = 0
    const double nan = __builtin_nan("");
    out[0] = nan;
    out[1] = has_positions ? 0.0 : nan;
    out[2] = nan;
}

template <typename T, int V>
fq_status launch(const DistillArgs &k, const Plan &pl, bool want_grad, hipStream_t st)
{
    distill_stats_kernel<T, V><<<pl.tiles, 64 * pl.groups, pl.stats_lds, st>>>(k);
    if (want_grad) {
        const unsigned grad_blocks = (pl.tiles * pl.grad_groups + kWaves - 1) / kWaves;
        distill_grad_kernel<T, V><<<grad_blocks, kThreads, 0, st>>>(k, pl.grad_groups, pl.grad_per_group);
        if (launch_fill_zero(k.coef, pl.bytes, st) != 0) return FQ_ERR_LAUNCH;
    } else {
        distill_finish_kernel<<<1, 1024, 0, st>>>(k);
    }
    return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_LAUNCH;
}

template <typename T, int SHAPE, int KCH, bool QUADS>
fq_status launch_fused(const DistillArgs &k, const Plan &pl, bool want_grad, hipStream_t st)
{
    const Divisor by = divisor(pl.tiles_per_n);
    const auto kernel = want_grad ? distill_fused_kernel<T, SHAPE, KCH, QUADS, true> : distill_fused_kernel<T, SHAPE, KCH, QUADS, false>;
    kernel<<<pl.tiles, kTileThreads[SHAPE], 0, st>>>(k.a, k.b, k.M, k.C, k.tiles_per_n, by.multiplier,
                                                     by.shift1 | (unsigned)by.shift2 << 16, pl.neighbours ? pl.tiles : 0u, k);
    if (!pl.one_launch) distill_finish_kernel<<<1, 1024, 0, st>>>(k);
    return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_LAUNCH;
}

template <typename T, int SHAPE, int KCH>
fq_status launch_fused(const DistillArgs &k, const Plan &pl, bool want_grad, hipStream_t st)
{
    return pl.quads ? launch_fused<T, SHAPE, KCH, true>(k, pl, want_grad, st) : launch_fused<T, SHAPE, KCH, false>(k, pl, want_grad, st);
}

template <typename T, int SHAPE>
fq_status launch_fused(const DistillArgs &k, const Plan &pl, bool want_grad, hipStream_t st)
{
    constexpr int most = most_channels_per_lane<T>(SHAPE);
    switch (pl.fused_kch) {
    case 2: return launch_fused<T, SHAPE, 2>(k, pl, want_grad, st);
    case 4: return launch_fused<T, SHAPE, 4>(k, pl, want_grad, st);
    case 6: if constexpr (most >= 6) return launch_fused<T, SHAPE, 6>(k, pl, want_grad, st); else break;
    case 8: if constexpr (most >= 8) return launch_fused<T, SHAPE, 8>(k, pl, want_grad, st); else break;
    case 12: if constexpr (most >= 12) return launch_fused<T, SHAPE, 12>(k, pl, want_grad, st); else break;
    case 16: if constexpr (most >= 16) return launch_fused<T, SHAPE, 16>(k, pl, want_grad, st); else break;
    }
    return FQ_ERR_SHAPE;                           // not reached: make_plan offers only the widths above
}

template <typename T>
fq_status launch_fused(const DistillArgs &k, const Plan &pl, bool want_grad, hipStream_t st)
{
    switch (pl.shape) {
    case kWide: return launch_fused<T, kWide>(k, pl, want_grad, st);
    case kLong: return launch_fused<T, kLong>(k, pl, want_grad, st);
    case kSmall: return launch_fused<T, kSmall>(k, pl, want_grad, st);
    default: return launch_fused<T, kNarrow>(k, pl, want_grad, st);
    }
}

// A number that no other call of this process has, and that memory does not hold by chance: a counter from
// an arbitrary start through a mixing function that is one-to-one (splitmix64's).
unsigned long long next_nonce()
{
    static std::atomic<unsigned long long> counter{
        (unsigned long long)std::chrono::steady_clock::now().time_since_epoch().count() * 0x9e3779b97f4a7c15ull ^
        (unsigned long long)(uintptr_t)&counter};
    for (;;) {
        unsigned long long z = counter.fetch_add(0x9e3779b97f4a7c15ull, std::memory_order_relaxed);
        z = (z ^ (z >> 30)) * 0xbf58476d1ce4e5b9ull;
        z = (z ^ (z >> 27)) * 0x94d049bb133111ebull;
        z ^= z >> 31;
        if (z != 0ull && ~z != 0ull) return z;     // 0 is an empty flag
    }
}

}  // namespace
}  // namespace fq

extern "C" {

int fq_distill_reads_of_pair(const fq_distill *d)
{
    fq::Plan pl;
    if (fq::make_plan(d, pl) != FQ_OK) return 0;
    if (d->n * d->inner == 0 || d->channels == 0) return 0;
    return pl.fused_kch && pl.quads ? 1 : (d->gstudent ? 2 : 1);
}

size_t fq_distill_workspace_bytes(const fq_distill *d)
{
    fq::Plan pl;
    return fq::make_plan(d, pl) == FQ_OK ? pl.bytes : 0;
}

static fq_status distill_loss(const fq_distill *d, void *workspace, size_t ws_bytes, void *hip_stream, unsigned poll_rounds)
{
    using namespace fq;
    Plan pl;
    const fq_status v = make_plan(d, pl);
    if (v != FQ_OK) return v;
    hipStream_t st = (hipStream_t)hip_stream;
    if (d->n * d->inner == 0 || d->channels == 0) {
        distill_empty_kernel<<<1, 1, 0, st>>>(d->out, d->n * d->inner != 0);
        return hipGetLastError() == hipSuccess ? FQ_OK : FQ_ERR_LAUNCH;
    }
    if (!workspace || ws_bytes < pl.bytes) return FQ_ERR_WORKSPACE;
    if ((uintptr_t)workspace % 256) return FQ_ERR_ALIGN;

    DistillArgs k;
    k.a = d->student;
    k.b = d->teacher;
    k.ga = d->gstudent;
    k.coef = d->gstudent ? (double *)workspace : nullptr;
    k.blocksum = (double *)((char *)workspace + pl.off_blocksum);
    k.out = d->out;
    k.M = d->inner;
    k.P = d->n * d->inner;
    k.C = (unsigned)d->channels;
    k.groups = pl.groups;
    k.per_group = pl.per_group;
    k.tiles_per_n = pl.tiles_per_n;
    k.tiles = pl.tiles;
    const double ncm = (double)d->n * (double)d->channels * (double)d->inner;
    const double nm = (double)d->n * (double)d->inner;
    k.k1u = (double)d->upstream * (2.0 / ncm);
    k.k2u = (double)d->upstream * ((double)d->lambda / nm);
    k.eps = (double)d->eps;
    k.lambda = (double)d->lambda;
    k.inv_ncm = 1.0 / ncm;
    k.inv_nm = 1.0 / nm;
    const bool grad = d->gstudent != nullptr;
    k.records = (unsigned long long *)workspace;
    k.nonce = pl.one_launch ? next_nonce() : 0ull;
    k.poll_rounds = poll_rounds;
    pl.neighbours = pl.fused_kch && (!pl.quads || d->inner * (d->dtype == FQ_F16 ? 2 : 4) % 128 != 0);
    if (pl.fused_kch) {
        k.coef = nullptr;
        return d->dtype == FQ_F16 ? launch_fused<_Float16>(k, pl, grad, st) : launch_fused<float>(k, pl, grad, st);
    }
    if (d->dtype == FQ_F16) {
        switch (pl.vec) {
        case 4: return launch<_Float16, 4>(k, pl, grad, st);
        case 2: return launch<_Float16, 2>(k, pl, grad, st);
        default: return launch<_Float16, 1>(k, pl, grad, st);
        }
    }
    switch (pl.vec) {
    case 4: return launch<float, 4>(k, pl, grad, st);
    case 2: return launch<float, 2>(k, pl, grad, st);
    default: return launch<float, 1>(k, pl, grad, st);
    }
}

fq_status fq_distill_loss(const fq_distill *d, void *workspace, size_t ws_bytes, void *hip_stream)
{
    return distill_loss(d, workspace, ws_bytes, hip_stream, fq::kPollRounds);
}

fq_status fq_distill_loss_no_poll(const fq_distill *d, void *workspace, size_t ws_bytes, void *hip_stream)
{
    return distill_loss(d, workspace, ws_bytes, hip_stream, 0u);
}

}  // extern "C"
