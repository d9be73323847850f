// gfx950 kernels for fused learnable-scale fake quantization (DPVO-QAT++ Sec. 3.2, Eq. (3)-(6),
// and the straight-through backward stated next to Eq. (5)).
//
// The work is HBM-bound elementwise traffic plus one per-channel reduction, so there is no MFMA
// here.  Each 256-thread block owns one chunk (at most 20 KiB of input) that lies inside a single
// [outer, channel] slab, so the scale is uniform over the block; lanes move 128-bit vectors
// (global_load/store_dwordx4, non-temporal), FP16 is widened/narrowed in registers.  Backward adds
// a DPP wavefront reduction, an LDS block reduction and a fixed-order combination of the blocks
// of a channel (direct, by atomic exchange, or gathered by one of them: see combine); no float atomics.
// Tensors whose slabs are short are cut per wavefront instead (one slab per wavefront, four to a
// block, no barrier: forward_dispatch, backward_waves) when the launch has blocks to spare.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>
#include <type_traits>

#include "fq_device.h"
#include "fq_internal.h"

namespace fq {

using namespace dev;

namespace {

template <typename T> struct VecOf;
template <> struct VecOf<float> {
    static constexpr int N = 4;
    typedef float type __attribute__((ext_vector_type(4)));
};
template <> struct VecOf<_Float16> {
    static constexpr int N = 8;
    typedef _Float16 type __attribute__((ext_vector_type(8)));
};

constexpr int kMaxRows = kChunkVecs / kBlock;   // vectors per thread per chunk, at most
static_assert(kChunkVecs % kBlock == 0, "chunk must be a whole number of block-wide vector rows");

// ---------------------------------------------------------------------------------------------
// Eq. (3)-(4): s = clip(softplus(theta) + eps, s_min, s_max).  Evaluated in binary64 and rounded
// to binary32 once, so the value does not depend on the accuracy of a binary32 exp/log.
struct Scale {
    float s;             // Eq. (3)-(4)
    bool clip_active;    // the clamp changed the value (its derivative is then zero)
    double sigmoid;      // d softplus / d theta
};

// What a block needs of its channel's scale (see block_params).
struct BlockScale {
    double rd;           // RN64(1 / s)
    double sigmoid;
    float s;
    unsigned clip_active;
};

// exp(-a) for a >= 0 in binary64, a few ulp: a = n ln2 + r with |r| <= ln2/2 (two-constant
// reduction, n ln2_hi is exact), exp(-r) by its Taylor polynomial of degree 13 (remainder below
// 2^-57), scaled by 2^-n.  Short on purpose: it sits in every block's prologue.
__device__ __forceinline__ double exp_neg(double a)
{
    if (!(a < 746.0)) return a != a ? a : 0.0;                   // underflows to 0; NaN stays NaN
    const double n = __builtin_rint(a * 1.4426950408889634074);      // a / ln2
    double r = __builtin_fma(-n, 6.93147180369123816490e-01, a);     // ln2_hi, 21 trailing zero bits
    r = __builtin_fma(-n, 1.90821492927058770002e-10, r);            // ln2_lo
    const double x = -r;
    double p = 1.0 / 6227020800.0;                                     // 1/13!
    p = __builtin_fma(p, x, 1.0 / 479001600.0);
    p = __builtin_fma(p, x, 1.0 / 39916800.0);
    p = __builtin_fma(p, x, 1.0 / 3628800.0);
    p = __builtin_fma(p, x, 1.0 / 362880.0);
    p = __builtin_fma(p, x, 1.0 / 40320.0);
    p = __builtin_fma(p, x, 1.0 / 5040.0);
    p = __builtin_fma(p, x, 1.0 / 720.0);
    p = __builtin_fma(p, x, 1.0 / 120.0);
    p = __builtin_fma(p, x, 1.0 / 24.0);
    p = __builtin_fma(p, x, 1.0 / 6.0);
    p = __builtin_fma(p, x, 0.5);
    p = __builtin_fma(p, x, 1.0);
    p = __builtin_fma(p, x, 1.0);
    return __builtin_ldexp(p, -(int)n);
}

// log(1 + e) for 0 <= e <= 1 in binary64, a few ulp: 2 atanh(z) with z = e / (2 + e) <= 1/3,
// odd series up to z^35 (next term below 2^-58 of the sum).  No cancellation for small e.
__device__ __forceinline__ double log1p_unit(double e)
{
    const double z = e / (2.0 + e);
    const double w = z * z;
    double p = 1.0 / 35.0;
    p = __builtin_fma(p, w, 1.0 / 33.0);
    p = __builtin_fma(p, w, 1.0 / 31.0);
    p = __builtin_fma(p, w, 1.0 / 29.0);
    p = __builtin_fma(p, w, 1.0 / 27.0);
    p = __builtin_fma(p, w, 1.0 / 25.0);
    p = __builtin_fma(p, w, 1.0 / 23.0);
    p = __builtin_fma(p, w, 1.0 / 21.0);
    p = __builtin_fma(p, w, 1.0 / 19.0);
    p = __builtin_fma(p, w, 1.0 / 17.0);
    p = __builtin_fma(p, w, 1.0 / 15.0);
    p = __builtin_fma(p, w, 1.0 / 13.0);
    p = __builtin_fma(p, w, 1.0 / 11.0);
    p = __builtin_fma(p, w, 1.0 / 9.0);
    p = __builtin_fma(p, w, 1.0 / 7.0);
    p = __builtin_fma(p, w, 1.0 / 5.0);
    p = __builtin_fma(p, w, 1.0 / 3.0);
    p = __builtin_fma(p, w, 1.0);
    return 2.0 * z * p;
}

// softplus(t) = max(t,0) + log1p(e) and sigmoid(t) = (t >= 0 ? 1 : e) / (1 + e), e = exp(-|t|):
// one exponential serves both.  The binary64 value is rounded to binary32 once; a few ulp of
// binary64 error move that rounding with probability ~1e-8 per channel.
template <bool NEED_SIGMOID>
__device__ __forceinline__ Scale compute_scale(float theta, float eps, float s_min, float s_max)
{
    const double t = (double)theta;
    const double e = exp_neg(__builtin_fabs(t));
    const double u = __builtin_fmax(t, 0.0) + log1p_unit(e) + (double)eps;
    const float uf = (float)u;
    Scale r;
    r.clip_active = !(uf >= s_min && uf <= s_max);
    float v = uf;
    v = v < s_min ? s_min : v;
    v = v > s_max ? s_max : v;
    r.s = v;
    r.sigmoid = NEED_SIGMOID ? (t >= 0.0 ? 1.0 : e) / (1.0 + e) : 0.0;
    return r;
}

// ---------------------------------------------------------------------------------------------
// Per-element arithmetic.
//
// Quotient.  v must be the correctly rounded binary32 value of x/s.  It is formed as
// (float)((double)x * rd) with rd = RN64(1/s): three full-rate instructions instead of the ~10 of
// the IEEE binary32 division expansion.  This rounds exactly like x/s: writing x = X*2^a and
// s = S*2^b with 24-bit integers X, S, the exact quotient is never half-way between two binary32
// values and its distance from the nearest half-way point is at least 1/(2S) > 2^-25 ulp, i.e.
// more than 2^-49 relative, while the binary64 product carries a relative error below 2^-52; so
// the final rounding to binary32 sees the same side of every rounding boundary.  Infinities, NaN,
// signed zeros and overflow behave as in x/s.  (Only a quotient in the binary32 subnormal range,
// |v| < 2^-126, may differ by one subnormal ulp; its code is 0 either way.)
//
// Clip + round.  v_med3_f32 returns lo for a NaN quotient, so NaN is put back afterwards
// (the per-operator definition propagates it: clamp and round keep NaN).
struct QParams {
    double rd;      // RN64(1 / s)
    float s, lo, hi;
    int ilo, ihi;   // the same bounds as integers (for the int8 codes)
};

__device__ __forceinline__ float quotient(float x, const QParams &p) { return (float)((double)x * p.rd); }

// y = s * round(clip(v)) for a quotient known not to be NaN (the clip would turn NaN into lo)
__device__ __forceinline__ float fq_value_finite(float v, const QParams &p)
{
    return __builtin_rintf(__builtin_amdgcn_fmed3f(v, p.lo, p.hi)) * p.s;
}

// forward value y = s * round(clip(v)); a NaN quotient gives NaN
__device__ __forceinline__ float fq_value(float v, const QParams &p)
{
    float q = __builtin_rintf(__builtin_amdgcn_fmed3f(v, p.lo, p.hi));
    float y = q * p.s;
    return v != v ? v : y;
}

// integer code clip(round(v)) (the same as round(clip(v)) for integer bounds), 0 for a NaN
// quotient.  v_cvt_i32_f32 itself maps NaN to 0 and saturates +-Inf and huge values, so no
// select is needed; it is written as an instruction because the C conversion of NaN/Inf is
// undefined.
__device__ __forceinline__ int fq_code(float v, const QParams &p)
{
    int c;
    asm("v_cvt_i32_f32 %0, %1" : "=v"(c) : "v"(__builtin_rintf(v)));
    c = c < p.ilo ? p.ilo : c;
    c = c > p.ihi ? p.ihi : c;
    return c;
}

// low bytes of four ints -> one dword (v_perm_b32 twice + or)
__device__ __forceinline__ unsigned pack_codes4(int c0, int c1, int c2, int c3)
{
    const unsigned lo = __builtin_amdgcn_perm((unsigned)c1, (unsigned)c0, 0x0c0c0400u);
    const unsigned hi = __builtin_amdgcn_perm((unsigned)c3, (unsigned)c2, 0x04000c0cu);
    return lo | hi;
}

// backward: returns t = dy/ds and whether the quotient is inside [lo, hi] (inclusive).
// in range: t = rint(v) - v;  below: lo;  above: hi;  NaN quotient: out of range, t = NaN.
__device__ __forceinline__ float ste_terms(float x, const QParams &p, bool &in_range, bool &is_nan)
{
    float v = quotient(x, p);
    float cl = __builtin_amdgcn_fmed3f(v, p.lo, p.hi);
    in_range = cl == v;                       // false for NaN
    is_nan = v != v;
    float r = __builtin_rintf(cl);            // the bound itself when clipped
    return r - (in_range ? v : 0.0f);
}

// Hold the wavefront until every vector memory operation it has issued (loads, stores, atomics)
// has been acknowledged; the "memory" clobber keeps the compiler from moving accesses across it.
__device__ __forceinline__ void wait_stores_acknowledged() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

// Collector side of the partial sums.  They are read with agent-scope atomic loads (global_load ...
// sc1), which are served from the level all XCDs share and never from a line cached by this XCD.
// This keeps the compiler from moving such reads to the other side of a publication.  (An acquire
// fence at agent scope would also invalidate this XCD's L2 under the blocks still streaming
// through it: measured 41 -> 45 us on a 15x128x120x160 FP16 tensor, for nothing.)
__device__ __forceinline__ void order_accesses() { asm volatile("" ::: "memory"); }

// Keeps the computation of a value at this point of the program: the compiler would otherwise
// sink it to its first use, behind the wait for a later load.  Emits no instruction.
__device__ __forceinline__ void pin_here(float &v) { asm volatile("" : "+v"(v)); }
__device__ __forceinline__ void pin_here(unsigned &v) { asm volatile("" : "+v"(v)); }

// Index of this wavefront in its block as a scalar: telling the compiler that it is uniform keeps
// everything derived from it (the unit's slab, channel, pointers, loop bounds) in SGPRs.
__device__ __forceinline__ unsigned wave_index() { return (unsigned)__builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6)); }

// ---------------------------------------------------------------------------------------------
// Chunk addressing shared by forward and backward.
struct Chunk {
    unsigned slab, channel;
    unsigned j;        // index of this unit among its channel's units
    long long first;   // flat element index of the chunk's first element
    int n;             // elements in the chunk
};

__device__ __forceinline__ Chunk locate_chunk(const DevTensor &d, unsigned local_block)
{
    Chunk c;
    c.slab = divide(local_block, d.by_cps);
    unsigned k = local_block - c.slab * d.cps;
    const unsigned o = divide(c.slab, d.by_channels);
    c.channel = c.slab - o * d.channels;
    c.j = o * d.cps + k;
    long long e0 = (long long)k * d.chunk;
    long long rem = d.inner - e0;
    c.n = rem < (long long)d.chunk ? (int)rem : (int)d.chunk;
    c.first = (long long)c.slab * d.inner + e0;
    return c;
}

// The chunk of this block in a single-tensor launch.  Such a launch normally has a grid of
// (chunks per slab, channels, outer), which names the chunk without any division (two integer
// divisions sit between a block's start and its first load otherwise); tensors with more than
// 65535 channels or outer slices keep the linear grid.
__device__ __forceinline__ Chunk own_chunk(const DevTensor &d)
{
    if (!d.grid3) return locate_chunk(d, blockIdx.x);
    Chunk c;
    c.channel = blockIdx.y;
    c.slab = blockIdx.z * d.channels + blockIdx.y;
    c.j = blockIdx.z * d.cps + blockIdx.x;
    const long long e0 = (long long)blockIdx.x * d.chunk;
    const long long rem = d.inner - e0;
    c.n = rem < (long long)d.chunk ? (int)rem : (int)d.chunk;
    c.first = (long long)c.slab * d.inner + e0;
    return c;
}

// elements before the first 16-byte boundary of p
template <typename T> __device__ __forceinline__ int head_elems(const void *p, int n)
{
    int h = (int)(((kVecBytes - ((uintptr_t)p & (kVecBytes - 1))) & (kVecBytes - 1)) / sizeof(T));
    return h < n ? h : n;
}

// The elements of a chunk that no whole vector covers: `head` of them before the first 16-byte
// boundary and the rest behind the last whole vector, fewer than two vectors in all.  Lane i < count
// takes the i-th of them.  They are read together with the vectors, because reading them afterwards
// adds one dependent trip to memory for either end to every misaligned chunk (3x131x4819 FP16: forward
// 4.3 us against 3.6, backward 7.15 against 6.1).
// They stay bit patterns in a register of their own (pin_here) until the vectors are done: the compiler
// would otherwise convert them where they are read, and wait for them there.
struct Edges {
    int count;     // 0 also where nothing can be read as vectors (the caller then goes element by element)
    int skip;      // elements covered by the vectors

    __device__ __forceinline__ int at(int lane, int head) const { return lane < head ? lane : skip + lane; }
};

__device__ __forceinline__ unsigned ld_bits(const float *p) { return ld_global((const unsigned *)p); }
__device__ __forceinline__ unsigned ld_bits(const _Float16 *p) { return ld_global((const unsigned short *)p); }
template <typename T> __device__ __forceinline__ T from_bits(unsigned b)
{
    typedef typename std::conditional<sizeof(T) == 2, unsigned short, unsigned>::type U;
    return __builtin_bit_cast(T, (U)b);
}

// Scale of this group's channel (G = 256 or 512: the block; G = 64: one wavefront).  Callers issue their
// first global loads before this, so the evaluation sits in the shadow of the memory latency.
// A block lets one wavefront (rotating with the block index, so the work spreads over the four
// SIMDs of a compute unit) evaluate Eq. (3)-(4), about a hundred binary64 instructions, and the
// others read it from LDS after a barrier; a lone wavefront evaluates it for itself.  G = 0: `group`
// says which, uniformly over the block.
template <bool NEED_SIGMOID, int G>
__device__ __forceinline__ QParams block_params(const DevTensor &d, float theta, BlockScale &bs, int group = G)
{
    if (group == 64) {
        const Scale sc = compute_scale<NEED_SIGMOID>(theta, d.eps, d.s_min, d.s_max);
        bs.s = sc.s;
        bs.rd = 1.0 / (double)sc.s;
        bs.sigmoid = sc.sigmoid;
        bs.clip_active = sc.clip_active ? 1u : 0u;
    } else {
        __shared__ BlockScale shared_scale;
        // (the sum of the indices, not the linear index: that takes the grid's extents, one more load)
        if ((threadIdx.x >> 6) == ((blockIdx.x + blockIdx.y + blockIdx.z) & ((G ? G : kBlock) / 64 - 1))) {
            const Scale sc = compute_scale<NEED_SIGMOID>(theta, d.eps, d.s_min, d.s_max);
            if ((threadIdx.x & 63) == 0) {
                shared_scale.s = sc.s;
                shared_scale.rd = 1.0 / (double)sc.s;
                shared_scale.sigmoid = sc.sigmoid;
                shared_scale.clip_active = sc.clip_active ? 1u : 0u;
            }
        }
        __syncthreads();
        bs = shared_scale;
    }
    QParams p;
    p.rd = bs.rd;
    p.s = bs.s;
    p.lo = d.lo;
    p.hi = d.hi;
    p.ilo = (int)d.lo;
    p.ihi = (int)d.hi;
    return p;
}

// ---------------------------------------------------------------------------------------------
// Forward.
template <typename T, bool WRITE_Y, bool EMIT_Q>
__device__ __forceinline__ void forward_elem(T x, T *y, int8_t *q, int i, const QParams &p)
{
    const float v = quotient((float)x, p);
    if (WRITE_Y) st_global(y + i, (T)fq_value(v, p));
    if (EMIT_Q) st_global(q + i, (int8_t)fq_code(v, p));
}

// WRITE_Y: write the dequantized tensor y.  EMIT_Q: write the int8 codes, N per lane packed into
// one 64-bit (FP16 input) or 32-bit (FP32 input) store.  At least one of the two.
// G: lanes that share the chunk.
// EARLY: theta is requested in front of the rows, and all rows have to be there when the scale is.  That is
// for launches of more than three blocks per compute unit, where some compute units get more blocks than others and
// blocks read while others write.  (Registers would let eight of these blocks reside on a compute unit: what
// counts is how evenly a launch fills the chip, not whether it has to wait for room.)  Measured on buffers that no cache
// holds, us, without / with: 780x10240 FP16 (780 blocks) 7.8 / 7.6, 850x9600 (850) 8.0 / 7.7, 512x19200 FP16 (1024) 8.7 /
// 8.1, 8x64x19200 FP16 (1024) 8.4 / 7.7, 15x128x19200 FP16 (3840) 26.35 / 25.9, 2x384x19200 FP32 (3072) 21.1 / 20.8, 64
// mixed tensors of 1 GiB forward + backward 930 / 918; but 384x19200 FP16 (768 blocks) 6.4 / 6.7, one scale 2457600 FP16
// (240) 3.7 / 4.2, and wavefront units 15x384x1200 FP16 6.99 / 7.07.  (The backward gains nothing by it: 384x19200 FP16
// 9.1 / 9.8.)
template <typename T, bool WRITE_Y, bool EMIT_Q, int G, int ROWS, bool EARLY>
__device__ __forceinline__ void forward_chunk(const DevTensor &d, const Chunk &ck)
{
    typedef typename VecOf<T>::type VT;
    constexpr int N = VecOf<T>::N;
    typedef unsigned QV __attribute__((ext_vector_type(N / 4)));
    const T *x = (const T *)d.x + ck.first;
    T *y = WRITE_Y ? (T *)d.y + ck.first : nullptr;
    int8_t *q = EMIT_Q ? d.q + ck.first : nullptr;
    const int tid = threadIdx.x & (G - 1);
    const float theta = EARLY ? ld_early(d.theta + ck.channel) : ld_uniform(d.theta + ck.channel);

    const bool vector_ok = !WRITE_Y || (((uintptr_t)x ^ (uintptr_t)y) & (kVecBytes - 1)) == 0;
    const int head = vector_ok ? head_elems<T>(x, ck.n) : ck.n;
    const int nvec = (ck.n - head) / N;
    const VT *xv = (const VT *)(x + head);
    VT *yv = WRITE_Y ? (VT *)(y + head) : nullptr;
    const bool q_packed = EMIT_Q && ((uintptr_t)(q + head) % N) == 0;
    const Edges edges = {vector_ok ? ck.n - nvec * N : 0, nvec * N};

    // Issue the first row of loads (straight-line: out-of-range lanes re-read the last vector)
    // before the long binary64 scale evaluation, which then runs under the memory latency.
    VT r[ROWS];
    if (nvec > 0) {
        const int last = nvec - 1;
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            int v = u * G + tid;
            r[u] = ld_stream(xv + (v < last ? v : last));
        }
    }
    unsigned ex = 0u;
    if (tid < edges.count) ex = ld_bits(x + edges.at(tid, head));

    BlockScale bs;
    const QParams p = block_params<false, G>(d, theta, bs);
    if (d.s && ck.first == (long long)ck.channel * d.inner && tid == 0) st_global(d.s + ck.channel, p.s);

#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        const int v = u * G + tid;
        if (v < nvec) {
            float quot[N];
#pragma unroll
            for (int e = 0; e < N; ++e) quot[e] = quotient((float)r[u][e], p);
            if (WRITE_Y) {
                // A NaN quotient must come out as NaN, and the clip swallows it.  Instead of a
                // compare and a select per element, the row's quotients are tested in pairs
                // (one unordered compare sees a NaN in either operand) and only a lane that
                // has found one goes back over its row.
                VT o;
                bool any_nan = false;
#pragma unroll
                for (int e = 0; e < N; e += 2) any_nan |= __builtin_isunordered(quot[e], quot[e + 1]);
#pragma unroll
                for (int e = 0; e < N; ++e) o[e] = (T)fq_value_finite(quot[e], p);
                if (__builtin_expect(any_nan, 0)) {
                    asm volatile("" ::: "memory");       // keep this a branch: it is almost never taken
#pragma unroll
                    for (int e = 0; e < N; ++e) o[e] = (T)fq_value(quot[e], p);
                }
                st_stream(yv + v, o);
            }
            if (EMIT_Q) {
                int c[N];
#pragma unroll
                for (int e = 0; e < N; ++e) c[e] = fq_code(quot[e], p);
                if (q_packed) {
                    QV codes;
#pragma unroll
                    for (int g = 0; g < N / 4; ++g)
                        codes[g] = pack_codes4(c[4 * g], c[4 * g + 1], c[4 * g + 2], c[4 * g + 3]);
                    st_stream((QV *)(q + head + v * N), codes);
                } else {
#pragma unroll
                    for (int e = 0; e < N; ++e) st_global(q + head + v * N + e, (int8_t)c[e]);
                }
            }
        }
    }

    pin_here(ex);
    if (tid < edges.count) forward_elem<T, WRITE_Y, EMIT_Q>(from_bits<T>(ex), y, q, edges.at(tid, head), p);
    if (!vector_ok) {               // x and y are misaligned relative to each other
        for (int i = tid; i < ck.n; i += G) forward_elem<T, WRITE_Y, EMIT_Q>(ld_global(x + i), y, q, i, p);
    }
}

// what one tensor asks of the forward pass: y only, y and codes, or codes only
template <typename T, int G, bool EARLY>
__device__ __forceinline__ void forward_variants(const DevTensor &d, unsigned unit)
{
    const Chunk ck = locate_chunk(d, unit);
    if (!d.q) forward_chunk<T, true, false, G, kMaxRows, EARLY>(d, ck);
    else if (d.y) forward_chunk<T, true, true, G, kMaxRows, EARLY>(d, ck);
    else forward_chunk<T, false, true, G, kMaxRows, EARLY>(d, ck);
}

// Tensors whose slabs are short (d.wave_units) give every wavefront a slab of its own: four
// slabs to a block, no barrier.  Otherwise the block owns one chunk.
template <typename T, bool EARLY>
__device__ __forceinline__ void forward_dispatch(const DevTensor &d, unsigned local_block)
{
    if (d.wave_units) {
        const unsigned unit = local_block * (kBlock / 64) + wave_index();
        if (unit < d.slabs * d.cps) forward_variants<T, 64, EARLY>(d, unit);
    } else {
        forward_variants<T, kBlock, EARLY>(d, local_block);
    }
}

// ---------------------------------------------------------------------------------------------
// Backward.
// gy*t is exact in binary64 (two 24-bit significands), so the per-channel sum differs from a
// sequential binary64 sum only by binary64 rounding, however badly the terms cancel.
template <typename T>
__device__ __forceinline__ double backward_elem(T x, T g, T *gx, int i, const QParams &p, double acc)
{
    bool in_range, is_nan;
    float t = ste_terms((float)x, p, in_range, is_nan);
    if (gx) st_global(gx + i, in_range ? g : (T)0.0f);
    acc = __builtin_fma((double)(float)g, (double)t, acc);
    return is_nan ? __builtin_nan("") : acc;
}

// Per-thread sum of gy*t over this thread's elements of the chunk (binary64).  GX: whether gx is
// written, kGxAsked: as the tensor's flags say.  G: lanes that share the chunk, 0: `group`, known at run
// time only.
enum { kGxNo = 0, kGxYes = 1, kGxAsked = 2 };

// The vectors of gx that a lane has worked out and not stored yet (bit patterns of either type).  Without gx none are
// worked out: what a lane holds then is never written or read.  (While they were, FP16 without gx was slower than with gx stored
// in front of the sum: 4x390x10074 15.0 / 15.2 / 14.8 us then, while, now; 5x209x34576 28.6 / 28.2 / 27.3.)
template <int ROWS> struct GxRows {
    typedef unsigned Bits __attribute__((ext_vector_type(4)));
    Bits v[ROWS];
    Bits *to;                  // nullptr: gx is not written
    int nvec, first, step;     // vector u of this lane is the chunk's (u * step + first)-th, if below nvec

    __device__ __forceinline__ void store() const
    {
        if (!to) return;
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const int i = u * step + first;
            if (i < nvec) st_stream(to + i, v[u]);
        }
    }
};
template <> struct GxRows<0> {         // gx is stored row by row, where it is worked out
    typedef unsigned Bits __attribute__((ext_vector_type(4)));
    __device__ __forceinline__ void store() const {}
};

template <typename T, int GX, int G, int ROWS, int HELD>
__device__ __forceinline__ double backward_chunk(const DevTensor &d, const Chunk &ck, BlockScale &bs, GxRows<HELD> &out,
                                                 const int group = G)
{
    typedef typename VecOf<T>::type VT;
    constexpr int N = VecOf<T>::N;
    const bool WRITE_GX = GX == kGxAsked ? !(d.flags & 1u) : GX == kGxYes;
    const T *x = (const T *)d.x + ck.first;
    const T *gy = (const T *)d.gy + ck.first;
    T *gx = WRITE_GX ? (T *)d.gx + ck.first : nullptr;
    const int tid = threadIdx.x & (group - 1);
    const float theta = ld_uniform(d.theta + ck.channel);

    uintptr_t mis = (uintptr_t)x ^ (uintptr_t)gy;
    if (WRITE_GX) mis |= (uintptr_t)x ^ (uintptr_t)gx;
    const bool vector_ok = (mis & (kVecBytes - 1)) == 0;
    const int head = vector_ok ? head_elems<T>(x, ck.n) : ck.n;
    const int nvec = (ck.n - head) / N;
    const VT *xv = (const VT *)(x + head);
    const VT *gv = (const VT *)(gy + head);
    VT *ov = WRITE_GX ? (VT *)(gx + head) : nullptr;
    const Edges edges = {vector_ok ? ck.n - nvec * N : 0, nvec * N};

    VT rx[ROWS], rg[ROWS];
    if (nvec > 0) {
        const int last = nvec - 1;
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            int v = u * group + tid;
            v = v < last ? v : last;
            rx[u] = ld_stream(xv + v);
            rg[u] = ld_stream(gv + v);
        }
    }
    unsigned ex = 0u, eg = 0u;
    if (tid < edges.count) {
        ex = ld_bits(x + edges.at(tid, head));
        eg = ld_bits(gy + edges.at(tid, head));
    }

    const QParams p = block_params<true, G>(d, theta, bs, group);

    double acc[ROWS];
#pragma unroll
    for (int u = 0; u < ROWS; ++u) acc[u] = 0.0;

#pragma unroll
    for (int u = 0; u < ROWS; ++u) {
        const int v = u * group + tid;
        if (v < nvec) {
            VT o;
            bool any_nan = false;
#pragma unroll
            for (int e = 0; e < N; ++e) {
                bool in_range, is_nan;
                float t = ste_terms((float)rx[u][e], p, in_range, is_nan);
                o[e] = in_range ? rg[u][e] : (T)0.0f;
                acc[u] = __builtin_fma((double)(float)rg[u][e], (double)t, acc[u]);
                any_nan |= is_nan;
            }
            if (any_nan) acc[u] = __builtin_nan("");   // a NaN quotient poisons its channel
            if constexpr (HELD == 0) {
                if (WRITE_GX) st_stream(ov + v, o);
            } else if constexpr (GX != kGxNo) {
                out.v[u] = __builtin_bit_cast(typename GxRows<HELD>::Bits, o);
            }
        }
    }
    if constexpr (HELD != 0) {
        out.to = (typename GxRows<HELD>::Bits *)ov;
        out.nvec = nvec;
        out.first = tid;
        out.step = group;
    }

    double sum = 0.0;
#pragma unroll
    for (int u = 0; u < ROWS; ++u) sum += acc[u];
    pin_here(ex);
    pin_here(eg);
    if (tid < edges.count) sum = backward_elem<T>(from_bits<T>(ex), from_bits<T>(eg), gx, edges.at(tid, head), p, sum);
    if (!vector_ok) {               // x, gy and gx are misaligned relative to each other
        for (int i = tid; i < ck.n; i += group)
            sum = backward_elem<T>(ld_global(x + i), ld_global(gy + i), gx, i, p, sum);
    }
    return sum;
}

// The same sum with the schedule for launches whose blocks are all resident at once (see burst_pays; a
// 1x384x9600 FP32 tensor).  Such a launch is one burst: every wavefront asks
// for its whole chunk at the start, the data trickles in over the next microseconds, and whatever a
// wavefront still has to compute after its last row has landed is added to the kernel's duration,
// with nothing left to hide it.  So all x rows are requested before all gy rows; what depends on x
// alone (quotient, clip, round, t, the mask: two thirds of the arithmetic) is done as the x rows
// arrive, while the gy rows are still on their way; only the products and the selects wait for the
// last row.  The price is registers (every row's t is kept: 124 VGPRs instead of 67 for five
// FP16 rows, four wavefronts per SIMD; 86 and five for FP32), so larger launches interleave.
// The arithmetic and its order are the same in both schedules; so are the bits.
template <typename T, int GX, int G, int ROWS>
__device__ __forceinline__ double backward_chunk_short(const DevTensor &d, const Chunk &ck, BlockScale &bs, GxRows<ROWS> &out,
                                                       const int group = G)
{
    constexpr bool WRITE_GX = GX == kGxYes;
    typedef typename VecOf<T>::type VT;
    constexpr int N = VecOf<T>::N;
    const T *x = (const T *)d.x + ck.first;
    const T *gy = (const T *)d.gy + ck.first;
    T *gx = WRITE_GX ? (T *)d.gx + ck.first : nullptr;
    const int tid = threadIdx.x & (group - 1);
    const float theta = ld_uniform(d.theta + ck.channel);

    uintptr_t mis = (uintptr_t)x ^ (uintptr_t)gy;
    if (WRITE_GX) mis |= (uintptr_t)x ^ (uintptr_t)gx;
    const bool vector_ok = (mis & (kVecBytes - 1)) == 0;
    const int head = vector_ok ? head_elems<T>(x, ck.n) : ck.n;
    const int nvec = (ck.n - head) / N;
    const VT *xv = (const VT *)(x + head);
    const VT *gv = (const VT *)(gy + head);
    VT *ov = WRITE_GX ? (VT *)(gx + head) : nullptr;
    const Edges edges = {vector_ok ? ck.n - nvec * N : 0, nvec * N};

    VT rx[ROWS], rg[ROWS];
    if (nvec > 0) {                   // out-of-range lanes re-read the last vector
        const int last = nvec - 1;
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const int v = u * group + tid;
            rx[u] = ld_stream(xv + (v < last ? v : last));
        }
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const int v = u * group + tid;
            rg[u] = ld_stream(gv + (v < last ? v : last));
        }
    }
    unsigned ex = 0u, eg = 0u;
    if (tid < edges.count) {
        ex = ld_bits(x + edges.at(tid, head));
        eg = ld_bits(gy + edges.at(tid, head));
    }

    const QParams p = block_params<true, G>(d, theta, bs, group);

    double acc[ROWS];
#pragma unroll
    for (int u = 0; u < ROWS; ++u) acc[u] = 0.0;

    if (nvec > 0) {
        float t[ROWS][N];
        unsigned inside[ROWS], nan_row[ROWS];
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            inside[u] = 0u;
            nan_row[u] = 0u;
#pragma unroll
            for (int e = 0; e < N; ++e) {
                bool in_range, is_nan;
                t[u][e] = ste_terms((float)rx[u][e], p, in_range, is_nan);
                inside[u] |= in_range ? 1u << e : 0u;
                nan_row[u] |= is_nan ? 1u : 0u;
                pin_here(t[u][e]);
            }
            pin_here(inside[u]);
            __builtin_amdgcn_sched_barrier(0);     // row by row: each waits for its own x alone
        }
#pragma unroll
        for (int u = 0; u < ROWS; ++u) {
            const int v = u * group + tid;
            if (v < nvec) {
                VT o;
#pragma unroll
                for (int e = 0; e < N; ++e) {
                    o[e] = (inside[u] >> e & 1u) ? rg[u][e] : (T)0.0f;
                    acc[u] = __builtin_fma((double)(float)rg[u][e], (double)t[u][e], acc[u]);
                }
                if (nan_row[u]) acc[u] = __builtin_nan("");   // a NaN quotient poisons its channel
                if (WRITE_GX) out.v[u] = __builtin_bit_cast(typename GxRows<ROWS>::Bits, o);
            }
        }
    }
    out.to = (typename GxRows<ROWS>::Bits *)ov;
    out.nvec = nvec;
    out.first = tid;
    out.step = group;

    double sum = 0.0;
#pragma unroll
    for (int u = 0; u < ROWS; ++u) sum += acc[u];
    pin_here(ex);
    pin_here(eg);
    if (tid < edges.count) sum = backward_elem<T>(from_bits<T>(ex), from_bits<T>(eg), gx, edges.at(tid, head), p, sum);
    if (!vector_ok) {               // x, gy and gx are misaligned relative to each other
        for (int i = tid; i < ck.n; i += group)
            sum = backward_elem<T>(ld_global(x + i), ld_global(gy + i), gx, i, p, sum);
    }
    return sum;
}

// Chain rule through Eq. (3)-(4) and the per-channel outputs of the backward pass.
__device__ __forceinline__ void write_channel_grads(const DevTensor &d, unsigned c, double total, const BlockScale &bs)
{
    const float g = bs.clip_active ? 0.0f : (float)(total * bs.sigmoid);
    if (d.gs) st_global(d.gs + c, (float)total);
    if (d.gtheta) st_global(d.gtheta + c, g);
    if (d.s) st_global(d.s + c, bs.s);
    if (__builtin_expect(d.adam_m != nullptr, 0)) {
        // One Adam step on theta_c (Kingma & Ba, Algorithm 1), binary32, each operation rounded
        // on its own.  Every block of this channel has finished reading theta_c by now (this
        // code runs after all of them have handed in their sums), so theta may be updated in
        // place.  A non-finite gradient leaves m, v and theta as they are.
        const float theta = ld_global(d.theta + c);
        float out = theta;
        if (__builtin_isfinite(g)) {
            const float m = d.adam_beta1 * ld_global(d.adam_m + c) + d.adam_one_minus_beta1 * g;
            const float v = d.adam_beta2 * ld_global(d.adam_v + c) + (d.adam_one_minus_beta2 * g) * g;
            const float mhat = m / d.adam_bc1, vhat = v / d.adam_bc2;
            st_global(d.adam_m + c, m);
            st_global(d.adam_v + c, v);
            out = theta - (d.adam_lr * mhat) / (__builtin_sqrtf(vhat) + d.adam_eps);
        }
        st_global(d.adam_theta_out + c, out);
    }
}

// The partial sums of channel c: one per unit, in index order.
__device__ __forceinline__ double *partials_of(const DevTensor &d, unsigned c)
{
    return d.partial + (size_t)c * (d.outer * d.cps);
}

__device__ __forceinline__ unsigned long long bits_of(double v) { return __builtin_bit_cast(unsigned long long, v); }

// A published sum differs from an empty (all zero) place: +0.0 travels as -0.0, which adds the same.
__device__ __forceinline__ double published(double v) { return bits_of(v) == 0ull ? -0.0 : v; }

// Up to this many units a channel's sums are added by one wavefront, lane l taking the sums l, l + 64, ... (at
// most four) in that order and wave_sum adding the lanes; beyond it by a block, thread t taking t, t + 256, ....
// A block that polls 150 to 240 sums with all its wavefronts and meets at a barrier afterwards is slower by 0.2 to
// 0.4 us (8x64x19200 FP16, 16 units: 12.65 / 12.25; 3x134x6588 FP32, 6 units: 8.93 / 8.50).
constexpr unsigned kWaveGather = 256;

// This thread's share of the partial sums of channel c, for a block (more than kWaveGather units): thread t adds the
// sums t, t+256, t+512, ... in that order, eight loads in flight.  looks > 0: a sum that is still zero is not
// published yet; the wavefront then looks at those eight rows again, and gives up (false) when it has looked in vain
// that often in all.  own >= 0: unit `own` is the caller's; its sum is `mine`, not in memory.
__device__ __forceinline__ bool add_partials_block(const DevTensor &d, unsigned c, unsigned own, double mine,
                                                   unsigned looks, double &acc)
{
    const unsigned bpc = d.outer * d.cps;
    constexpr unsigned kBatch = 8;
    const bool wait = looks != 0u;
    double *const parts = partials_of(d, c);
    acc = 0.0;
    for (unsigned first = wave_index() * 64u; first < bpc; first += kBlock * kBatch) {
        const unsigned j0 = first + (threadIdx.x & 63);
        double part[kBatch];
        for (;;) {
            order_accesses();
            bool here = true;
#pragma unroll
            for (unsigned i = 0; i < kBatch; ++i) {
                const unsigned j = j0 + i * kBlock;
                part[i] = mine;
                if (j < bpc && j != own)
                    part[i] = __hip_atomic_load(&parts[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (unsigned i = 0; i < kBatch; ++i) {
                const unsigned j = j0 + i * kBlock;
                if (j < bpc && j != own) here = here && bits_of(part[i]) != 0ull;
            }
            if (!wait || __builtin_amdgcn_ballot_w64(!here) == 0ull) break;
            if (--looks == 0u) return false;
        }
#pragma unroll
        for (unsigned i = 0; i < kBatch; ++i)
            if (j0 + i * kBlock < bpc) acc += part[i];
    }
    return true;
}

// Put the partial sums of channel c back to zero, for the next call.
template <int G>
__device__ __forceinline__ void clear_partials(const DevTensor &d, unsigned c)
{
    const unsigned bpc = d.outer * d.cps;
    double *const parts = partials_of(d, c);
    for (unsigned j = threadIdx.x & (G - 1); j < bpc; j += G)
        __hip_atomic_store(&parts[j], 0.0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// value of v in the given lane, as a wavefront-uniform scalar
__device__ __forceinline__ double read_lane(double v, int lane)
{
    const unsigned long long bits = __builtin_bit_cast(unsigned long long, v);
    const unsigned lo = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)bits, lane);
    const unsigned hi = (unsigned)__builtin_amdgcn_readlane((int)(unsigned)(bits >> 32), lane);
    return __builtin_bit_cast(double, ((unsigned long long)hi << 32) | lo);
}

// The sum of channel c's partial sums by a single wavefront: the way of up to kWaveGather units, and beyond
// that the block's, bit for bit: the block-wide version gives thread t the sums t, t+256, ... and adds wavefront 0's
// tree to wavefront 1's, 2's and 3's in that order; here the one wavefront plays the four, 256 sums in flight
// (4000x4x100 FP32, 4000 units per channel: 30.8 us with one row of 64 at a time, 21.9 now).  looks and own as above,
// looks = 0 for up to kWaveGather units only.
// clear: put the sums back to zero as soon as they are all here (up to kWaveGather units; `own' was never there).
__device__ __forceinline__ bool add_partials_wave(const DevTensor &d, unsigned c, unsigned own, double mine,
                                                  unsigned looks, bool clear, double &total)
{
    constexpr unsigned kWaves = kBlock / 64;
    static_assert(kWaveGather == kWaves * 64, "one batch of four loads per lane");
    const unsigned bpc = d.outer * d.cps;
    const unsigned lane = threadIdx.x & 63;
    const bool wait = looks != 0u;
    double *const parts = partials_of(d, c);
    if (bpc <= 64u) {                              // the usual case, in less code (5x1500x72 FP16 7.5 us instead of 7.7)
        double part = mine;
        for (;;) {
            order_accesses();
            if (lane < bpc && lane != own)
                part = __hip_atomic_load(&parts[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (!wait || __builtin_amdgcn_ballot_w64(lane < bpc && lane != own && bits_of(part) == 0ull) == 0ull) break;
            if (--looks == 0u) return false;
        }
        if (clear && lane < bpc) st_global(&parts[lane], 0.0);
        double one = 0.0;
        if (lane < bpc) one += part;
        total = 0.0 + read_lane(wave_sum(one), kSumLane);
        return true;
    }
    // (The same look twice: with the way of up to kWaveGather units inside the loop of the other, each of its rounds
    // was 0.06 us longer, 16000x1x100 FP32 59.4 / 56.8 us; as a function of its own it waited for every load, 97.)
    if (bpc <= kWaveGather) {
        double part[kWaves], one = 0.0;
        for (;;) {
            order_accesses();
            bool here = true;
#pragma unroll
            for (unsigned w = 0; w < kWaves; ++w) {
                const unsigned j = w * 64 + lane;
                part[w] = mine;
                if (w * 64 < bpc && j < bpc && j != own)
                    part[w] = __hip_atomic_load(&parts[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (unsigned w = 0; w < kWaves; ++w) {
                const unsigned j = w * 64 + lane;
                if (j < bpc && j != own) here = here && bits_of(part[w]) != 0ull;
            }
            if (!wait || __builtin_amdgcn_ballot_w64(!here) == 0ull) break;
            if (--looks == 0u) return false;
        }
#pragma unroll
        for (unsigned w = 0; w < kWaves; ++w) {
            const unsigned j = w * 64 + lane;
            if (clear && j < bpc) st_global(&parts[j], 0.0);
            if (j < bpc) one += part[w];
        }
        total = 0.0 + read_lane(wave_sum(one), kSumLane);
        return true;
    }
    double acc[kWaves];
#pragma unroll
    for (unsigned w = 0; w < kWaves; ++w) acc[w] = 0.0;
    for (unsigned first = 0; first < bpc; first += kBlock) {
        double part[kWaves];
        for (;;) {
            order_accesses();
            bool here = true;
#pragma unroll
            for (unsigned w = 0; w < kWaves; ++w) {
                const unsigned j = first + w * 64 + lane;
                part[w] = mine;
                if (first + w * 64 < bpc && j < bpc && j != own)
                    part[w] = __hip_atomic_load(&parts[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
#pragma unroll
            for (unsigned w = 0; w < kWaves; ++w) {
                const unsigned j = first + w * 64 + lane;
                if (j < bpc && j != own) here = here && bits_of(part[w]) != 0ull;
            }
            if (__builtin_amdgcn_ballot_w64(!here) == 0ull) break;
            if (--looks == 0u) return false;
        }
#pragma unroll
        for (unsigned w = 0; w < kWaves; ++w)
            if (first + w * 64 + lane < bpc) acc[w] += part[w];
    }
    total = 0.0;
#pragma unroll
    for (unsigned w = 0; w < kWaves; ++w) total += read_lane(wave_sum(acc[w]), kSumLane);
    return true;
}

// Second launch of the two-launch mode: the sum of all partial sums of channel c, the channel's gradients, and the
// partial sums back to zero.  Block-wide; lds holds kBlock/64 doubles.
__device__ __forceinline__ void finalize_channel(const DevTensor &d, unsigned c, const BlockScale &bs, double *lds)
{
    double total = 0.0;
    if (d.outer * d.cps <= kWaveGather) {
        if (threadIdx.x >= 64) return;
        add_partials_wave(d, c, ~0u, 0.0, 0u, true, total);
    } else {
        double acc;
        add_partials_block(d, c, ~0u, 0.0, 0u, acc);
        acc = wave_sum(acc);
        clear_partials<kBlock>(d, c);
        if ((threadIdx.x & 63) == kSumLane) lds[threadIdx.x >> 6] = acc;
        __syncthreads();
#pragma unroll
        for (int w = 0; w < kBlock / 64; ++w) total += lds[w];
    }
    if (threadIdx.x == 0) write_channel_grads(d, c, total, bs);
}

// How the units (blocks, or wavefronts of short-slab tensors) of a channel combine their sums
// (FUSED; no float atomics, fixed order):
//   1 unit per channel    the unit writes the channel's gradients itself;
//   2 units per channel   each swaps its sum into the channel's 64-bit slot; the one that finds
//                         its partner's sum there adds the two (a+b = b+a) and clears the slot:
//                         one atomic round trip, the payload travels in the atomic itself;
//   3 or 4                two rounds of that exchange, pairs first (two more slots per channel);
//   more                  each unit publishes its sum in partial[] and the channel's last unit in
//                         index order, its collector, gathers them: see publish and collect.
// Slots and partial sums are zero between calls.
// Without FUSED the sums are only stored and finalize_kernel adds them in a second launch.
//
// Called by one wavefront per unit with the unit's total, for up to kTreeBlocks units per channel and
// without FUSED; its first lane does the work.  store_gx: what the wavefront still has to store, behind the exchange.
template <bool FUSED, typename F>
__device__ __forceinline__ void combine(const DevTensor &d, const Chunk &ck, double total, const BlockScale &bs, F store_gx)
{
    const unsigned bpc = d.outer * d.cps;
    const bool first_lane = (threadIdx.x & 63) == 0;
    if (!FUSED || bpc == 1u) {
        if (first_lane) {
            if (FUSED) write_channel_grads(d, ck.channel, total, bs);
            else __hip_atomic_store(&partials_of(d, ck.channel)[ck.j], total, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        store_gx();
    } else if (bpc == 2u) {
        unsigned long long theirs = 0ull;
        if (first_lane)
            theirs = __hip_atomic_exchange(&d.slot[ck.channel], bits_of(published(total)), __ATOMIC_RELAXED,
                                           __HIP_MEMORY_SCOPE_AGENT);
        store_gx();
        if (theirs != 0ull) {
            __hip_atomic_store(&d.slot[ck.channel], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            const double both = (__builtin_bit_cast(double, theirs) + total) + 0.0;
            write_channel_grads(d, ck.channel, both, bs);
        }
    } else {
        // Three or four units: two rounds of the same exchange, associated as finalize_channel
        // associates its sums, (p0 + p1) + (p2 + p3) with an absent p3 counting as +0.0, so the
        // bits equal those of the two-launch mode.
        const unsigned j = ck.j;
        const bool paired = !(bpc == 3u && j == 2u);   // unit 2 of 3 has no partner
        unsigned long long *pair = d.slot + d.channels + (size_t)ck.channel * 2u + (j >> 1);
        unsigned long long theirs = 0ull;
        if (first_lane && paired)
            theirs = __hip_atomic_exchange(pair, bits_of(published(total)), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        store_gx();
        double pair_sum = total + 0.0;
        if (theirs != 0ull) {
            __hip_atomic_store(pair, 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            pair_sum = __builtin_bit_cast(double, theirs) + total;
        }
        if (first_lane && (theirs != 0ull || !paired)) {
            const unsigned long long others = __hip_atomic_exchange(&d.slot[ck.channel], bits_of(published(pair_sum)),
                                                                    __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            if (others != 0ull) {
                __hip_atomic_store(&d.slot[ck.channel], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                const double all = (__builtin_bit_cast(double, others) + pair_sum) + 0.0;
                write_channel_grads(d, ck.channel, all, bs);
            }
        }
    }
}

// More than kTreeBlocks units per channel.  What bounds the end of such a launch is the number of
// dependent trips to memory behind the last unit's sum, about 0.5 us each: with arrival tickets there
// were four (store acknowledged, first-level ticket, top ticket, sums re-read).  Here there are two: the
// unit's sum reaches memory, and the collector, which is polling the channel's sums (up to four per lane of one
// wavefront, beyond kWaveGather units eight per thread of the block, where what has been added is not read again),
// sees it.  A sum announces itself: its place was zero and a published sum never is.  A channel's sums lie next to
// each other, so a trip is one or two cache lines.  What it takes (stamps of the clock in the blocks, one scale, 921600
// FP16 in 225 units, us): loads requested 0.1, scale there 0.6, last row done 1.4, last sum published 1.6, seen by the
// collector 2.3, added 2.4 (2.75 while four wavefronts' trees were added apart), gradients in memory 3.
// Measured, back to back, with tickets / polled by the whole block with gx in front / now: one scale, 153600 FP32 in
// 150 units 6.0 / 4.4 / 3.8; 2457600 FP16 in 240 units 7.9 / 6.2 / 5.5; 39321600 FP16 in 3840 units 44.4 / 42.8 / 40.7;
// 15x128x19200 FP16, 30 units per channel 40.1 / 39.9 / 37.6; 15x384x1200 FP16, 15 wavefront units 11.9 / 11.3 / 9.8.
//
// No wait is without end and nothing rests on the order in which blocks are dispatched: beside the one pass
// that the adding takes anyhow, the collector looks at most kPollRounds times in vain (a few tens of
// microseconds, whatever the number of units; normally one to three).  If a sum is still missing then, it publishes its own, raises the channel's slot to kGivenUp, and looks once more after the
// flag has been acknowledged.  Every unit reads the flag after its own sum has been acknowledged, so
// either the collector's last look sees that sum or the unit sees the flag; a unit that sees the flag
// looks at all sums itself, and the last one to arrive finds them complete.  Whoever finds them complete
// after the flag was raised claims the channel by a compare-exchange of the slot, so that one of them
// writes the gradients, and puts the slot back to zero.
constexpr unsigned long long kGivenUp = 1ull, kClaimed = 2ull;
constexpr unsigned kPollRounds = 32;

// (Tried and slower, one scale, 921600 FP16 in 225 units, 5.1 us at the time: looks in flight side by side, two 6.6,
// four 8.0, because they hold up the sums that are on their way to the same lines; reading again only what was
// missing 5.2; a sum per cache line 5.0 to 5.25, but 6.6 instead of 6.2 for 2457600; sums of one XCD next to each other 5.3.)

// The flag is up: one wavefront looks at all sums (`own`: none, all are in memory) and finishes the
// channel if they are complete and no other unit has claimed it.
__device__ __forceinline__ void finish_if_complete(const DevTensor &d, unsigned c, const BlockScale &bs)
{
    double total;
    if (!add_partials_wave(d, c, ~0u, 0.0, 1u, false, total)) return;
    unsigned won = 0u;
    if ((threadIdx.x & 63) == 0) {
        unsigned long long expected = kGivenUp;
        won = __hip_atomic_compare_exchange_strong(&d.slot[c], &expected, kClaimed, __ATOMIC_RELAXED, __ATOMIC_RELAXED,
                                                   __HIP_MEMORY_SCOPE_AGENT) ? 1u : 0u;
    }
    if (!__builtin_amdgcn_readfirstlane((int)won)) return;
    order_accesses();
    clear_partials<64>(d, c);
    if ((threadIdx.x & 63) == 0) {
        write_channel_grads(d, c, total, bs);
        __hip_atomic_store(&d.slot[c], 0ull, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// A unit that is not its channel's collector (one wavefront; total is uniform).  The sum goes out with an
// agent-scope store (global_store ... sc1: written through to the memory level that all XCDs share).
// Stores count in vmcnt on this target and an agent-scope store is acknowledged only once it has reached
// that level, so after s_waitcnt vmcnt(0) the sum is visible to every XCD, and the flag is read after
// that.  A release fence at agent scope would give the same order but also write back the whole L2.
template <typename F>
__device__ __forceinline__ void publish(const DevTensor &d, const Chunk &ck, double total, const BlockScale &bs, F store_gx)
{
    if ((threadIdx.x & 63) == 0)
        __hip_atomic_store(&partials_of(d, ck.channel)[ck.j], published(total), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    order_accesses();
    store_gx();
    wait_stores_acknowledged();
    const unsigned long long flag = __hip_atomic_load(&d.slot[ck.channel], __ATOMIC_RELAXED,
                                                      __HIP_MEMORY_SCOPE_AGENT);
    if (__builtin_expect(__builtin_amdgcn_readfirstlane((int)(unsigned)flag) == (int)kGivenUp, 0))
        finish_if_complete(d, ck.channel, bs);
}

// The collector has stopped polling (one wavefront; total is uniform).
__device__ __forceinline__ void give_up(const DevTensor &d, const Chunk &ck, double total, const BlockScale &bs)
{
    if ((threadIdx.x & 63) == 0)
        __hip_atomic_store(&partials_of(d, ck.channel)[ck.j], published(total), __ATOMIC_RELAXED,
                           __HIP_MEMORY_SCOPE_AGENT);
    wait_stores_acknowledged();
    if ((threadIdx.x & 63) == 0)
        __hip_atomic_store(&d.slot[ck.channel], kGivenUp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    wait_stores_acknowledged();
    finish_if_complete(d, ck.channel, bs);
}

// What follows the chunk of a block: the block's sum, its combination with the channel's others, and gx.
// FEW: the launch has no channel whose sums are gathered.  store_gx stores this thread's rows of gx.
//
// The sum goes out in front of gx, whose stores would otherwise lie ahead of it in the memory pipeline; the
// exchange or the gathering then runs while they drain.  Measured with gx in front of the sum / behind it, us:
// 15x128x19200 FP16 39.9 / 38.05, 1x384x19200 FP16 9.3 / 8.95, 8x64x19200 FP16 13.7 / 12.8, 15x384x1200 FP16 (wavefront
// units) 11.35 / 10.25, 3x131x4819 FP16 5.9 / 5.5, 1x1x4915200 FP16 9.0 / 8.2, 384x3456 FP32 5.2 / 4.8.  The collector
// stores its own gx in front of the first look, which would come too early otherwise (one scale, 921600 FP16:
// 4.8 / 4.5), and which leaves the registers to the sums.
template <bool FUSED, bool FEW, typename F>
__device__ __forceinline__ void combine_block(const DevTensor &d, const Chunk &ck, double sum, const BlockScale &bs, F store_gx)
{
    __shared__ double wave_part[kBlock / 64];
    __shared__ double fin_part[kBlock / 64];
    __shared__ unsigned missing[kBlock / 64];

    sum = wave_sum(sum);
    if ((threadIdx.x & 63) == kSumLane) wave_part[threadIdx.x >> 6] = sum;
    __syncthreads();
    const unsigned bpc = d.outer * d.cps;
    const bool gathered = FUSED && !FEW && bpc > kTreeBlocks;
    // the channel's last unit in index order: normally dispatched after the others
    const bool collector = gathered && ck.j + 1u == bpc;
    if (threadIdx.x >= 64 && !(collector && bpc > kWaveGather)) {
        store_gx();
        return;
    }
    double total = 0.0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) total += wave_part[w];
    if (!gathered) {
        combine<FUSED>(d, ck, total, bs, store_gx);
        return;
    }
    if (!collector) {
        publish(d, ck, total, bs, store_gx);
        return;
    }
    store_gx();
    const unsigned looks = d.flags & 4u ? 0u : kPollRounds;       // FQ_FLAG_NO_POLL
    if (bpc <= kWaveGather) {
        double all = 0.0;
        // A look costs about 0.5 us, and one that comes too early costs that for nothing.  Many units of one channel
        // end together, so the first look waits 0.2 us for their sums (us, without / with: 921600 FP16, 225 units, 4.45 /
        // 4.18, 2457600 FP16, 240 units, 5.98 / 5.60); few units of many channels don't (3x134x6588 FP32, 6 units, 8.2 / 8.4).
        if (bpc > 64u) __builtin_amdgcn_s_sleep(8);
        if (looks && add_partials_wave(d, ck.channel, bpc - 1u, total, looks, true, all)) {
            if (threadIdx.x == 0) write_channel_grads(d, ck.channel, all, bs);
        } else {
            give_up(d, ck, total, bs);
        }
        return;
    }
    double acc = 0.0;
    const bool present = looks && add_partials_block(d, ck.channel, bpc - 1u, total, looks, acc);
    acc = wave_sum(acc);
    if ((threadIdx.x & 63) == kSumLane) {
        fin_part[threadIdx.x >> 6] = acc;
        missing[threadIdx.x >> 6] = present ? 0u : 1u;
    }
    __syncthreads();
    unsigned any_missing = 0u;
    double all = 0.0;
#pragma unroll
    for (int w = 0; w < kBlock / 64; ++w) {
        any_missing |= missing[w];
        all += fin_part[w];
    }
    if (__builtin_expect(any_missing != 0u, 0)) {
        if (threadIdx.x < 64) give_up(d, ck, total, bs);
        return;
    }
    if (threadIdx.x == 0) write_channel_grads(d, ck.channel, all, bs);
    clear_partials<kBlock>(d, ck.channel);
}

// The same for a unit that is a wavefront: the block never meets at a barrier.
template <bool FUSED, typename F>
__device__ __forceinline__ void combine_wave(const DevTensor &d, const Chunk &ck, double sum, const BlockScale &bs, F store_gx)
{
    const double total = read_lane(wave_sum(sum), kSumLane);
    const unsigned bpc = d.outer * d.cps;
    if (!FUSED || bpc <= kTreeBlocks) {
        combine<FUSED>(d, ck, total, bs, store_gx);
        return;
    }
    if (ck.j + 1u != bpc) {
        publish(d, ck, total, bs, store_gx);
        return;
    }
    store_gx();
    double all = 0.0;
    const bool present = !(d.flags & 4u) &&                       // FQ_FLAG_NO_POLL
                         add_partials_wave(d, ck.channel, bpc - 1u, total, kPollRounds, true, all);
    if (__builtin_expect(!present, 0)) {
        give_up(d, ck, total, bs);
        return;
    }
    if ((threadIdx.x & 63) == 0) write_channel_grads(d, ck.channel, all, bs);
    if (bpc > kWaveGather) clear_partials<64>(d, ck.channel);
}

// One block of the backward grid, owning one chunk of one slab.
template <typename T, bool FUSED, int ROWS, bool SHORT>
__device__ __forceinline__ void backward_block(const DevTensor &d, const Chunk &ck)
{
    const bool write_gx = d.gx != nullptr;
    BlockScale bs;
    // Nothing waits for the sum of a two-launch backward: there gx is stored row by row, which takes fewer registers and
    // instructions.  Held until behind the sum, short slabs in many blocks were slower, us, row by row / held: 2464x855x2 FP16 621 / 653,
    // 98x23995x21 1242 / 1279, 219x4128x1 FP32 270 / 279.
    GxRows<FUSED ? ROWS : 0> gx;
    double sum;
    if constexpr (SHORT) sum = write_gx ? backward_chunk_short<T, kGxYes, kBlock, ROWS>(d, ck, bs, gx) : backward_chunk_short<T, kGxNo, kBlock, ROWS>(d, ck, bs, gx);
    else sum = write_gx ? backward_chunk<T, kGxYes, kBlock, ROWS>(d, ck, bs, gx) : backward_chunk<T, kGxNo, kBlock, ROWS>(d, ck, bs, gx);
    combine_block<FUSED, SHORT>(d, ck, sum, bs, [&] { gx.store(); });
}

// One block of the backward grid for a tensor with short slabs: every wavefront owns a slab (a
// unit) of its own.
template <typename T, bool FUSED, int ROWS>
__device__ __forceinline__ void backward_waves(const DevTensor &d, unsigned local_block)
{
    const unsigned unit = local_block * (kBlock / 64) + wave_index();
    if (unit >= d.slabs * d.cps) return;
    const bool write_gx = d.gx != nullptr;
    const Chunk ck = locate_chunk(d, unit);
    BlockScale bs;
    GxRows<FUSED ? ROWS : 0> gx;
    const double sum = write_gx ? backward_chunk<T, kGxYes, 64, ROWS>(d, ck, bs, gx) : backward_chunk<T, kGxNo, 64, ROWS>(d, ck, bs, gx);
    combine_wave<FUSED>(d, ck, sum, bs, [&] { gx.store(); });
}

// ---------------------------------------------------------------------------------------------
// Multi-tensor grid: the table lives at the start of the workspace, and behind it the first block of each
// tensor once more, packed.  Block -> tensor: last entry whose first block is <= block.  Up to 64 entries the
// lanes of a wavefront look at once, one trip to the cache for two lines where a binary search over the
// descriptors takes up to six dependent ones; longer lists are halved down to that first.  Measured, us, binary
// search / lanes: 22 weight tensors of 1.3 M elements forward 8.4 / 7.4, backward 10.2 / 9.7; 64 tensors of 1 GiB
// 385 / 379, 552 / 547.  (Lanes that look at the descriptors themselves, a line each: 7.3, 9.7, but 395 and 568.)
__device__ __forceinline__ int find_by_block(const DevTensor *table, int n, unsigned block)
{
    const unsigned *begins = (const unsigned *)(table + n);
    int lo = 0, hi = n - 1;
    while (hi - lo >= 64) {
        int mid = (lo + hi + 1) >> 1;
        if (ld_uniform(begins + mid) <= block) lo = mid; else hi = mid - 1;
    }
    const int mine = lo + (int)(threadIdx.x & 63);
    const bool begun = mine <= hi && ld_global(begins + (mine <= hi ? mine : hi)) <= block;
    return lo + (int)__popcll(__builtin_amdgcn_ballot_w64(begun)) - 1;
}

__device__ __forceinline__ int find_by_channel(const FQ_CONST DevTensor *table, int n, unsigned chan)
{
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        int mid = (lo + hi + 1) >> 1;
        if (table[mid].chan_begin <= chan) lo = mid; else hi = mid - 1;
    }
    return lo;
}

// copy one table entry into registers, word by word through the scalar cache
__device__ __forceinline__ DevTensor fetch(const DevTensor *table, int i)
{
    static_assert(sizeof(DevTensor) % 4 == 0, "descriptor is copied as 32-bit words");
    DevTensor d;
    const FQ_CONST unsigned *src = (const FQ_CONST unsigned *)(table + i);
    unsigned *dst = (unsigned *)&d;
#pragma unroll
    for (unsigned w = 0; w < sizeof(DevTensor) / 4; ++w) dst[w] = src[w];
    return d;
}

// Single tensor: descriptor in the kernel arguments (SGPRs), dtype fixed at compile time.
// What the first loads' addresses are made of stands in front of the descriptor as arguments of its own: the build has
// the leading 14 dwords of arguments put into registers with the launch (build.py), so that no wavefront waits for the
// descriptor, one trip to memory, before it requests its rows.  channels is 0 where the grid is linear.  us, before / with:
// forward of 153600 FP32 2.34 / 2.22, 64x576 FP32 2.25 / 2.16, 2457600 FP16 3.46 / 3.35, 384x19200 FP16 6.49 / 6.36, backward
// 3.62 / 3.49, 2.91 / 2.80, 5.80 / 5.69, 3x131x4819 FP16 5.77 / 5.55, 15x128x19200 FP16 38.8 / 38.4; list of 22 FP32 weight tensors
// forward 4.72 / 4.55 (the table's address and length); distillation of 1x128x1200 FP16 5.30 / 5.17.
// G: lanes that share a chunk: 64 (the tensor's slabs are short and every wavefront owns one), or the block's
// threads, kBlock or kWideBlock (chosen by the launcher).  ROWS: the vectors per lane that a whole chunk has, at most.
template <typename T, bool WRITE_Y, bool EMIT_Q, int G, int ROWS, bool EARLY>
__global__ void __launch_bounds__(G == 64 ? kBlock : G)
forward_kernel(const void *x, void *y, const float *theta, long long inner, unsigned chunk, unsigned channels, const DevTensor rest)
{
    DevTensor d = rest;
    d.x = x;
    d.y = y;
    d.theta = theta;
    d.inner = inner;
    d.chunk = chunk;
    d.grid3 = channels != 0u;
    if (d.grid3) d.channels = channels;
    if (G == 64) {
        const unsigned unit = blockIdx.x * (kBlock / 64) + wave_index();
        if (unit < d.slabs * d.cps) forward_chunk<T, WRITE_Y, EMIT_Q, 64, ROWS, EARLY>(d, locate_chunk(d, unit));
    } else {
        forward_chunk<T, WRITE_Y, EMIT_Q, G, ROWS, EARLY>(d, own_chunk(d));
    }
}

// The code of the multi-tensor kernels is kept short: blocks of one launch run through different parts of
// it, and two compute units share 64 KB of instruction cache.  So the number of rows is rounded up to 1, 2 or
// kMaxRows, and the backward is told at run time which lanes share a chunk (a block's or a wavefront's) and
// whether gx is written (72 KB -> 45 KB at the time; now 61 KB, 31 KB of it without the combination of the units' sums, whose
// ways for different numbers of units stand apart).  The forward, which is shorter, loses by the former (us, told at run
// time / compiled in: lists of 16 mixed tensors and 20 M elements 28.2 / 27.7, 40 and 60 M 66.2 / 65.0, 4x(128x9600)
// FP16 5.72 / 5.64).
template <typename F> __device__ __forceinline__ void for_rows(int rows, F f)
{
    if (rows == 1) f(std::integral_constant<int, 1>());
    else if (rows == 2) f(std::integral_constant<int, 2>());
    else f(std::integral_constant<int, kMaxRows>());
}

// ANY_Q = false: no tensor of the list wants codes (the usual case; keeps the kernel lean)
template <bool ANY_Q, bool EARLY>
__global__ void __launch_bounds__(kBlock) forward_multi_kernel(const DevTensor *table, int n)
{
    const DevTensor d = fetch(table, find_by_block(table, n, blockIdx.x));
    const unsigned local = blockIdx.x - d.block_begin;
    if (ANY_Q) {
        if (d.dtype == 0) forward_dispatch<_Float16, EARLY>(d, local);
        else forward_dispatch<float, EARLY>(d, local);
        return;
    }
    const unsigned unit = d.wave_units ? local * (kBlock / 64) + wave_index() : local;
    if (unit >= d.slabs * d.cps) return;
    const Chunk ck = locate_chunk(d, unit);
    if (d.wave_units) {
        if (d.dtype == 0) forward_chunk<_Float16, true, false, 64, kMaxRows, EARLY>(d, ck);
        else forward_chunk<float, true, false, 64, kMaxRows, EARLY>(d, ck);
    } else {
        for_rows(d.rows, [&](auto rows) {
            if (d.dtype == 0) forward_chunk<_Float16, true, false, kBlock, decltype(rows)::value, EARLY>(d, ck);
            else forward_chunk<float, true, false, kBlock, decltype(rows)::value, EARLY>(d, ck);
        });
    }
}

// gx: nullptr where the gradient of x is not asked for.
// SHAPE: 0 = one chunk per block; 1 = one slab per wavefront (short slabs); 2 = one chunk per block
// with the burst schedule (see backward_chunk_short and launch_backward_shaped).
template <typename T, bool FUSED, int SHAPE, int ROWS>
__global__ void __launch_bounds__(kBlock)
backward_kernel(const void *x, const void *gy, void *gx, const float *theta, long long inner, unsigned chunk, unsigned cps,
                unsigned channels, const DevTensor rest)
{
    DevTensor d = rest;
    d.x = x;
    d.gy = gy;
    d.gx = gx;
    d.theta = theta;
    d.inner = inner;
    d.chunk = chunk;
    d.cps = cps;
    d.grid3 = channels != 0u;
    if (d.grid3) d.channels = channels;
    if (SHAPE == 1) {
        backward_waves<T, FUSED, ROWS>(d, blockIdx.x);
    } else {
        backward_block<T, FUSED, ROWS, SHAPE == 2>(d, own_chunk(d));
    }
}

// bias: the bias corrections of the Adam steps, where they are the same for all tensors and not those that the
// table holds.  The first block of each tensor puts them there as well, for the launches to come.
template <bool FUSED>
__global__ void __launch_bounds__(kBlock) backward_multi_kernel(const DevTensor *table, int n, const AdamBias bias)
{
    const int index = find_by_block(table, n, blockIdx.x);
    DevTensor d = fetch(table, index);
    const unsigned local = blockIdx.x - d.block_begin;
    if (bias.set) {
        d.adam_bc1 = bias.bc1;
        d.adam_bc2 = bias.bc2;
        if (local == 0 && threadIdx.x == 0 && d.adam_m) {
            st_global(const_cast<float *>(&table[index].adam_bc1), bias.bc1);
            st_global(const_cast<float *>(&table[index].adam_bc2), bias.bc2);
        }
    }
    const unsigned unit = d.wave_units ? local * (kBlock / 64) + wave_index() : local;
    if (unit >= d.slabs * d.cps) return;
    const Chunk ck = locate_chunk(d, unit);
    const int group = d.wave_units ? 64 : kBlock;
    BlockScale bs;
    // (gx in front of the sum: behind it, held in registers over the five ways to work it out, a list of 64 mixed
    // tensors takes 551 us instead of 547, and 22 weight tensors the same.)
    GxRows<0> gx;
    double sum = 0.0;
    for_rows(d.rows, [&](auto rows) {
        if (d.dtype == 0) sum = backward_chunk<_Float16, kGxAsked, 0, decltype(rows)::value>(d, ck, bs, gx, group);
        else sum = backward_chunk<float, kGxAsked, 0, decltype(rows)::value>(d, ck, bs, gx, group);
    });
    if (d.wave_units) combine_wave<FUSED>(d, ck, sum, bs, [] {});
    else combine_block<FUSED, false>(d, ck, sum, bs, [] {});
}

// one block per channel: second pass of the two-pass backward, and the whole backward of tensors
// that have channels but no elements (their gradients are zero)
__global__ void __launch_bounds__(kBlock) finalize_kernel(const KArgs a)
{
    __shared__ double fin_part[kBlock / 64];
    const DevTensor d = a.table ? fetch(a.table, find_by_channel((const FQ_CONST DevTensor *)a.table, a.n, blockIdx.x))
                                : a.one;
    const unsigned c = blockIdx.x - d.chan_begin;
    BlockScale bs;
    block_params<true, kBlock>(d, ld_uniform(d.theta + c), bs);
    finalize_channel(d, c, bs, fin_part);
}

// s[c] for every channel; used when a tensor has channels but no elements (forward)
__global__ void __launch_bounds__(kBlock) scale_kernel(const KArgs a, unsigned total_channels)
{
    unsigned g = blockIdx.x * kBlock + threadIdx.x;
    if (g >= total_channels) return;
    const DevTensor *dp = a.table ? &a.table[find_by_channel((const FQ_CONST DevTensor *)a.table, a.n, g)] : &a.one;
    unsigned c = g - dp->chan_begin;
    if (dp->s) dp->s[c] = compute_scale<false>(dp->theta[c], dp->eps, dp->s_min, dp->s_max).s;
}

__global__ void __launch_bounds__(kBlock) fill_zero_kernel(unsigned *p, size_t words)
{
    size_t i = (size_t)blockIdx.x * kBlock + threadIdx.x;
    const size_t stride = (size_t)gridDim.x * kBlock;
    for (; i < words; i += stride) p[i] = 0u;
}

}  // namespace

// ---------------------------------------------------------------------------------------------
// Measurement aid (fq_probe_stream): streaming kernels with no arithmetic in the launch shape of the
// forward and backward kernels (256-thread blocks, one chunk of kChunkVecs 128-bit vectors each,
// every load issued before the first store, non-temporal).  What they take is what the memory
// system and the launch cost alone take for the same bytes.
namespace {
typedef unsigned probe_vec __attribute__((ext_vector_type(4)));

template <int INPUTS>
__global__ void __launch_bounds__(kBlock) probe_kernel(const probe_vec *a, const probe_vec *b, probe_vec *out, size_t nvec)
{
    constexpr int kRows = kChunkVecs / kBlock;
    if (INPUTS == 0) return;
    const size_t first = (size_t)blockIdx.x * kChunkVecs + threadIdx.x;
    probe_vec ra[kRows], rb[kRows];
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
        size_t v = first + (size_t)u * kBlock;
        v = v < nvec ? v : nvec - 1;
        ra[u] = ld_stream(a + v);
        if (INPUTS == 2) rb[u] = ld_stream(b + v);
    }
#pragma unroll
    for (int u = 0; u < kRows; ++u) {
        const size_t v = first + (size_t)u * kBlock;
        if (v < nvec) st_stream(out + v, INPUTS == 2 ? ra[u] ^ rb[u] : ra[u]);
    }
}
}  // namespace

int launch_probe(int inputs, const void *a, const void *b, void *out, size_t bytes, void *stream)
{
    const size_t nvec = bytes / kVecBytes;
    if (nvec == 0) return 0;
    const unsigned blocks = (unsigned)((nvec + kChunkVecs - 1) / kChunkVecs);
    hipStream_t st = (hipStream_t)stream;
    const probe_vec *pa = (const probe_vec *)a, *pb = (const probe_vec *)b;
    probe_vec *po = (probe_vec *)out;
    if (inputs == 0) hipLaunchKernelGGL(probe_kernel<0>, dim3(blocks), dim3(kBlock), 0, st, pa, pb, po, nvec);
    else if (inputs == 1) hipLaunchKernelGGL(probe_kernel<1>, dim3(blocks), dim3(kBlock), 0, st, pa, pb, po, nvec);
    else hipLaunchKernelGGL(probe_kernel<2>, dim3(blocks), dim3(kBlock), 0, st, pa, pb, po, nvec);
    return (int)hipGetLastError();
}

// ---------------------------------------------------------------------------------------------
// Built-in scratch memory for callers that cannot allocate (fq_backward_static).  One array per
// GPU, held from the moment the code object is loaded until the process ends.  In host code the
// array's name stands for the symbol, not for a device address: the address on the current
// device comes from hipGetSymbolAddress, once per device, and only that pointer is ever handed
// to kernels.
static __device__ __align__(256) unsigned char scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex scratch_mutex;
void *scratch_ptr[kMaxDevices];     // per device; nullptr until the first call on that device
}  // namespace

// Device address of the scratch array on the current device (0 = success, else a hipError_t).
// The first call on a device also zeroes it with a fill kernel on `stream`; the loader has zeroed
// it already and every completed backward leaves it zero, this only makes the starting state explicit.
int static_scratch(void **ptr, void *stream)
{
    int device = -1;
    hipError_t e = hipGetDevice(&device);
    if (e != hipSuccess) return (int)e;
    if (device < 0 || device >= kMaxDevices) return (int)hipErrorInvalidDevice;
    std::lock_guard<std::mutex> lock(scratch_mutex);
    if (!scratch_ptr[device]) {
        void *p = nullptr;
        e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess) return (int)e;
        if (!p) return (int)hipErrorInvalidSymbol;
        const int rc = launch_fill_zero(p, kStaticScratchBytes, stream);
        if (rc != 0) return rc;
        scratch_ptr[device] = p;
    }
    *ptr = scratch_ptr[device];
    return 0;
}

// ---------------------------------------------------------------------------------------------
// Launchers.
template <typename K, typename... Args>
static void launch(K kernel, unsigned blocks, hipStream_t st, Args... args)
{
    hipLaunchKernelGGL(kernel, dim3(blocks), dim3(kBlock), 0, st, args...);
}

// Single-tensor launch: grid (chunks per slab, channels, outer) where d.grid3 says so.
typedef void (*ForwardKernel)(const void *, void *, const float *, long long, unsigned, unsigned, const DevTensor);
typedef void (*BackwardKernel)(const void *, const void *, void *, const float *, long long, unsigned, unsigned, unsigned,
                               const DevTensor);

// (hipLaunchKernel, not the triple-chevron form, which stores the configuration away and fetches it again: 2.48 / 2.31
// us of host time per launch.)
static void launch_tensor(ForwardKernel kernel, unsigned blocks, hipStream_t st, const DevTensor &d, unsigned threads = kBlock)
{
    const dim3 grid = d.grid3 ? dim3(d.cps, d.channels, d.outer) : dim3(blocks);
    unsigned channels = d.grid3 ? d.channels : 0u;
    const void *args[] = {&d.x, &d.y, &d.theta, &d.inner, &d.chunk, &channels, &d};
    (void)hipLaunchKernel((const void *)kernel, grid, dim3(threads), const_cast<void **>(args), 0, st);
}

static void launch_tensor(BackwardKernel kernel, unsigned blocks, hipStream_t st, const DevTensor &d)
{
    const dim3 grid = d.grid3 ? dim3(d.cps, d.channels, d.outer) : dim3(blocks);
    void *gx = d.flags & 1u ? nullptr : d.gx;
    unsigned channels = d.grid3 ? d.channels : 0u;
    const void *args[] = {&d.x, &d.gy, &gx, &d.theta, &d.inner, &d.chunk, &d.cps, &channels, &d};
    (void)hipLaunchKernel((const void *)kernel, grid, dim3(kBlock), const_cast<void **>(args), 0, st);
}

// Vectors in a whole chunk.
template <typename T> static unsigned chunk_vecs(const DevTensor &d) { return (d.chunk + VecOf<T>::N - 1) / VecOf<T>::N; }

// Calls f with the number of rows as a compile-time constant.  A kernel built for exactly the rows of the
// tensor issues no loads past the end of a chunk and runs through less code; short chunks feel both.
template <typename F> static void with_rows(int rows, F f)
{
    switch (rows) {
    case 1: return f(std::integral_constant<int, 1>());
    case 2: return f(std::integral_constant<int, 2>());
    case 3: return f(std::integral_constant<int, 3>());
    case 4: return f(std::integral_constant<int, 4>());
    default: return f(std::integral_constant<int, kMaxRows>());
    }
}

// Forward, us before -> with exactly one or two rows: 153600 FP32 elements 2.47 -> 2.31; 64x147 FP32 3.05 ->
// 2.65; 384x3456 FP32 3.31 -> 3.19.  With three rows exactness loses (3x128x4800 FP16: 3.42 -> 3.48), and
// so it does for wavefront units (15x384x1200 FP16: 6.70 -> 6.94), so those take kMaxRows.
template <typename T, int G, bool EARLY>
static void launch_forward_full(const DevTensor &d, unsigned blocks, hipStream_t st)
{
    constexpr int rows = G == 64 ? kMaxRows : (kChunkVecs + G - 1) / G;
    constexpr unsigned threads = G == 64 ? kBlock : G;
    if (!d.q) launch_tensor(forward_kernel<T, true, false, G, rows, EARLY>, blocks, st, d, threads);
    else if (d.y) launch_tensor(forward_kernel<T, true, true, G, rows, EARLY>, blocks, st, d, threads);
    else launch_tensor(forward_kernel<T, false, true, G, rows, EARLY>, blocks, st, d, threads);
}

// Whether a chunk is shared by kWideBlock threads.  The chunk is the same; its rows are requested, worked out and
// stored by twice the wavefronts, so what a wavefront still has to do when its last row has landed is shorter.  That
// pays in small launches, whose compute units have one or two blocks and would run one or two wavefronts per SIMD, and
// in those of many rounds; in between, where every compute unit holds four or five blocks, the smaller blocks end more
// evenly.  Buffers that no cache holds, us, kBlock / kWideBlock threads, blocks x vectors:
//   FP16  225 x 512 2.86 / 2.68   240 x 1280 3.72 / 3.52   256 x 603 3.33 / 3.12   384 x 1200 4.90 / 4.73
//         480 x 1280 5.49 / 5.20   540 x 1200 6.09 / 5.63   600 x 1200 6.29 / 6.05   660 x 1200 6.39 / 6.29
//         880 x 1200 7.90 / 8.12   960 7.62 / 8.40   1024 7.65 / 8.35   1280 9.75 / 10.87   1536 11.8 / 12.3
//         1800 x 1200 14.12 / 13.83   2560 18.5 / 18.2   3840 25.9 / 25.2   2000 x 600 9.07 / 8.35
//         3000 x 512 10.58 / 9.80   3000 x 375 8.58 / 8.68   4000 x 313 9.71 / 10.54 (three of eight wavefronts idle)
//         200 x 300 2.94 / 2.77   200 x 400 2.70 / 2.53   300 x 263 3.12 / 3.06   300 x 450 3.29 / 3.18   384 x 257 3.19 / 3.14
//         384 x 375 3.27 / 3.21   512 x 263 3.23 / 3.23   512 x 320 2.94 / 2.94   512 x 450 3.50 / 3.40   (no shape of 128 to 512
//         blocks of 257 to 512 vectors is slower in either type, three of eight wavefronts idle or not)
//   FP32  200 x 263 2.82 / 2.66   300 x 300 2.70 / 2.61   384 x 450 3.18 / 3.07   512 x 257 3.10 / 3.07;  200 x 600 2.66 / 2.71
//         512 x 576 3.30 / 3.28   512 x 1200 5.03 / 4.95   804 x 824 6.12 / 5.81   1024 x 1200 7.7 / 8.6
//         1800 x 1200 13.6 / 13.4   3000 x 640 12.35 / 11.95;   768 x 432 3.42 / 3.73 (one row each instead of two)
//   codes alone, FP16  128 x 603 3.22 / 3.08   240 x 1280 3.68 / 3.43   400 x 1200 4.53 / 4.21   768 x 1200 5.90 / 6.14
//         2000 x 600 7.58 / 8.21   3840 x 1200 20.2 / 20.9
// With more than kEarlyBlocks blocks theta goes in front of the rows there too (768 x 1200 FP16 6.68 / 6.73 without it and
// 6.44 with it, FP32 6.39 / 6.75 / 6.05; but 540 x 1200 5.63 without and 5.96 with it).  kEarlyBlocks stands where FP16 stops losing,
// us, without / with: 576 x 1200 5.97 / 6.14   600 x 1200 6.08 / 6.17   620 x 1200 6.20 / 6.22   640 x 1200 6.38 / 6.33   660 x 1200 6.42 /
// 6.41   680 x 1200 6.57 / 6.39   704 x 1200 6.70 / 6.38 (1100 vectors: from 600 on 1 to 5 % with it); FP32 gains from about 560 on
// (540 x 1200 5.63 / 5.80, 600 6.22 / 5.93, 660 6.55 / 6.03).
constexpr int kWideBlock = 2 * kBlock, kWideRows = (kChunkVecs + kWideBlock - 1) / kWideBlock;
constexpr unsigned kEarlyBlocks = 640, kWideFewBlocks = 512, kWideManyBlocks = 1800;
static bool wide_pays(unsigned blocks, unsigned vecs, bool codes)
{
    if (blocks <= kWideFewBlocks) return vecs > (unsigned)kBlock;
    if (codes) return false;
    return blocks <= kResidentBlocks ? vecs > 2u * kWideBlock : blocks >= kWideManyBlocks && vecs > kWideBlock * 7u / 8u;
}

template <typename T>
static void launch_forward_single(const DevTensor &d, unsigned blocks, hipStream_t st)
{
    const unsigned vecs = chunk_vecs<T>(d);
    if (d.wave_units) launch_forward_full<T, 64, false>(d, blocks, st);
    else if (wide_pays(blocks, vecs, d.q != nullptr)) {
        if (!d.q && vecs <= (unsigned)kWideBlock) launch_tensor(forward_kernel<T, true, false, kWideBlock, 1, false>, blocks, st, d, kWideBlock);
        else if (!d.q && vecs <= 2u * kWideBlock) launch_tensor(forward_kernel<T, true, false, kWideBlock, 2, false>, blocks, st, d, kWideBlock);
        else if (blocks > kEarlyBlocks) launch_tensor(forward_kernel<T, true, false, kWideBlock, kWideRows, true>, blocks, st, d, kWideBlock);
        else launch_forward_full<T, kWideBlock, false>(d, blocks, st);
    } else if (!d.q && d.rows == 1) launch_tensor(forward_kernel<T, true, false, kBlock, 1, false>, blocks, st, d);
    else if (!d.q && d.rows == 2) launch_tensor(forward_kernel<T, true, false, kBlock, 2, false>, blocks, st, d);
    else if (blocks > kResidentBlocks) launch_forward_full<T, kBlock, true>(d, blocks, st);
    else launch_forward_full<T, kBlock, false>(d, blocks, st);
}

int launch_forward(const KArgs &a, unsigned blocks, bool emit_q, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    if (a.table) {
        // Lists with codes run the code for kMaxRows rows whatever their chunks have, so that blocks of fewer rows wait
        // for loads that they do not need: there theta in front of the rows pays for whole chunks only.  us, in front /
        // behind: whole chunks 16x(2x128x9600) FP16 36.3 / 37.3, 6x(200x9600) 12.4 / 13.0, 8x(8x128x9600) FP32 120.1 /
        // 122.2; others 12x(128x4800) FP16 11.4 / 10.5, 64x(64x4800) 27.9 / 26.2, 22x(64x576) FP32 5.3 / 4.8.
        if (emit_q && a.whole && blocks > kResidentBlocks) launch(forward_multi_kernel<true, true>, blocks, st, a.table, a.n);
        else if (emit_q) launch(forward_multi_kernel<true, false>, blocks, st, a.table, a.n);
        else if (blocks > kResidentBlocks) launch(forward_multi_kernel<false, true>, blocks, st, a.table, a.n);
        else launch(forward_multi_kernel<false, false>, blocks, st, a.table, a.n);
    } else if (a.one.dtype == 0) {
        launch_forward_single<_Float16>(a.one, blocks, st);
    } else {
        launch_forward_single<float>(a.one, blocks, st);
    }
    return (int)hipGetLastError();
}

// Backward, us before -> with exactly the tensor's rows: 1x512x4800 FP16 (three rows) 5.1 -> 4.6; 64x576 FP32
// (one) 3.3 -> 2.9; 15x384x1200 FP16 (three, wavefront units) 11.5 -> 10.9.
template <typename T, int SHAPE>
static void launch_backward_typed(const DevTensor &d, unsigned blocks, bool fused_finalize, hipStream_t st)
{
    if (!fused_finalize) {
        launch_tensor(backward_kernel<T, false, SHAPE, kMaxRows>, blocks, st, d);
        return;
    }
    with_rows(d.rows, [&](auto rows) {
        launch_tensor(backward_kernel<T, true, SHAPE, decltype(rows)::value>, blocks, st, d);
    });
}

// The burst schedule (backward_chunk_short) pays in launches that are resident at once and move much data: its
// arithmetic lies in front of the last loads, but it is more arithmetic and more registers.  Since gx goes out behind
// the sum in both schedules, FP16 gains by it only where each compute unit has a fourth block, and loses with three
// (registers let it hold four blocks of burst FP16, seven interleaved).  Measured against the interleaved schedule, us,
// burst / interleaved:
//   FP16  300 x 1200 x 2 (600 blocks) 9.0 / 8.6   660 9.07 / 8.65   768 x 1200 vectors 9.3 to 10.4 / 9.4   768 x 800 7.6 / 7.15
//         800 x 1200 10.62 / 10.76   800, two units apart 10.89 / 11.10   960 11.74 / 12.05   1000 x 1000 10.14 / 10.31
//         1024 x 1200 12.5 / 12.5
//   FP32  768 x 1200 9.53 / 9.77   512 x 1200 6.9 / 7.1   400 x 1200 6.1 / 6.3   768 x 600 4.95 / 5.3
//         512 x 600 4.2 / 4.3   400 x 600 4.1 / 4.0   768 x 432 5.0 / 4.9   64 x 144 3.0 / 2.9
// Where the sums are gathered it is not used, and the kernel with it leaves the gathering out (one scale, 153600 FP32
// elements 4.13 / 3.87, 921600 FP16 4.77 / 4.40, 4915200 FP16 8.6 / 8.0).
template <typename T> static bool burst_pays(const DevTensor &d, unsigned blocks)
{
    const bool half = sizeof(T) == 2;
    return blocks <= (half ? kBurstMostBlocksF16 : kBurstMostBlocksF32) && blocks >= (half ? kBurstLeastBlocksF16 : kBurstLeastBlocksF32) &&
           chunk_vecs<T>(d) >= (half ? kBurstLeastVecsF16 : kBurstLeastVecsF32);
}

template <typename T>
static void launch_backward_shaped(const DevTensor &d, unsigned blocks, bool fused_finalize, hipStream_t st)
{
    const bool gathered = fused_finalize && d.outer * d.cps > kTreeBlocks;
    if (d.wave_units) launch_backward_typed<T, 1>(d, blocks, fused_finalize, st);
    else if (fused_finalize && !gathered && burst_pays<T>(d, blocks)) {
        if (d.rows <= 3) launch_tensor(backward_kernel<T, true, 2, 3>, blocks, st, d);
        else if (d.rows == 4) launch_tensor(backward_kernel<T, true, 2, 4>, blocks, st, d);
        else launch_tensor(backward_kernel<T, true, 2, kMaxRows>, blocks, st, d);
    } else launch_backward_typed<T, 0>(d, blocks, fused_finalize, st);
}

static void launch_backward_single(const DevTensor &d, unsigned blocks, bool fused_finalize, hipStream_t st)
{
    if (d.dtype == 0) launch_backward_shaped<_Float16>(d, blocks, fused_finalize, st);
    else launch_backward_shaped<float>(d, blocks, fused_finalize, st);
}

int launch_backward(const KArgs &a, unsigned blocks, bool fused_finalize, void *stream)
{
    hipStream_t st = (hipStream_t)stream;
    if (a.table) {
        if (fused_finalize) launch(backward_multi_kernel<true>, blocks, st, a.table, a.n, a.bias);
        else launch(backward_multi_kernel<false>, blocks, st, a.table, a.n, a.bias);
    } else {
        launch_backward_single(a.one, blocks, fused_finalize, st);
    }
    return (int)hipGetLastError();
}

int launch_finalize(const KArgs &a, unsigned total_channels, void *stream)
{
    hipLaunchKernelGGL(finalize_kernel, dim3(total_channels), dim3(kBlock), 0, (hipStream_t)stream, a);
    return (int)hipGetLastError();
}

int launch_scale_only(const KArgs &a, unsigned total_channels, void *stream)
{
    unsigned blocks = (total_channels + kBlock - 1) / kBlock;
    hipLaunchKernelGGL(scale_kernel, dim3(blocks), dim3(kBlock), 0, (hipStream_t)stream, a, total_channels);
    return (int)hipGetLastError();
}

int launch_fill_zero(void *p, size_t bytes, void *stream)
{
    size_t words = bytes / 4;
    if (words == 0) return 0;
    size_t want = (words + kBlock - 1) / kBlock;
    unsigned blocks = (unsigned)(want < 4096 ? want : 4096);
    hipLaunchKernelGGL(fill_zero_kernel, dim3(blocks), dim3(kBlock), 0, (hipStream_t)stream,
                       (unsigned *)p, words);
    return (int)hipGetLastError();
}

}  // namespace fq
