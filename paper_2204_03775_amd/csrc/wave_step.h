// libwave.so: time stepping of the 3-D acoustic wave equation with the
// 25-point, 8th-order Laplacian inside a leapfrog update (paper Section III:
// Eq. 2, the Laplacian and Algorithm 1), written for MI355X (gfx950, CDNA4,
// wave64).  The C ABI is declared in include/wave.h.
//
// Kernel design.  The paper maps X and Y onto its processor grid and keeps
// the whole Z column in each processor's memory (Section IV-B); a GPU has a
// memory hierarchy instead, so the mapping here is the usual 2.5-D one:
//   - a work-group owns an x-y tile and a range of z planes and marches
//     through them;
//   - each thread owns 4 consecutive x cells in RY rows and keeps its z
//     column z-4 .. z+4 in a register queue (the GPU counterpart of the
//     paper's z update from local memory, Section IV-C);
//   - the centre plane of the tile, with a 4-cell halo in x and y, is
//     staged in LDS (double buffered: one barrier per plane) and the x and
//     y taps are read from there;
//   - the next plane, the halo and u^{n-1}, k are prefetched one plane
//     ahead so that HBM reads overlap the arithmetic;
//   - sponge, source injection and receiver sampling are fused: the
//     update, the source add and a per-work-group receiver epilogue happen
//     in the same launch.
// The step is bound by HBM bandwidth (about 3 flop per byte against a ridge
// near 20 for FP32 vector math), so nothing here uses the matrix cores.
//
// Laplacian form.  With FP32 fields the Laplacian is evaluated as
//   sum_a sum_m (c_m / h_a^2) (u(+m e_a) + u(-m e_a) - 2 u),
// which equals the paper's form because c_0 = -2 sum c_m, and which maps a
// constant to exactly zero whatever the rounding of the FP32 weights.  The
// classic form c_0 u + sum c_m (...) with FP32-rounded weights does not,
// and the small spurious mass term it leaves shifts the phase by about
// 2e-5 over five wavelengths at 17 cells per wavelength.  16-bit storage
// rounds each stored value far more coarsely than that, so those kernels
// keep the classic form and its 12 fewer operations per cell.
//
// Storage.  Fields are FP32, or FP16 / BF16 with FP32 arithmetic: a 16-bit
// field holds x * 2^-e for one exponent e per time level, chosen on the
// device when the level is written so that the largest value stays below
// 2^14 (see step_scales).  Decoding multiplies by 2^e, which is exact.

#pragma once

#include <type_traits>
#include <utility>

#include "wave_dev.h"
#include "wave_kernels.h"

namespace wavek {

__device__ __forceinline__ float src_value(const StepArgs &a)
{
    return a.src_ptr ? a.src_ptr[0] : a.src_val;
}

// x * g rounded on its own.  The adjoint scales every loaded value by the
// sponge factor; if that product were contracted into the first sum that
// uses it (an FMA), the value would enter that sum unrounded and the other
// operand rounded, so the result would depend on which of u[z+m], u[z-m]
// was loaded last, i.e. on the direction of the z-march.
__device__ __forceinline__ float mul_rounded(float x, float g)
{
#pragma clang fp contract(off)
    return x * g;
}

// Work-groups are handed to the 8 XCDs round-robin by block index (the
// starting XCD follows on from the previous launch, so blocks with equal
// b % 8 share an XCD, not necessarily XCD b % 8); map block b to logical
// work-group (b % 8) * (G / 8) + b / 8 so that each XCD gets a contiguous
// run of neighbouring tiles whose halos share its L2.
// (G, the grid, is the work-groups rounded up to a multiple of 8.)
__device__ __forceinline__ int logical_wg(const StepArgs &a)
{
    const int b = blockIdx.x;
    const int per = (a.nwg + 7) >> 3;
    return (b & 7) * per + (b >> 3);
}

// ---------------------------------------------------------------------------
// storage formats

template <int KIND>
struct Store;
template <>
struct Store<WAVE_F32> {
    static constexpr bool scaled = false;
    static constexpr bool uv = false;
    static constexpr unsigned bytes = 4;
};
template <>
struct Store<WAVE_F16> {
    static constexpr bool scaled = true;
    static constexpr bool uv = false;
    static constexpr unsigned bytes = 2;
    static __device__ __forceinline__ float dec(unsigned bits)
    {
        return (float)__builtin_bit_cast(_Float16, (unsigned short)bits);
    }
    static __device__ __forceinline__ unsigned enc(float x)
    {
        return __builtin_bit_cast(unsigned short, (_Float16)x);
    }
    // two values packed low, high: one packed conversion (round to nearest
    // even, as the scalar one) instead of two
    static __device__ __forceinline__ unsigned enc2(float lo, float hi)
    {
        typedef float f2v __attribute__((ext_vector_type(2)));
        typedef _Float16 h2v __attribute__((ext_vector_type(2)));
        const f2v f = {lo, hi};
        return __builtin_bit_cast(unsigned, __builtin_convertvector(f, h2v));
    }
};
template <>
struct Store<WAVE_BF16> {
    static constexpr bool scaled = true;
    static constexpr bool uv = false;
    static constexpr unsigned bytes = 2;
    static __device__ __forceinline__ float dec(unsigned bits) { return __uint_as_float(bits << 16); }
    static __device__ __forceinline__ unsigned enc(float x)
    {
        return __builtin_bit_cast(unsigned short, (__bf16)x);
    }
    static __device__ __forceinline__ unsigned enc2(float lo, float hi) { return enc(lo) | (enc(hi) << 16); }
};
// u and its step change d = u^n - u^{n-1}, same 16-bit encodings
template <>
struct Store<WAVE_F16_UV> : Store<WAVE_F16> {
    static constexpr bool uv = true;
};
template <>
struct Store<WAVE_BF16_UV> : Store<WAVE_BF16> {
    static constexpr bool uv = true;
};

// Vector arithmetic (first) or LDS accesses stay on their side of this point.
__device__ __forceinline__ void in_order() { __builtin_amdgcn_sched_barrier(0x3f4); }
__device__ __forceinline__ void reads_in_order() { __builtin_amdgcn_sched_barrier(0x7f); }

// Raw buffer access.  A buffer resource covers one plane of one field; any
// byte offset at or past its size reads as zero and drops stores, which is
// how out-of-range tile cells are masked without branches.
typedef unsigned u4raw __attribute__((vector_size(16)));
typedef unsigned u2raw __attribute__((vector_size(8)));
constexpr int kRsrcWord3 = 0x00020000;  // 32-bit data format, raw (stride 0) access
constexpr unsigned kOff = 0xffffffffu;  // an offset outside every resource

__device__ __forceinline__ __amdgpu_buffer_rsrc_t plane_rsrc(const void *field, long long plane_bytes,
                                                            int z)
{
    const char *p = reinterpret_cast<const char *>(field) + (long long)(z + kGhost) * plane_bytes;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p), (short)0, (int)plane_bytes,
                                             kRsrcWord3);
}

// A resource for the plane at p, empty (loads return zero, stores are
// dropped) when it is not to be touched.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t rsrc_at(const char *p, long long plane_bytes, bool live = true)
{
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p), (short)0, live ? (int)plane_bytes : 0,
                                             kRsrcWord3);
}

// Compiles to nothing, but code after it in a branch is not turned into
// selects: for wave-uniform branches that are rarely taken.
__device__ __forceinline__ void keep_branch() { asm volatile(""); }

// The same for a plane the stencil may reach outside the grid (z < 0 or
// z >= nz): a ghost plane gets an empty resource, so its loads return the
// zeros it holds without reading memory.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t stencil_plane_rsrc(const void *field, long long plane_bytes,
                                                                    int z, int nz)
{
    const char *p = reinterpret_cast<const char *>(field) + (long long)(z + kGhost) * plane_bytes;
    const int size = (z >= 0 && z < nz) ? (int)plane_bytes : 0;
    return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p), (short)0, size, kRsrcWord3);
}

// Cache policy of a buffer access (gfx950 encoding of the aux operand):
// bit 1 = non-temporal.  u^{n-1} and k are read exactly once per step and
// u^{n+1} is not read again in the step, so they are streamed
// non-temporally; u^n is read by the neighbouring tiles as their halo and
// keeps the default policy, so it stays resident in L2.
typedef double dv2 __attribute__((ext_vector_type(2)));

constexpr int kKeep = 0;
constexpr int kStream = 2;
// device scope (sc1): the load misses the CU's L1 and is served by the L2,
// so it sees what other CUs of the same XCD stored (their stores have
// reached the L2 before they signal completion)
constexpr int kCoh = 16;

// Four consecutive cells as stored (16 bytes of FP32, 8 bytes of 16-bit
// values), and decoded to FP32 (times `scale` for 16-bit data).  Values
// loaded ahead of their use are held raw, so that a 16-bit prefetch holds
// half the registers of its decoded form.
template <int KIND>
using Raw4 = std::conditional_t<KIND == WAVE_F32, u4raw, u2raw>;

template <int KIND, int POL>
__device__ __forceinline__ Raw4<KIND> load_raw4(__amdgpu_buffer_rsrc_t r, unsigned off)
{
    if constexpr (KIND == WAVE_F32)
        return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, POL);
    else
        return __builtin_amdgcn_raw_buffer_load_b64(r, off, 0, POL);
}

template <int KIND>
__device__ __forceinline__ f4 decode4(const Raw4<KIND> &v, float scale = 1.f)
{
    f4 o;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        if constexpr (KIND == WAVE_F32)
            o.v[e] = __uint_as_float(v[e]);
        else
            o.v[e] = Store<KIND>::dec((v[e >> 1] >> (16 * (e & 1))) & 0xffffu) * scale;
    }
    return o;
}

template <int KIND, int POL>
__device__ __forceinline__ f4 load4(__amdgpu_buffer_rsrc_t r, unsigned off, float scale)
{
    return decode4<KIND>(load_raw4<KIND, POL>(r, off), scale);
}

template <int KIND>
__device__ __forceinline__ void store4(__amdgpu_buffer_rsrc_t r, unsigned off, const f4 &v, float inv)
{
    if constexpr (KIND == WAVE_F32) {
        u4raw w;
#pragma unroll
        for (int e = 0; e < 4; ++e)
            w[e] = __float_as_uint(v.v[e]);
        __builtin_amdgcn_raw_buffer_store_b128(w, r, off, 0, kStream);
    } else {
        u2raw w;
#pragma unroll
        for (int h = 0; h < 2; ++h)
            w[h] = Store<KIND>::enc2(v.v[2 * h] * inv, v.v[2 * h + 1] * inv);
        __builtin_amdgcn_raw_buffer_store_b64(w, r, off, 0, kStream);
    }
}

// Element read outside the hot loop (receivers, exports).
template <int KIND>
__device__ __forceinline__ float read_elem(const void *f, long long i, float scale)
{
    if constexpr (KIND == WAVE_F32)
        return static_cast<const float *>(f)[i];
    else
        return Store<KIND>::dec(static_cast<const unsigned short *>(f)[i]) * scale;
}

// Scales of one step with 16-bit storage.  u^{n+1} is bounded by
// 7 max(|u^n|, |u^{n-1}|) + |s_n| (2 + 1 from the time levels, 4 from
// k |lap| under the stability limit, G <= 1); its exponent is chosen so
// that 8 M + |s_n| < 2^(e + 14), which leaves a factor 4 below the FP16
// maximum.  All work-groups compute the same value from the same inputs.
struct Scales {
    float cur, prev, out_inv, out;
    int e_out;
};

// slot s of the running maximum of level n (float bits), each on a cache
// line of its own
__device__ __forceinline__ unsigned *max_slot(const StepArgs &a, int n, int s)
{
    return a.maxes + ((n & 3) * kMaxSlots + s) * kMaxStride;
}

// The same step in the stored (scaled) units.  With U, P, K the decoded
// but unscaled u^n, u^{n-1}, k and every scale a power of two, the stored
// u^{n+1} is
//   O = g (fma(K, LAP_C(U), 2A U) - g B P),
//   A = sc_cur / sc_out, B = sc_prev / sc_out, C = k_scale * A,
// with LAP_C the Laplacian whose weights are multiplied by C.  Scaling by
// a power of two commutes with every FP32 rounding, so this is bit for bit
// the decode -> compute -> encode sequence, without the per-value
// multiplies.
//
// With u-and-change storage the second input is D, the stored d^n =
// u^n - u^{n-1} (exponent one above u^n's), and u^{n-1} in output units is
// A U - B D with B = sc_d / sc_out; the same expression follows.  The new
// change d^{n+1} = u^{n+1} - u^n is formed in FP32 before either is
// rounded and stored with the exponent of u^{n+1} plus one (it is bounded
// by |u^{n+1}| + |u^n| < 2^(e + 15)).
struct Folded {
    Coefs c;       // weights times C
    float two_a;   // 2 A
    float b;       // B
    float a;       // A
};

__device__ __forceinline__ Folded fold_scales(const Coefs &c, const Scales &sc, float k_scale)
{
    Folded f;
    const float A = sc.cur * sc.out_inv;
    const float C = k_scale * A;
    f.c.ctr = c.ctr * C;
#pragma unroll
    for (int m = 0; m < 4; ++m) {
        f.c.cx[m] = c.cx[m] * C;
        f.c.cy[m] = c.cy[m] * C;
        f.c.cz[m] = c.cz[m] * C;
    }
    f.two_a = 2.f * A;
    f.b = sc.prev * sc.out_inv;
    f.a = A;
    return f;
}

// The running maxima of levels n and n - 1 are kept in kMaxSlots slots each
// (see fold_max): every wave reads one slot per lane, half a wave per level,
// and reduces them.
template <int KIND>
__device__ __forceinline__ Scales step_scales(const StepArgs &a)
{
    static_assert(2 * kMaxSlots == 64, "one slot per lane");
    const int n = a.step;
    const int lane = threadIdx.x & 63;
    unsigned mb = *max_slot(a, lane < kMaxSlots ? n : n + 3, lane & (kMaxSlots - 1));
#pragma unroll
    for (int d = 32; d > 0; d >>= 1)
        mb = max(mb, (unsigned)__shfl_xor((int)mb, d));
    const float m = __uint_as_float(__builtin_amdgcn_readfirstlane(mb));
    const float s = a.src_z >= 0 ? fabsf(src_value(a)) : 0.f;
    const float bound = 8.f * m + s;
    int e = 0;
    if (bound > 0.f && bound < INFINITY) {
        int ex;
        (void)frexpf(bound, &ex);  // bound < 2^ex
        e = min(max(ex - kScaledTopExp, -110), 110);
    }
    Scales sc;
    sc.cur = ldexpf(1.f, a.exps[n & 3]);
    // second input: u^{n-1}, or d^n (exponent of u^n plus one)
    sc.prev = Store<KIND>::uv ? ldexpf(1.f, a.exps[n & 3] + 1) : ldexpf(1.f, a.exps[(n + 3) & 3]);
    sc.out = ldexpf(1.f, e);
    sc.out_inv = ldexpf(1.f, -e);
    sc.e_out = e;
    return sc;
}

// Publish this step's exponent and clear the max slots the next step fills
// after this one (level n + 2's, which no launch of this step reads).
__device__ __forceinline__ void publish_scale(const StepArgs &a, const Scales &sc, int lid, int tid)
{
    if (lid == 0) {
        if (tid == 0)
            a.exps[(a.step + 1) & 3] = sc.e_out;
        if (tid < kMaxSlots)
            *max_slot(a, a.step + 2, tid) = 0u;
    }
}

// Fold a per-thread max |u^{n+1}| into the level's running maximum: a
// reduction across each wave, one across the work-group's waves, then one
// atomic (on the float bit pattern, valid for non-negative values) into slot
// lid % kMaxSlots.  Atomics on one address from work-groups on 8 XCDs are
// served one after another in the memory behind the L2s, about 10 ns each,
// and a launch ends with all of them: one per wave on a single address (2048
// a launch) took 20 us of the 30 us step of 128^3 FP16 u-and-change and 9 of
// the 69 us one of 320x288x272 FP16 (512^3: 259 -> 250; with the plans and
// the plane loop as they are, the first two steps now take 8.5 and 40 us).
__device__ __forceinline__ void fold_max(const StepArgs &a, int lid, float m)
{
    __shared__ float part[16];
#pragma unroll
    for (int d = 32; d > 0; d >>= 1)
        m = fmaxf(m, __shfl_xor(m, d));
    const int wave = threadIdx.x >> 6, waves = (blockDim.x + 63) >> 6;
    if ((threadIdx.x & 63) == 0)
        part[wave] = m;
    __syncthreads();
    if (threadIdx.x == 0) {
        for (int w = 1; w < waves; ++w)
            m = fmaxf(m, part[w]);
        if (m > 0.f)
            atomicMax(max_slot(a, a.step + 1, lid & (kMaxSlots - 1)), __float_as_uint(m));
    }
}

// n / d for the tile numbers: the high word of (n + 1) m with m =
// floor((2^32 - 1) / d), exact for (n + 1) d <= 2^32 (the host sets m = 0
// beyond), instead of a division's 30 instructions at the head of every launch.
__device__ __forceinline__ int div_by(int n, int d, unsigned m)
{
    unsigned q = __umulhi((unsigned)n + 1u, m);
    if (__builtin_expect(m == 0, 0)) {
        keep_branch();
        q = (unsigned)n / (unsigned)d;
    }
    return (int)q;
}

// Receiver epilogue: after the whole tile column is written, copy the
// receivers this work-group owns (r0 .. r1 - 1 of its tables, looked up
// before the march) into the trace row.  A thread's first table entries are
// loaded before the wait for the column's stores, so that on small grids,
// where a launch is a chain of memory latencies, they add none to it.
template <int KIND>
__device__ __forceinline__ void sample_receivers(const StepArgs &a, int r0, int r1, int tid, int nt, float scale)
{
    if (r0 == r1)
        return;
    int i = r0 + tid;
    long long off = 0;
    int idx = 0;
    if (i < r1) {
        off = a.rec_off[i];
        idx = a.rec_idx[i];
    }
    __syncthreads();
    while (i < r1) {
        a.trace_row[idx] = read_elem<KIND>(a.out, off, scale);
        i += nt;
        if (i < r1) {
            off = a.rec_off[i];
            idx = a.rec_idx[i];
        }
    }
}

// The adjoint step's counterpart: once the tile column holds phi^{m-1}, add
// k * (sum of the trace derivatives of row m-2) at the receiver cells this
// work-group owns (rec_start ranges over the cells: rec_off the cell's
// offset, rec_idx its range in inj_rec, the receivers in a fixed order).
// A launch of its own took 4.7 us a step plus the gap before it.
__device__ __forceinline__ void inject_cells(const StepArgs &a, int r0, int r1, int tid, int nt)
{
    if (r0 == r1)
        return;
    __syncthreads();
    for (int c = r0 + tid; c < r1; c += nt) {
        float s = 0.f;
        for (int i = a.rec_idx[c]; i < a.rec_idx[c + 1]; ++i)
            s += a.trace_row[a.inj_rec[i]];
        const long long o = a.rec_off[c];
        float *p = static_cast<float *>(a.out) + o;
        *p = fmaf(static_cast<const float *>(a.k)[o], s, *p);
    }
}

// Calls f(integral_constant<int, S>) for S = B, B+1, ... < E while f
// returns true: a loop unrolled at compile time, so every index that
// depends on S is a constant and register arrays stay in registers.
template <int B, int E, class F>
__device__ __forceinline__ void static_for_while(F &&f)
{
    if constexpr (B < E) {
        if (f(std::integral_constant<int, B>{}))
            static_for_while<B + 1, E>(f);
    }
}

// ---------------------------------------------------------------------------
// the step

// One work-group's share of a step: the tile and z-chunk numbered `lid`
// (tiles x fastest, then y, then chunks) of the grid described by `a`.
// DRAIN: the march starts when every load of the prologue has arrived (see there).
template <int KIND, int TXV, int TY, int RY, int MODE = kFwd, bool COH = false, bool CACHED = false, bool DRAIN = false>
__device__ __forceinline__ void tile_step(const StepArgs &a, int lid)
{
    constexpr int NT = TXV * TY;
    constexpr int TYR = TY * RY;             // tile rows
    // float4 per LDS row: one halo float4 each side.  A wave of a 16-wide tile
    // reads four rows at once, without bank conflicts only if they lie a
    // multiple of 16 float4 apart (rows of 18: 42 % of the LDS cycles were
    // conflicts; rows of 32: 11 %)
    constexpr int LW = TXV == 16 ? 32 : TXV + 2;
    constexpr int LH = TYR + 8;              // LDS rows: 4 halo rows each side
    constexpr int NH = 8 * TXV + 2 * TYR;    // halo float4 per plane
    constexpr int HPT = (NH + NT - 1) / NT;  // halo float4 per thread
    constexpr int QS = 10;                   // queue slots: 9 live planes + 1 being filled
    constexpr unsigned EB = Store<KIND>::bytes;
    constexpr bool SCALED = Store<KIND>::scaled;
    constexpr bool UV = Store<KIND>::uv;          // second input is d^n, also written
    constexpr bool LAP = MODE == kLap;            // forward step that also stores lap u^n
    constexpr bool FUS = MODE == kFus;            // adjoint step + the imaging terms of the levels it reads
    constexpr bool ADJ = MODE == kAdj || FUS;     // the stencil field is phi, scaled by G on load
    static_assert(MODE == kFwd || KIND == WAVE_F32, "Laplacian stores and adjoint steps are FP32 only");
    // load policies of the wave fields (k never changes during a run);
    // CACHED: u^{n-1} and k too keep the default policy, for grids whose
    // fields fit in the memory-side cache together.  The step change d^n of
    // the u-and-change forms keeps it too: with the z-march reversed every
    // launch, the d planes one launch touches last are the next one's first,
    // and the memory-side cache serves part of them (512^3: FP16 513 -> 526,
    // BF16 519 -> 546 Gpts/s; also keeping k was slower, and so was keeping
    // u^{n-1} and k in the two-level forms)
    constexpr int PK = kKeep | (COH ? kCoh : 0);
    constexpr int PS = ((CACHED || UV) ? kKeep : kStream) | (COH ? kCoh : 0);
    constexpr int PKK = CACHED ? kKeep : kStream;
    __shared__ f4 lds[2][LH][LW];

    const int rest = div_by(lid, a.ntx, a.mtx), tx = lid - rest * a.ntx;
    const int ch = div_by(rest, a.nty, a.mty), ty = rest - ch * a.nty;
    const int z0 = ch * a.zc;
    const int z1 = min(z0 + a.zc, a.nz);
    // the chunk's planes in march order: march position l is plane zp(l)
    // (positions -4 .. -1 and len .. len + 3 are the chunk's z halo)
    const int len = z1 - z0;
    const bool down = a.zdown & 1;
    const int zb = down ? z1 - 1 : z0, dz = down ? -1 : 1;
    auto zp = [&](int l) { return zb + dz * l; };

    const int tid = threadIdx.x;
    const int lx = tid % TXV;
    const int ly = tid / TXV;
    const int xq0 = tx * TXV;          // first 4-cell column of the tile
    const int y0 = ty * TYR;           // first row of the tile
    const int xq = xq0 + lx;           // this thread's 4-cell column
    const int x = 4 * xq;

    // Only 4-cell groups holding interior cells are read (the ragged last
    // group's right-ghost lanes with them); ghost rows, columns and planes
    // hold zero, and their loads are masked so that they return zero without
    // reading memory.
    const bool col_interior = x < a.nx;
    // whether this tile holds the grid's ragged last group (uniform)
    const bool ragged = (a.nx & 3) != 0 && tx == a.ntx - 1;

    // own rows: byte offsets within a plane (kOff when masked)
    int row[RY];
    bool row_int[RY];
    unsigned own_ld[RY], own_in[RY];
#pragma unroll
    for (int r = 0; r < RY; ++r) {
        row[r] = y0 + ly * RY + r;
        row_int[r] = col_interior && row[r] < a.ny;
        const unsigned b = EB * unsigned((row[r] + kGhost) * a.px + a.x0 + x);
        own_in[r] = row_int[r] ? b : kOff;
        own_ld[r] = own_in[r];
    }

    // halo items of this thread: 8 rows of the tile's width above and below
    // it, then the columns left and right (selects, no branches: a small
    // grid's launch is as long as one wave's instructions)
    auto halo_item = [](int i, int &hr, int &hc) {
        const int band = i / TXV, j = i - 8 * TXV;
        const bool rows = i < 8 * TXV;
        hr = rows ? band - 4 + (band < 4 ? 0 : TYR) : j % TYR;
        hc = rows ? i % TXV : j < TYR ? -1 : TXV;
    };
    unsigned h_b[HPT];
    int h_lds[HPT];  // flat LDS index (row * LW + col), -1 when unused
#pragma unroll
    for (int h = 0; h < HPT; ++h) {
        int hr, hc;
        halo_item(tid + h * NT, hr, hc);
        const bool use = tid + h * NT < NH;
        h_lds[h] = use ? (hr + 4) * LW + (hc + 1) : -1;
        const int gy = y0 + hr;
        const int gq = xq0 + hc;
        const bool ok = use & ((unsigned)gy < (unsigned)a.ny) & ((unsigned)gq < (unsigned)a.nxq);
        h_b[h] = EB * unsigned((gy + kGhost) * a.px + a.x0 + 4 * gq) | (ok ? 0u : kOff);
    }
    const long long pbytes = a.plane * (long long)EB;
    const __amdgpu_buffer_rsrc_t gz_r = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(a.gz), (short)0, a.nz * (int)sizeof(float), kRsrcWord3);

    // register queue: at phase s the plane of march position l - 4 + i
    // lives in slot (s + i) % QS
    auto gz_at = [&](int z) {  // g_z, zero outside the interior (reads nothing there)
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(gz_r, 4u * unsigned(z), 0, 0));
    };
    // The prologue issues every load of the first plane before anything that
    // waits for one (scales, sponge factors, the source's value), and gets
    // there in few instructions: a small grid's launch is the serial chain of
    // one wave, half of it instructions and half memory latency, and the first
    // load used to be the 290th instruction (now the 140th).  64^3 under graph
    // replay 3.59 -> 3.43 us a step, 37 x 21 x 19 3.39 -> 3.18; FP16 at 64^3
    // 5.39 -> 5.22, FP16 u and step change at 128^3 9.08 -> 8.87; 256^3 and up
    // as before.
    f4 q[QS][RY];
    float gzi[ADJ ? 8 : 1];
    const long long zstep = down ? -pbytes : pbytes;
    const long long zfirst = (long long)(zp(0) + kGhost) * pbytes;
    const char *pq = reinterpret_cast<const char *>(a.cur) + zfirst - 4 * zstep;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int zi = zp(i - 4);
        const __amdgpu_buffer_rsrc_t rc = rsrc_at(pq, pbytes, (unsigned)zi < (unsigned)a.nz);
        pq += zstep;
#pragma unroll
        for (int r = 0; r < RY; ++r)
            q[i][r] = load4<KIND, PK>(rc, own_ld[r], 1.f);
        if constexpr (ADJ)
            gzi[i] = gz_at(zi);
    }

    // values of the next plane, loaded one plane ahead into the set of the
    // other parity (no copies, so no wait before the next loads are issued)
    Raw4<KIND> pv[2][RY], kv[2][RY], hv[2][HPT];
    // fused mode: the Laplacians of the two forward levels, and the sum
    Raw4<WAVE_F32> lv[FUS ? 2 : 1][2][RY];
    dv2 gacc[FUS ? 2 : 1][RY][2];
    const int lbytes = (int)(a.lplane * 4);
    const bool two = FUS && a.dlt != nullptr;  // also the term of the level before (phi^{m+1})
    const bool keep_sum = FUS && !a.first;     // the first term overwrites the accumulator
    unsigned own_lap[RY];
#pragma unroll
    for (int r = 0; r < RY; ++r)
        own_lap[r] = row_int[r] ? 4u * unsigned(row[r] * a.lpx + x) : kOff;
    auto lap_rsrc = [&](const void *f, int z, bool live) {
        const char *p = reinterpret_cast<const char *>(f) + (long long)z * lbytes;
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<char *>(p), (short)0, live ? lbytes : 0, kRsrcWord3);
    };
    // an accumulator cell group is two aligned 16-byte pairs
    auto sum_at = [&](int z, int r) {
        return reinterpret_cast<dv2 *>(a.grad + (long long)z * a.lplane + own_lap[r] / 4);
    };
    float gzv[2], gzq[2];  // FP32: g_z of the plane, and (adjoint) of the queue plane four positions on
    // Addresses of the planes being loaded and written.  16-bit storage
    // advances them by one plane per iteration, two scalar adds per field in
    // place of the multiplies of an absolute address (83 -> 54 scalar
    // instructions a plane: 512^3 FP16 u-and-change 250 -> 244 us, 256^3 FP16
    // 32.0 -> 30.4); the FP32 kernels, which have issue slots to spare, run
    // 0.5-1 % faster with absolute ones (256^3 39.5 against 39.8 us).
    constexpr bool INC = SCALED;
    const char *ph = reinterpret_cast<const char *>(a.cur) + zfirst;
    const char *pp = reinterpret_cast<const char *>(UV ? a.dlt : a.nxt) + zfirst;
    const char *pk = reinterpret_cast<const char *>(a.k) + zfirst;
    const char *po = reinterpret_cast<const char *>(a.out) + zfirst;
    const char *pd = UV ? reinterpret_cast<const char *>(a.dlt) + zfirst : nullptr;
    const int nq = min(len, down ? z1 - 4 : a.nz - 4 - z0);  // positions whose queue plane is in the grid
    // loads march position l, which must follow the one loaded before; past
    // the chunk's end the last position is loaded again (and goes unused)
    auto prefetch = [&](int l, int slot, int set) {
        if constexpr (!INC)
            l = min(l, len - 1);
        const int z = zp(INC ? min(l, len - 1) : l);
        const __amdgpu_buffer_rsrc_t rq =
            INC ? rsrc_at(pq, pbytes, l < nq) : stencil_plane_rsrc(a.cur, pbytes, zp(l + 4), a.nz);
        const __amdgpu_buffer_rsrc_t rp = INC ? rsrc_at(pp, pbytes) : plane_rsrc(UV ? a.dlt : a.nxt, pbytes, z);
        const __amdgpu_buffer_rsrc_t rk = INC ? rsrc_at(pk, pbytes) : plane_rsrc(a.k, pbytes, z);
        const __amdgpu_buffer_rsrc_t rh = INC ? rsrc_at(ph, pbytes) : plane_rsrc(a.cur, pbytes, z);
#pragma unroll
        for (int r = 0; r < RY; ++r) {
            q[slot][r] = load4<KIND, PK>(rq, own_ld[r], 1.f);
            pv[set][r] = load_raw4<KIND, PS>(rp, own_in[r]);
            kv[set][r] = load_raw4<KIND, PKK>(rk, own_in[r]);
        }
#pragma unroll
        for (int h = 0; h < HPT; ++h)
            hv[set][h] = load_raw4<KIND, PK>(rh, h_b[h]);
        if constexpr (FUS) {
            const __amdgpu_buffer_rsrc_t r0 = lap_rsrc(a.aux, z, true), r1 = lap_rsrc(a.dlt, z, two);
#pragma unroll
            for (int r = 0; r < RY; ++r) {
                lv[set][0][r] = load_raw4<WAVE_F32, kStream>(r0, own_lap[r]);
                lv[set][1][r] = load_raw4<WAVE_F32, kStream>(r1, own_lap[r]);
                // Each cell of the sum is read and written once per launch, but
                // with the z-march reversed every launch the planes a launch
                // touches last are the first the next one touches: the default
                // cache policy lets the memory-side cache serve part of it
                gacc[set][r][0] = gacc[set][r][1] = dv2{0.0, 0.0};
                if (keep_sum && row_int[r]) {
                    const dv2 *gp = sum_at(z, r);
                    gacc[set][r][0] = gp[0];
                    gacc[set][r][1] = gp[1];
                }
            }
        }
        if constexpr (!SCALED)
            gzv[set] = gz_at(z);
        if constexpr (ADJ)
            gzq[set] = gz_at(zp(l + 4));
        if constexpr (INC) {
            const long long st = l + 1 < len ? zstep : 0;
            pq += st;
            ph += st;
            pp += st;
            pk += st;
        }
    };
    prefetch(0, 8, 0);
    // 16-bit storage: g_z of the aligned 64 march positions around l, one a
    // lane, and of the next 64.  A load a plane was the sixth part of the
    // loads of steps that keep the address units busy half the time (us a
    // step: 320x288x272 FP16 41.2 -> 40.4, 512^3 200.7 -> 193.4; u and change
    // 401x397x300 BF16 111.8 -> 108.7, 256^3 FP16 33.8 -> 33.2).  FP32 steps
    // keep it: 512^3 323 -> 322, but 256^3 42.0 -> 42.2, 64^3 3.78 -> 3.84.
    const int lane = tid & 63;
    float gzw = 1.f, gzn = 1.f;
    if constexpr (SCALED) {
        gzw = gz_at(zp(lane));
        if (len > 64)
            gzn = gz_at(zp(64 + lane));
    }

    // this work-group's receivers (adjoint: receiver cells)
    int rec0 = 0, rec1 = 0;
    if (a.trace_row) {
        rec0 = a.rec_start[lid];
        rec1 = a.rec_start[lid + 1];
    }

    // sponge factors that do not change along z (masked cells' are never used)
    const __amdgpu_buffer_rsrc_t gx_r = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(a.gx), (short)0, 4 * a.nxq * (int)sizeof(float), kRsrcWord3);
    const __amdgpu_buffer_rsrc_t gy_r = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<float *>(a.gy), (short)0, a.ny * (int)sizeof(float), kRsrcWord3);
    auto gx_at = [&](int x4) {  // four factors (x4 a multiple of 4; the table is padded to whole groups)
        return decode4<WAVE_F32>(__builtin_amdgcn_raw_buffer_load_b128(gx_r, 4u * unsigned(x4), 0, 0));
    };
    auto gy_at = [&](int y) {
        return __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(gy_r, 4u * unsigned(y), 0, 0));
    };
    const f4 gxv = gx_at(x);
    float gyv[RY];
#pragma unroll
    for (int r = 0; r < RY; ++r)
        gyv[r] = gy_at(row[r]);
    // adjoint: g_x g_y of every cell this thread loads (zero outside the
    // grid, whose cells hold zeros)
    f4 gh[ADJ ? HPT : 1];
    f4 gown[ADJ ? RY : 1];
    if constexpr (ADJ) {
        f4 fx[HPT];
        float fy[HPT];
#pragma unroll
        for (int h = 0; h < HPT; ++h) {
            int hr, hc;
            halo_item(tid + h * NT, hr, hc);
            fx[h] = gx_at(4 * (xq0 + hc));
            fy[h] = gy_at(y0 + hr);
        }
#pragma unroll
        for (int h = 0; h < HPT; ++h)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                gh[h].v[e] = fx[h].v[e] * fy[h];
#pragma unroll
        for (int r = 0; r < RY; ++r)
#pragma unroll
            for (int e = 0; e < 4; ++e)
                gown[r].v[e] = gxv.v[e] * gyv[r];
#pragma unroll
        for (int i = 0; i < 8; ++i)
#pragma unroll
            for (int r = 0; r < RY; ++r)
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    q[i][r].v[e] = mul_rounded(q[i][r].v[e], gown[r].v[e] * gzi[i]);
    }

    Scales sc{1.f, 1.f, 1.f, 1.f, 0};
    Folded fd{a.c, 2.f, 1.f, 1.f};
    if constexpr (SCALED) {
        sc = step_scales<KIND>(a);
        publish_scale(a, sc, lid, tid);
        fd = fold_scales(a.c, sc, a.k_scale);
    }

    // source ownership (the value is read once, before the march)
    int src_r = -1, src_e = 0;
    if (a.src_z >= z0 && a.src_z < z1 && (a.src_x >> 2) == xq) {
#pragma unroll
        for (int r = 0; r < RY; ++r)
            if (row[r] == a.src_y)
                src_r = r;
        src_e = a.src_x & 3;
    }
    const float sval = src_r >= 0 ? src_value(a) * sc.out_inv : 0.f;

    float tmax = 0.f;  // max |stored u^{n+1}| written by this thread (16-bit storage)
    const Coefs c = fd.c;
    // A batch item's tables and source are read through generic pointers.  With
    // such a load under way, which either counter may report, the compiler
    // waits for every load there is: in the march's first plane and, the march
    // being one loop of ten planes, in every tenth, a full memory latency, 50 ns
    // a plane.  Waited for here, both counters are known (a shot of 512x256x100
    // in 256 x 8 tiles of the whole depth: 103.2 -> 95.8 us a step).  16-bit
    // items wait for them with their scales.
    if constexpr (DRAIN)
        __builtin_amdgcn_s_waitcnt(0x0070);  // vmcnt(0) lgkmcnt(0)
    for (int lb = 0; lb < len; lb += QS) {
        static_for_while<0, QS>([&](auto phase) __attribute__((always_inline)) -> bool {
            constexpr int s = decltype(phase)::value;
            const int l = lb + s;
            if (l >= len)
                return false;
            const int z = zp(l);
            constexpr int cur_set = s & 1;
            if constexpr (SCALED) {
                if (l > 0 && (l & 63) == 0) {
                    keep_branch();
                    gzw = gzn;
                    gzn = gz_at(zp(l + 64 + lane));
                }
            }
            prefetch(l + 1, (s + 9) % QS, cur_set ^ 1);
            if constexpr (ADJ) {
                // psi = G phi: the plane that just entered the queue (four positions on)
                // and this plane's halo
#pragma unroll
                for (int r = 0; r < RY; ++r)
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        q[(s + 8) % QS][r].v[e] =
                            mul_rounded(q[(s + 8) % QS][r].v[e], gown[r].v[e] * gzq[cur_set]);
            }
            const int b = l & 1;
            f4 *L = &lds[b][0][0];
#pragma unroll
            for (int r = 0; r < RY; ++r)
                L[(4 + ly * RY + r) * LW + lx + 1] = q[(s + 4) % QS][r];
#pragma unroll
            for (int h = 0; h < HPT; ++h) {
                f4 hd = decode4<KIND>(hv[cur_set][h]);
                if constexpr (ADJ) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        hd.v[e] = mul_rounded(hd.v[e], gh[h].v[e] * gzv[cur_set]);
                }
                if (h_lds[h] >= 0)
                    L[h_lds[h]] = hd;
            }
            __syncthreads();

            // y taps: LDS rows ly*RY - 4 .. ly*RY + RY + 3 of this column,
            // own rows straight from the queue; x taps: the groups left and
            // right of the own rows'.  16-bit storage reads them in the order
            // of their use.
            f4 ycol[RY + 8], xlr[RY][2];
            auto x_taps = [&](int r) {
                xlr[r][0] = L[(4 + ly * RY + r) * LW + lx];
                xlr[r][1] = L[(4 + ly * RY + r) * LW + lx + 2];
            };
#pragma unroll
            for (int r = 0; r < RY; ++r) {
                ycol[4 + r] = q[(s + 4) % QS][r];
                if constexpr (SCALED)
                    x_taps(r);
            }
#pragma unroll
            for (int m = 1; m <= 4; ++m) {
                if constexpr (SCALED)
                    reads_in_order();
                ycol[4 - m] = L[(ly * RY + 4 - m) * LW + lx + 1];
                ycol[3 + RY + m] = L[(ly * RY + 3 + RY + m) * LW + lx + 1];
            }
            const float gz = SCALED ? __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(gzw), l & 63))
                                    : gzv[cur_set];
            const __amdgpu_buffer_rsrc_t ro = INC ? rsrc_at(po, pbytes) : plane_rsrc(a.out, pbytes, z);
            const __amdgpu_buffer_rsrc_t rdl = rsrc_at(UV ? pd : po, pbytes);
            if constexpr (INC)
                po += zstep;
            if constexpr (UV)
                pd += zstep;
#pragma unroll
            for (int r = 0; r < RY; ++r) {
                if constexpr (!SCALED)
                    x_taps(r);
                const f4 xl = xlr[r][0], xr = xlr[r][1];
                const f4 ctr = q[(s + 4) % QS][r];
                float xs[12];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    xs[e] = xl.v[e];
                    xs[4 + e] = ctr.v[e];
                    xs[8 + e] = xr.v[e];
                }
                // 16-bit storage: the z sums, which need no LDS, while its
                // reads are on the way, then sums and FMAs four cells at a
                // time: an instruction that needs the one before it waits
                // 8 cycles instead of 4, and left to itself the compiler
                // finishes one cell after the other.  (us a step, before ->
                // now with the LDS rows above: 320x288x272 FP16 44.1 -> 41.3,
                // 200x190x180 FP16 21.2 -> 18.8, 512^3 205 -> 201; u and change
                // 128^3 8.82 -> 8.50, 256^3 36.0 -> 33.9, 512^3 239 -> 235.
                // FP32 steps, which wait for bandwidth, gain nothing and pay
                // 20 registers: 755x994x200 407 -> 410.)
                float lapc[4];
                if constexpr (SCALED) {
                    float zs[4][4], ts[4];
#pragma unroll
                    for (int m = 1; m <= 4; ++m)
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            zs[m - 1][e] = q[(s + 4 + m) % QS][r].v[e] + q[(s + 4 - m + QS) % QS][r].v[e];
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        lapc[e] = c.ctr * ctr.v[e];
#pragma unroll
                    for (int m = 1; m <= 4; ++m) {
                        in_order();
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            ts[e] = xs[4 + e + m] + xs[4 + e - m];
                        in_order();
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            lapc[e] = fmaf(c.cx[m - 1], ts[e], lapc[e]);
                        in_order();
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            ts[e] = ycol[4 + r + m].v[e] + ycol[4 + r - m].v[e];
                        in_order();
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            lapc[e] = fmaf(c.cy[m - 1], ts[e], lapc[e]);
                        in_order();
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            lapc[e] = fmaf(c.cz[m - 1], zs[m - 1][e], lapc[e]);
                    }
                    in_order();
                }
                const f4 pvd = decode4<KIND>(pv[cur_set][r]);
                const f4 kvd = decode4<KIND>(kv[cur_set][r]);
                f4 out, lapv;
                float img[FUS ? 2 : 1][4];  // imaging terms: of phi^m (centre) and of phi^{m+1}
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    float lap;
                    if constexpr (SCALED) {
                        lap = lapc[e];
                    } else {
                        const float u2 = 2.f * ctr.v[e];
                        lap = 0.f;
#pragma unroll
                        for (int m = 1; m <= 4; ++m) {
                            lap = fmaf(c.cx[m - 1], (xs[4 + e + m] + xs[4 + e - m]) - u2, lap);
                            lap = fmaf(c.cy[m - 1], (ycol[4 + r + m].v[e] + ycol[4 + r - m].v[e]) - u2,
                                       lap);
                            lap = fmaf(c.cz[m - 1],
                                       (q[(s + 4 + m) % QS][r].v[e] + q[(s + 4 - m + QS) % QS][r].v[e]) -
                                           u2,
                                       lap);
                        }
                    }
                    const float g = gxv.v[e] * gyv[r] * gz;
                    if constexpr (LAP)
                        lapv.v[e] = lap;
                    if constexpr (ADJ) {
                        const float t = fmaf(kvd.v[e], lap, 2.f * ctr.v[e]);
                        out.v[e] = fmaf(-g * g, pvd.v[e], t);
                        if constexpr (FUS) {
                            // (G phi / k) lap a; the centre already holds G phi
                            img[0][e] = ctr.v[e] / kvd.v[e] * __uint_as_float(lv[cur_set][0][r][e]);
                            if (two) {
                                keep_branch();
                                img[1][e] = (g * pvd.v[e]) / kvd.v[e] * __uint_as_float(lv[cur_set][1][r][e]);
                            }
                        }
                    } else {
                        float t, pe;
                        if constexpr (SCALED) {
                            t = fmaf(kvd.v[e], lap, fd.two_a * ctr.v[e]);
                            if constexpr (UV)  // u^{n-1} = u^n - d^n
                                pe = fmaf(-fd.b, pvd.v[e], fd.a * ctr.v[e]);
                            else
                                pe = fd.b * pvd.v[e];
                        } else {
                            t = fmaf(kvd.v[e], lap, 2.f * ctr.v[e]);
                            pe = pvd.v[e];
                        }
                        t = fmaf(-g, pe, t);
                        out.v[e] = g * t;
                    }
                }
                if constexpr (FUS) {
                    // the older level's term first, as one term per launch would add them
                    dv2 g0 = gacc[cur_set][r][0], g1 = gacc[cur_set][r][1];
                    if (two) {
                        keep_branch();
                        g0 += dv2{(double)img[1][0], (double)img[1][1]};
                        g1 += dv2{(double)img[1][2], (double)img[1][3]};
                    }
                    g0 += dv2{(double)img[0][0], (double)img[0][1]};
                    g1 += dv2{(double)img[0][2], (double)img[0][3]};
                    if (row_int[r]) {
                        dv2 *gp = sum_at(z, r);
                        gp[0] = g0;
                        gp[1] = g1;
                    }
                }
                if constexpr (LAP)
                    store4<WAVE_F32>(lap_rsrc(a.dlt, z, true), own_lap[r], lapv, 1.f);
                if (z == a.src_z) {
                    keep_branch();  // one plane of the grid
                    if (src_r == r) {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            if (e == src_e)
                                out.v[e] += sval;
                    }
                }
                f4 dn;  // d^{n+1} in its own units (u-and-change storage)
                if constexpr (UV) {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        dn.v[e] = 0.5f * (out.v[e] - fd.a * ctr.v[e]);
                }
                // In a ragged last group the cells past nx are right-ghost
                // cells, which hold zero: writing zero there keeps them so and
                // lets the group go out as one whole store (no partial writes).
                if (ragged) {
                    keep_branch();  // the last tile column of a grid with nx % 4 != 0
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (x + e >= a.nx) {
                            out.v[e] = 0.f;
                            if constexpr (UV)
                                dn.v[e] = 0.f;
                        }
                }
                store4<KIND>(ro, own_in[r], out, 1.f);
                if constexpr (UV)
                    store4<KIND>(rdl, own_in[r], dn, 1.f);
                if constexpr (SCALED) {
                    if (row_int[r]) {
#pragma unroll
                        for (int e = 0; e < 4; ++e)
                            tmax = fmaxf(tmax, fabsf(out.v[e]));
                    }
                }
            }
            return true;
        });
    }

    if constexpr (SCALED)
        fold_max(a, lid, tmax * sc.out);
    if constexpr (ADJ)
        inject_cells(a, rec0, rec1, tid, NT);
    else
        sample_receivers<KIND>(a, rec0, rec1, tid, NT, sc.out);
}

template <int KIND, int TXV, int TY, int RY>
__global__ __launch_bounds__(TXV *TY) void step_tiled(StepArgs a)
{
    const int lid = logical_wg(a);
    if (lid >= a.nwg)
        return;
    tile_step<KIND, TXV, TY, RY>(a, lid);
}

// The FP32 step with every field read with the default cache policy: for
// grids whose three fields fit in the GPU's memory-side cache together, so
// that u^{n-1} and k, read once per step, are still cached at the next step
// (the host picks it; same arithmetic as step_tiled).
template <int TXV, int TY, int RY>
__global__ __launch_bounds__(TXV *TY) void step_tiled_cached(StepArgs a)
{
    const int lid = logical_wg(a);
    if (lid >= a.nwg)
        return;
    tile_step<WAVE_F32, TXV, TY, RY, kFwd, false, true>(a, lid);
}

// The FP32 step that also stores the Laplacian it computes: the forward run
// of a gradient, whose imaging terms then read a value per cell instead of a
// second stencil field (written with the streaming policy: the adjoint run
// reads it once, many steps later).  Fields in or out of the memory-side
// cache as above.  With the forward levels themselves stored, the adjoint
// step carried two stencil fields in 237 registers and two LDS tiles: 105 us
// at 256^3 for one imaging term.  Now the adjoint steps are bound by
// bandwidth: 256^3 x 150 gradient 22.6 -> 18.6 ms.
template <bool CACHED, int TXV, int TY, int RY>
__global__ __launch_bounds__(TXV *TY) void step_tiled_lap(StepArgs a)
{
    const int lid = logical_wg(a);
    if (lid >= a.nwg)
        return;
    tile_step<WAVE_F32, TXV, TY, RY, kLap, false, CACHED>(a, lid);
}

template <int MODE, int TXV, int TY, int RY>
__global__ __launch_bounds__(TXV *TY) void adjoint_tiled(StepArgs a)
{
    const int lid = logical_wg(a);
    if (lid >= a.nwg)
        return;
    tile_step<WAVE_F32, TXV, TY, RY, MODE>(a, lid);
}




// ---------------------------------------------------------------------------
// many shots per launch


constexpr int kEarlyTicketPlanes = 8;

// The items of one time step j of every shot in a group: work-group b runs
// on XCD b % 8 (blocks are dealt to the XCDs round-robin) and takes items
// of that XCD's range until it is exhausted, so long and short items balance
// dynamically while neighbouring tiles still share an XCD's L2.  Its first
// item is its own number on the XCD; the next ones come by atomic ticket.
// Each XCD's counter has a cache line of its own: atomics on one line are
// served one after another, about 10 ns each, and with the eight counters on
// one line the tickets of 12 shots of 32..96 cells a side were most of a
// step (57 us, now 40).  Short items (chunks of at most kEarlyTicketPlanes
// planes) draw the next ticket while they are computed, which hides its
// latency; long ones draw it when they are done, since an item held by a
// work-group that is busy for long is an item no idle one can take
// (16 shots of 96..320 cells x 60: 29.8 ms drawn early, 28.8 late).
// Step j draws from counter set j & 1 and clears set
// (j + 1) & 1 for the next step, which starts only after this one has ended
// (a launch boundary, or a grid barrier in the single-launch run).
template <int KIND, int TXV, int TY, int RY>
__device__ __forceinline__ void batch_step_items(const ShotDesc *__restrict__ shots, const BatchItems &it, int j,
                                                 int &ticket)
{
    const int xcd = blockIdx.x & 7;
    int *cnt = it.counters + kTicketStride * (8 * (j & 1) + xcd);
    if (blockIdx.x == 0 && threadIdx.x < 8)
        it.counters[kTicketStride * (8 * ((j + 1) & 1) + threadIdx.x)] = 0;
    const int first = it.xcd_start[xcd], last = it.xcd_start[xcd + 1];
    const int groups = gridDim.x >> 3;  // work-groups per XCD
    int next = blockIdx.x >> 3;
    while (first + next < last) {
        const int item = first + next;
        const ShotDesc &d = shots[it.shot[item]];
        StepArgs a = d.a;
        if (j & 1) {
            const void *t = a.cur;
            a.cur = a.nxt;
            a.nxt = const_cast<void *>(t);
        }
        a.out = a.nxt;  // in place
        const int n = d.n0 + j;
        a.step = n & 0x3fffffff;
        a.zdown = n & 1;
        a.trace_row = d.traces ? d.traces + (size_t)n * d.nrec : nullptr;
        a.src_ptr = d.src ? d.src + j : nullptr;
        a.src_val = 0.f;
        if (!d.src)
            a.src_z = -1;  // no source values given: no injection
        const bool early = a.zc <= kEarlyTicketPlanes;
        int drawn = 0;
        if (early && threadIdx.x == 0)
            drawn = atomicAdd(cnt, 1);
        tile_step<KIND, TXV, TY, RY, kFwd, false, false, KIND == WAVE_F32>(a, it.lid[item]);
        if (!early && threadIdx.x == 0)
            drawn = atomicAdd(cnt, 1);
        if (threadIdx.x == 0)
            ticket = groups + drawn;
        __syncthreads();
        next = __builtin_amdgcn_readfirstlane(ticket);
        __syncthreads();  // all threads have read the ticket (and left the LDS of this item)
    }
}

// One time step of every shot in a group as a persistent launch: the grid
// holds as many work-groups as fit on the GPU at once.
template <int KIND, int TXV, int TY, int RY>
__global__ __launch_bounds__(TXV *TY, batch_waves(KIND, TXV, TY, RY)) void step_batch(
    const ShotDesc *__restrict__ shots, BatchItems it, int j)
{
    __shared__ int ticket;
    batch_step_items<KIND, TXV, TY, RY>(shots, it, j, ticket);
}

// Every step of a run of every shot in a group in one cooperative launch
// (all work-groups resident at once).  Each step is the work of step_batch;
// a grid-wide barrier replaces the launch boundary between steps.  Before
// a work-group arrives, its stores are made visible device-wide: every
// thread waits for its own stores to complete, then thread 0 arrives with an
// agent-scope release (which writes back its XCD's L2).  It leaves after an
// agent-scope acquire, so a step reads what the step before wrote on any
// XCD.  Every wait is bounded by a wall-clock limit and a shared abort flag:
// a wait that runs past the limit raises the flag, every work-group stops
// at its next barrier, and the host reports the run as failed.
template <int KIND, int TXV, int TY, int RY>
__global__ __launch_bounds__(TXV *TY) void step_batch_run(const ShotDesc *__restrict__ shots, BatchItems it,
                                                           RunSync rs)
{
    __shared__ int ticket;
    __shared__ int stop;
    const unsigned long long deadline = wall_clock64() + rs.timeout;
    unsigned gen = 0;  // barriers this work-group has passed
    for (int jj = 0; jj < rs.nsteps; ++jj) {
        batch_step_items<KIND, TXV, TY, RY>(shots, it, rs.j0 + jj, ticket);
        if (jj + 1 == rs.nsteps)
            break;  // the launch boundary orders the last step
        __builtin_amdgcn_s_waitcnt(0);  // this thread's stores have completed
        __syncthreads();
        if (threadIdx.x == 0) {
            stop = 0;
            const unsigned arrived =
                __hip_atomic_fetch_add(rs.count, 1u, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            if (arrived + 1 == gridDim.x) {
                // the last to arrive opens the barrier for everyone
                __hip_atomic_store(rs.count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                __hip_atomic_store(rs.gen, gen + 1, __ATOMIC_RELEASE, __HIP_MEMORY_SCOPE_AGENT);
            } else {
                while (__hip_atomic_load(rs.gen, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == gen) {
                    if (wall_clock64() > deadline ||
                        __hip_atomic_load(rs.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                        __hip_atomic_store(rs.abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                        stop = 1;
                        break;
                    }
                    __builtin_amdgcn_s_sleep(1);
                }
            }
            __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
            ++gen;
        }
        __syncthreads();
        if (stop)
            return;
    }
}

// Schedule 2 (switched off in the host code; see there): every step of
// every shot of a group in one launch (FP32).
// A work item is (step j, shot, tile, z-chunk).  The shots are pinned to
// XCDs (blocks with equal b mod 8 run on one XCD; which one depends on the
// launches before), so producers and consumers of a
// shot's fields share one L2; each XCD hands out its items by ticket in
// step order.  An item of step j starts when its own tile/chunk and the
// tiles and chunks its stencil reads from have completed step j - 1, which
// also means none of them still reads the buffer the item overwrites.  A
// work-group only waits for items with lower tickets, which running
// work-groups hold, so the waits always end; each wait is still bounded
// (FlowPlan::wait_limit polls), and a wait that gives up raises the abort
// flag, on which every work-group stops at its next check.

// Whether every item that item (j, lid) of shot fs depends on has completed
// step j - 1 (steps counted from the launch's first step).
__device__ __forceinline__ bool flow_ready(const FlowPlan &p, const FlowShot &fs, int lid, int j)
{
    if (j == 0)
        return true;
    if (p.wait_limit < 0)  // failure-path hook: every wait gives up
        return false;
    const int tiles = fs.ntx * fs.nty;
    const int tx = lid % fs.ntx, ty = (lid / fs.ntx) % fs.nty, ch = lid / tiles;
    const int *done = p.done + fs.done;
    int polls = 0;
    auto wait_for = [&](int l) -> bool {
        while (__hip_atomic_load(done + l, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < j) {
            if (polls >= p.wait_limit || __hip_atomic_load(p.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT))
                return false;
            ++polls;
            __builtin_amdgcn_s_sleep(2);
        }
        return true;
    };
    const int c0 = max(0, ch - fs.zreach), c1 = min(fs.nch - 1, ch + fs.zreach);
    for (int c = c0; c <= c1; ++c)
        if (!wait_for(c * tiles + ty * fs.ntx + tx))
            return false;
    const int base = ch * tiles;
    if (tx > 0 && !wait_for(base + ty * fs.ntx + tx - 1))
        return false;
    if (tx + 1 < fs.ntx && !wait_for(base + ty * fs.ntx + tx + 1))
        return false;
    if (ty > 0 && !wait_for(base + (ty - 1) * fs.ntx + tx))
        return false;
    if (ty + 1 < fs.nty && !wait_for(base + (ty + 1) * fs.ntx + tx))
        return false;
    return true;
}

template <int TXV, int TY, int RY>
__global__ __launch_bounds__(TXV *TY) void step_flow(const ShotDesc *__restrict__ shots, FlowPlan p)
{
    __shared__ int item[3];  // step, FlowShot index, tile/chunk; step < 0: stop
    const int xcd = blockIdx.x & 7;
    const int per = p.xcd_items[xcd];
    const int total = per * p.nsteps;
    for (;;) {
        if (threadIdx.x == 0) {
            int j = -1, k = 0, lid = 0;
            const int t = atomicAdd(&p.tickets[xcd], 1);
            if (t < total && !__hip_atomic_load(p.abort, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) {
                j = t / per;
                const int r = t - j * per;
                k = p.xcd_shot[xcd];
                while (k + 1 < p.xcd_shot[xcd + 1] && r >= p.shots[k].base + p.shots[k].items)
                    ++k;
                lid = r - p.shots[k].base;
                if (!flow_ready(p, p.shots[k], lid, j)) {
                    __hip_atomic_store(p.abort, 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    j = -1;
                }
            }
            item[0] = j;
            item[1] = k;
            item[2] = lid;
        }
        __syncthreads();
        const int j = item[0], k = item[1], lid = item[2];
        __syncthreads();  // all threads have read the item (and left the LDS of the last one)
        if (j < 0)
            break;
        const FlowShot &fs = p.shots[k];
        const ShotDesc &d = shots[fs.desc];
        const int jj = p.j0 + j;  // step within the run
        StepArgs a = d.a;
        if (jj & 1) {
            const void *t = a.cur;
            a.cur = a.nxt;
            a.nxt = const_cast<void *>(t);
        }
        a.out = a.nxt;  // in place
        const int n = d.n0 + jj;
        a.step = n & 0x3fffffff;
        a.zdown = 0;
        a.trace_row = d.traces ? d.traces + (size_t)n * d.nrec : nullptr;
        a.src_ptr = d.src ? d.src + jj : nullptr;
        a.src_val = 0.f;
        if (!d.src)
            a.src_z = -1;
        tile_step<WAVE_F32, TXV, TY, RY, kFwd, true>(a, lid);
        // completion: every thread's stores have reached the L2 (the wait
        // covers stores on this architecture) before the counter moves
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __builtin_amdgcn_s_waitcnt(0);
        __atomic_signal_fence(__ATOMIC_SEQ_CST);
        __syncthreads();
        if (threadIdx.x == 0)
            __hip_atomic_store(p.done + fs.done + lid, j + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
}

// One thread per interior cell, every tap read from global memory: a
// deliberately plain kernel used to cross-check the tiled one.  Same FP32
// operations in the same order, so the two agree bit for bit.
template <int KIND>
__global__ __launch_bounds__(256) void step_naive(StepArgs a)
{
    constexpr bool SCALED = Store<KIND>::scaled;
    Scales sc{1.f, 1.f, 1.f, 1.f, 0};
    Folded fd{a.c, 2.f, 1.f, 1.f};
    if constexpr (SCALED) {
        sc = step_scales<KIND>(a);
        publish_scale(a, sc, blockIdx.x, threadIdx.x);
        fd = fold_scales(a.c, sc, a.k_scale);
    }
    const Coefs &c = fd.c;
    const long long n = (long long)a.nx * a.ny * a.nz;
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    float amax = 0.f;
    if (i < n) {
        const int x = (int)(i % a.nx);
        const int y = (int)((i / a.nx) % a.ny);
        const int z = (int)(i / ((long long)a.nx * a.ny));
        const long long p =
            (long long)(z + kGhost) * a.plane + (long long)(y + kGhost) * a.px + a.x0 + x;
        auto U = [&](long long q) { return read_elem<KIND>(a.cur, q, 1.f); };
        const float u = U(p);
        // same form and order as the tiled kernel (difference form for FP32)
        const float u2 = SCALED ? 0.f : 2.f * u;
        float lap = SCALED ? c.ctr * u : 0.f;
        for (int m = 1; m <= 4; ++m) {
            lap = fmaf(c.cx[m - 1], (U(p + m) + U(p - m)) - u2, lap);
            lap = fmaf(c.cy[m - 1], (U(p + (long long)m * a.px) + U(p - (long long)m * a.px)) - u2, lap);
            lap = fmaf(c.cz[m - 1], (U(p + m * a.plane) + U(p - m * a.plane)) - u2, lap);
        }
        const float g = a.gx[x] * a.gy[y] * a.gz[z];
        const float kk = read_elem<KIND>(a.k, p, 1.f);
        const float pp = read_elem<KIND>(Store<KIND>::uv ? a.dlt : a.nxt, p, 1.f);
        float t, pe;
        if constexpr (SCALED) {
            t = fmaf(kk, lap, fd.two_a * u);
            if constexpr (Store<KIND>::uv)
                pe = fmaf(-fd.b, pp, fd.a * u);
            else
                pe = fd.b * pp;
        } else {
            t = fmaf(kk, lap, 2.f * u);
            pe = pp;
        }
        t = fmaf(-g, pe, t);
        float v = g * t;
        if (z == a.src_z && y == a.src_y && x == a.src_x)
            v += src_value(a) * sc.out_inv;
        if constexpr (KIND == WAVE_F32) {
            static_cast<float *>(a.out)[p] = v;
            if (a.dlt)  // gradient runs: the Laplacian's own layout
                static_cast<float *>(a.dlt)[z * a.lplane + (long long)y * a.lpx + x] = lap;
        } else {
            static_cast<unsigned short *>(a.out)[p] = (unsigned short)Store<KIND>::enc(v);
            if constexpr (Store<KIND>::uv)
                static_cast<unsigned short *>(a.dlt)[p] =
                    (unsigned short)Store<KIND>::enc(0.5f * (v - fd.a * u));
            amax = fabsf(v);
        }
    }
    if constexpr (SCALED)
        fold_max(a, blockIdx.x, amax * sc.out);
}

// Receivers for the naive kernel (separate launch: it has no tile
// epilogue).  With 16-bit storage the scale of u^{n+1} is the one the step
// just published.
template <int KIND>
__global__ void sample_naive(const void *__restrict__ f, const long long *__restrict__ off, int nrec,
                             float *row, const int *exps, int slot)
{
    const int r = blockIdx.x * blockDim.x + threadIdx.x;
    if (r < nrec) {
        const float scale = Store<KIND>::scaled ? ldexpf(1.f, exps[slot]) : 1.f;
        row[r] = read_elem<KIND>(f, off[r], scale);
    }
}


// Interior copy between two layouts with an exact power-of-two rescale:
// FP32 k into 16-bit storage (init), or a field of any storage into FP32
// (export).  `exps`/`slot` select a device exponent for the source scale.
template <int SRC, int DST>
__global__ __launch_bounds__(256) void convert_interior(const void *__restrict__ src, void *dst, int nx,
                                                        int ny, int nz, int spx, int sx0,
                                                        long long splane, int dpx, int dx0,
                                                        long long dplane, float scale,
                                                        const int *exps, int slot)
{
    const float sc = exps ? ldexpf(1.f, exps[slot]) : scale;
    for_interior_groups(nx, ny, nz, [&](int z, int y, int x, int n) {
        const long long si = (long long)(z + kGhost) * splane + (long long)(y + kGhost) * spx + sx0 + x;
        const long long di = (long long)(z + kGhost) * dplane + (long long)(y + kGhost) * dpx + dx0 + x;
        // the whole group is read (right-ghost cells past nx are allocated)
        // and, unless it is a ragged one, written whole
        Raw4<SRC> in;
        if constexpr (SRC == WAVE_F32)
            in = *reinterpret_cast<const u4raw *>(static_cast<const float *>(src) + si);
        else
            in = *reinterpret_cast<const u2raw *>(static_cast<const unsigned short *>(src) + si);
        f4 v = decode4<SRC>(in);
        for (int e = 0; e < 4; ++e)
            v.v[e] *= sc;
        if constexpr (DST == WAVE_F32) {
            float *d = static_cast<float *>(dst) + di;
            if (n == 4)
                *reinterpret_cast<f4 *>(d) = v;
            if (n & 2)
                *reinterpret_cast<float2 *>(d) = float2{v.v[0], v.v[1]};
            if (n & 1)
                d[n & 2] = (n & 2) ? v.v[2] : v.v[0];
        } else {
            unsigned short *d = static_cast<unsigned short *>(dst) + di;
            if (n == 4)
                *reinterpret_cast<ushort4 *>(d) =
                    ushort4{(unsigned short)Store<DST>::enc(v.v[0]), (unsigned short)Store<DST>::enc(v.v[1]),
                            (unsigned short)Store<DST>::enc(v.v[2]), (unsigned short)Store<DST>::enc(v.v[3])};
            else
#pragma unroll
                for (int e = 0; e < 3; ++e)
                    if (e < n)
                        d[e] = (unsigned short)Store<DST>::enc(v.v[e]);
        }
    });
}

}  // namespace wavek
