// sne_kernels.hip - fused three-filters-to-normal stencil for gfx950.
//
// Compiled once per raw input kind (-DSNE_KIND=0..3) so the template
// instantiations build in parallel.
//
// Work decomposition.  A tile is `64 * PX` columns by `rows` rows of one
// frame and belongs to one 64-lane wavefront (or, in half-wave mode, two
// tiles of `32 * PX` columns, one above the other, belong to the two halves of
// a wavefront); lane l owns columns c0 + l*PX .. c0 + l*PX + PX-1 and walks
// down the rows of its tile keeping a three-row window in registers.
// Horizontal neighbours that live in the adjacent lane arrive by DPP wave
// shifts; the two columns just outside a tile are loaded by its first and
// last lanes and enter through the DPP "old" operand.
// No barriers are involved (and LDS only to turn packed output rows around
// within a wavefront), so a tile's arithmetic is the same instruction sequence
// whatever the launch shape: results are bitwise identical alone, in a uniform
// batch and in an uneven persistent batch.
//
// Arithmetic (FP32), per pixel p with raw value z (depth) or d (disparity):
//   s = 1/z (depth) or d (disparity): the image the gradient filters see
//   (Sec. III and eq. nx2_ny2_nz3).  A difference s_a - s_b of inverse depths
//   is formed as (z_b - z_a) * (s_a * s_b): the raw difference is exact for
//   nearby samples (Sterbenz) and the product is symmetric, so mirrored
//   windows cancel exactly and near-equal depths keep full relative accuracy.
//   G_u, G_v: the filter as weighted central differences of s.
//   Candidates.  With (u, v) the pixel, B = (u - u0) G_u + (v - v0) G_v and
//   rho_j = 1 / (raw_j - raw) the candidate of eq. nx2_ny2_nz2 equals
//       c_j = B + t_j,  t_j = N_j w_j,  N_j = du_j G_u + dv_j G_v,
//   with w_j = z_j / (z_j - z) = 1 + z rho_j for depth and
//   w_j = d / (d - d_j) = -d rho_j for disparity (substitute the
//   back-projection of eq. intrinisc_matrix into dX, dY, dZ; f_x, f_y and the
//   stereo baseline cancel).  Each pair reciprocal rho is computed once per
//   pixel pair and used by both pixels of the pair.
//   Filter 3 runs on t_j (mean or median commute with adding B).  Neighbours
//   with raw_j == raw are left out.  Median: a branch-free network over the
//   8 slots; left-out slots are padded alternately +inf / -inf in slot order,
//   which puts the middle of the kept values at sorted positions 3 and 4
//   whatever their number m; odd m takes position 3.
//   Output: (-f_x G_u, -f_y G_v, B + Phi) / norm, the camera-facing unit
//   normal; m = 0 or a zero vector gives (0, 0, -1); masked pixels +0.
//
// Lenient rule (LEN): a wavefront holding a valid pixel whose window is not
// fully valid (a hole nearby, or the frame border, which loads as 0) forms
// each gradient line from its two outer samples, else from its middle and one
// outer sample at twice the one-sided difference, rescales the available
// lines to the filter's full weight, and leaves invalid neighbours out of
// filter 3.  The mask is then: valid centre and a line for each gradient.  On
// a full window every step is the strict one, bit for bit.
#include "sne_internal.h"

#ifndef SNE_KIND
#error "compile with -DSNE_KIND=<0..3>"
#endif

// Minimum wavefronts per SIMD the register allocator has to leave room for
// (0: the compiler's choice).
#ifndef SNE_WAVES_PER_EU
#define SNE_WAVES_PER_EU 0
#endif
#if SNE_WAVES_PER_EU > 0
#define SNE_OCCUPANCY __attribute__((amdgpu_waves_per_eu(SNE_WAVES_PER_EU)))
#else
#define SNE_OCCUPANCY
#endif

// The persistent kernel keeps the tile loop's state live across tiles and
// would otherwise exceed 128 registers at 4 columns per lane (3 wavefronts
// per SIMD); holding it to 4 costs a few spilled dwords and is faster.
#ifndef SNE_BATCH_WAVES_PER_EU
#define SNE_BATCH_WAVES_PER_EU 4
#endif
// The lenient rule's extra line arithmetic does not fit that budget without
// spilling: its instantiations get the compiler's choice.
#if SNE_BATCH_WAVES_PER_EU > 0
#define SNE_BATCH_OCCUPANCY \
    __attribute__((amdgpu_waves_per_eu(LEN ? 1 : SNE_BATCH_WAVES_PER_EU)))
#else
#define SNE_BATCH_OCCUPANCY
#endif

// Rows whose loads are in flight while a row is computed (1 or 2).
#ifndef SNE_PREFETCH_ROWS
#define SNE_PREFETCH_ROWS 1
#endif

namespace sne {
namespace {

constexpr float kInf = __builtin_huge_valf();
// class-test mask (v_cmp_class) of the positive finite non-zero values:
// +denormal | +normal, i.e. 0 < x <= FLT_MAX
constexpr int kPosFinite = (1 << 7) | (1 << 8);

// lane l receives lane l-1's `src`; lane 0 (no source) keeps `old`.
__device__ __forceinline__ float from_left(float old, float src) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        __builtin_bit_cast(int, old), __builtin_bit_cast(int, src), 0x138 /*wave_shr:1*/, 0xf,
        0xf, false));
}
// lane l receives lane l+1's `src`; lane 63 (no source) keeps `old`.
__device__ __forceinline__ float from_right(float old, float src) {
    return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(
        __builtin_bit_cast(int, old), __builtin_bit_cast(int, src), 0x130 /*wave_shl:1*/, 0xf,
        0xf, false));
}

__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }

// Min/max of values the compiler cannot prove canonical (they come from
// other basic blocks or earlier loop iterations) would each be preceded by a
// quieting v_max x, x, x in IEEE mode.  For every pixel whose result is kept
// the operands are finite or infinite, never NaN (a NaN can only arise in a
// window with an invalid sample, whose output is replaced by zeros), so the
// instructions are issued directly.
__device__ __forceinline__ float vmin(float a, float b) {
    float r;
    asm("v_min_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float vmax(float a, float b) {
    float r;
    asm("v_max_f32 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}
__device__ __forceinline__ float vmin3(float a, float b, float c) {
    float r;
    asm("v_min3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
// max over |r_0| .. |r_7|.  The operands are reciprocals straight from
// v_rcp: a transcendental result needs one wait state before a VALU reads it,
// which the compiler inserts for its own instructions but not for inline asm,
// hence the leading s_nop.
__device__ __forceinline__ float vmax8abs(float r0, float r1, float r2, float r3, float r4,
                                          float r5, float r6, float r7) {
    float out, m1, m2, m3;
    asm("s_nop 0\n\t"
        "v_max3_f32 %[m1], |%[r0]|, |%[r1]|, |%[r2]|\n\t"
        "v_max3_f32 %[m2], |%[r3]|, |%[r4]|, |%[r5]|\n\t"
        "v_max3_f32 %[m3], |%[r6]|, |%[r7]|, %[m1]\n\t"
        "v_max_f32 %[out], %[m2], %[m3]"
        : [out] "=&v"(out), [m1] "=&v"(m1), [m2] "=&v"(m2), [m3] "=&v"(m3)
        : [r0] "v"(r0), [r1] "v"(r1), [r2] "v"(r2), [r3] "v"(r3), [r4] "v"(r4), [r5] "v"(r5),
          [r6] "v"(r6), [r7] "v"(r7));
    return out;
}
__device__ __forceinline__ float vmax3(float a, float b, float c) {
    float r;
    asm("v_max3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}
// x * y, and +0 if y is 0 whatever x is (infinities and NaN included): one
// select of the factor y then blanks all products it enters.  Full rate.
__device__ __forceinline__ float mul_or_zero(float x, float y) {
    float r;
    asm("v_mul_legacy_f32 %0, %1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}
// The same as the compiler's own instruction, which may read a transcendental
// result (inline asm gets no wait state after one).
extern "C" __device__ float mul_legacy(float, float) __asm("llvm.amdgcn.fmul.legacy");
__device__ __forceinline__ float neg_mul_or_zero(float x, float y) {  // -x * y
    float r;
    asm("v_mul_legacy_f32 %0, -%1, %2" : "=v"(r) : "v"(x), "v"(y));
    return r;
}
__device__ __forceinline__ float vmed3(float a, float b, float c) {
    float r;
    asm("v_med3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}


// ---------------------------------------------------------------- raw input
template <int KIND> struct Raw;
template <> struct Raw<KIND_F32> {
    using T = float;
    __device__ static bool ok(T x) { return __builtin_amdgcn_classf(x, kPosFinite); }
    __device__ static float value(T x) { return ok(x) ? x : 0.f; }
    // in the register window samples stay as they are, valid or not: masks
    // say which are (see Mask)
    __device__ static float window(T x) { return x; }
};
template <> struct Raw<KIND_DISP> : Raw<KIND_F32> {};
template <> struct Raw<KIND_U16> {
    using T = uint16_t;
    __device__ static bool ok(T x) { return x != 0; }
    __device__ static float value(T x) { return (float)x; }  // 0 = invalid
    __device__ static float window(T x) { return (float)x; }
};
template <> struct Raw<KIND_F16> {
    using T = uint16_t;  // binary16 bits
    __device__ static float window(T x) { return (float)__builtin_bit_cast(_Float16, x); }
    __device__ static bool ok(T x) { return __builtin_amdgcn_classf(window(x), kPosFinite); }
    __device__ static float value(T x) { return ok(x) ? window(x) : 0.f; }
};

// One bit per lane.  (The predicate `lane` makes of a mask is used from a
// variable: inside a conditional operator it would become a branch.)
// Validity is kept as such masks in scalar registers: a
// window's validity is a few scalar ands, which issue beside the vector
// instructions of other wavefronts, instead of minima over the nine samples
// and a compare per pixel, and holds no vector registers.  Together with one
// select per pixel for the three channels (mul_or_zero) and the middle row's
// pairs formed last, this took the 4-column FP32 Sobel-median kernel from
// 127 to 114 registers and 48 to 40 half-rate instructions per pixel:
// 64 x 480x640 in 57.6 instead of 60.4 us with the input in the last-level
// cache (5.8 TB/s of algorithmic bytes, 0.94 of the rate of a kernel of the same
// streams without arithmetic; 68 us, 0.79 of it, where the input comes from HBM),
// 1024 uneven u16 frames FD-mean in 1.91 instead of 2.0 ms.
using Mask = uint64_t;
__device__ __forceinline__ Mask mask_of(bool b) { return __builtin_amdgcn_ballot_w64(b); }
__device__ __forceinline__ bool lane(Mask m) { return __builtin_amdgcn_inverse_ballot_w64(m); }

template <typename T, int N> struct alignas(sizeof(T) * N) Vec { T v[N]; };

template <int KIND, int PX> struct RawRow {
    Vec<typename Raw<KIND>::T, PX> x;
    typename Raw<KIND>::T h;  // halo: a tile's first lane loads the column left
                              // of it, its last lane the column right of it
};

// A frame's input as a buffer resource: loads outside [0, bytes) return 0
// without touching memory, which covers the rows above and below the frame,
// the columns past its width and the halo of lanes that load none.
struct InBuf {
    __amdgpu_buffer_rsrc_t rsrc;
    int pitch_bytes;
};

__device__ __forceinline__ InBuf make_inbuf(const void *base, int64_t pitch, int H, int elem) {
    InBuf b;
    b.rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(base), (short)0,
                                               (int)((int64_t)H * pitch * elem), 0x00020000);
    b.pitch_bytes = (int)(pitch * elem);
    return b;
}

// Column offset of a lane that loads nothing.  With the frame's input below
// 2^31 - 2 pitches (checked by the host), kOOB + r * pitch for the rows
// -1 <= r <= H + 1 lands at or past the end of the buffer, as does any
// in-frame column at row -1 (the offset wraps past 2^31); further rows never
// feed a stored output.
constexpr int kOOB = 0x7fffffff;

template <typename T, int N> __device__ __forceinline__ Vec<T, N> buf_load(const InBuf &b, int off);
template <> __device__ __forceinline__ Vec<float, 1> buf_load<float, 1>(const InBuf &b, int off) {
    return __builtin_bit_cast(Vec<float, 1>, __builtin_amdgcn_raw_buffer_load_b32(b.rsrc, off, 0, 0));
}
template <> __device__ __forceinline__ Vec<float, 2> buf_load<float, 2>(const InBuf &b, int off) {
    return __builtin_bit_cast(Vec<float, 2>, __builtin_amdgcn_raw_buffer_load_b64(b.rsrc, off, 0, 0));
}
template <> __device__ __forceinline__ Vec<float, 4> buf_load<float, 4>(const InBuf &b, int off) {
    return __builtin_bit_cast(Vec<float, 4>, __builtin_amdgcn_raw_buffer_load_b128(b.rsrc, off, 0, 0));
}
template <> __device__ __forceinline__ Vec<uint16_t, 1> buf_load<uint16_t, 1>(const InBuf &b, int off) {
    return __builtin_bit_cast(Vec<uint16_t, 1>, __builtin_amdgcn_raw_buffer_load_b16(b.rsrc, off, 0, 0));
}
template <> __device__ __forceinline__ Vec<uint16_t, 2> buf_load<uint16_t, 2>(const InBuf &b, int off) {
    return __builtin_bit_cast(Vec<uint16_t, 2>, __builtin_amdgcn_raw_buffer_load_b32(b.rsrc, off, 0, 0));
}
template <> __device__ __forceinline__ Vec<uint16_t, 4> buf_load<uint16_t, 4>(const InBuf &b, int off) {
    return __builtin_bit_cast(Vec<uint16_t, 4>, __builtin_amdgcn_raw_buffer_load_b64(b.rsrc, off, 0, 0));
}

// The lane that holds a row's last columns when the width is not a multiple
// of PX.  It loads the row's last PX samples (all inside the frame) and moves
// the ones it owns to the front; the columns past the width become 0, which
// is invalid.  `any` is wave-uniform: tiles without such a lane pass by.
struct Tail {
    bool any;  // a lane of this tile is cut
    int skip;  // samples this lane drops from the front (0 for whole lanes)
};
template <int PX>
__device__ __forceinline__ void shift_down(Vec<float, PX> &x, int skip) {
    if constexpr (PX == 4) {
        const bool two = (skip & 2) != 0;
        x.v[0] = two ? x.v[2] : x.v[0];
        x.v[1] = two ? x.v[3] : x.v[1];
        x.v[2] = two ? 0.f : x.v[2];
        x.v[3] = two ? 0.f : x.v[3];
    }
    if constexpr (PX >= 2) {
        const bool one = (skip & 1) != 0;
#pragma unroll
        for (int k = 0; k < PX; ++k) x.v[k] = one ? (k + 1 < PX ? x.v[k + 1] : 0.f) : x.v[k];
    }
}
template <int PX>
__device__ __forceinline__ void shift_down(Vec<uint16_t, PX> &x, int skip) {
    if constexpr (PX == 4)
        x = __builtin_bit_cast(Vec<uint16_t, PX>,
                               __builtin_bit_cast(uint64_t, x) >> (16 * skip));
    if constexpr (PX == 2)
        x = __builtin_bit_cast(Vec<uint16_t, PX>,
                               __builtin_bit_cast(uint32_t, x) >> (16 * skip));
}

// Issue the loads of row r; everything outside the frame reads as 0.
// col_off / halo_off: this lane's byte offsets within a row, kOOB-based when
// the lane loads nothing.
template <int KIND, int PX>
__device__ __forceinline__ void load_raw(const InBuf &b, int r, int col_off, int halo_off,
                                         RawRow<KIND, PX> &o) {
    using T = typename Raw<KIND>::T;
    const unsigned row = (unsigned)r * (unsigned)b.pitch_bytes;  // wraps for r = -1
    o.x = buf_load<T, PX>(b, (int)(row + (unsigned)col_off));
    o.h = buf_load<T, 1>(b, (int)(row + (unsigned)halo_off)).v[0];
}

// Per-row state.  Index i of z/s is column (lane base + i - 1): 0 and PX+1
// are the neighbours from the adjacent lanes.
template <int PX> struct Row {
    float z[PX + 2];   // raw value (Raw::window)
    float s[PX + 2];   // filtered image
    float D[PX];       // s[k+1] - s[k-1] (horizontal central difference)
    float rE[PX + 1];  // rE[i] = 1 / (z[i+1] - z[i])
    Mask ok[PX + 2];   // sample valid
    Mask hok[PX];      // columns k-1..k+1 valid
    Mask kE[PX + 1];   // kPairMean: pair rE[i] gives its two pixels a candidate
    float mid[PX];     // kPairCount: how many of a pixel's two do
    // lenient rule with a 3-row filter only: the row's horizontal gradient
    // line at columns 1..PX and whether it has one (computed once, used by
    // the three output rows whose window holds this row)
    float Lh[PX];
    Mask hh[PX];
};

// Lanes at the inner edges of two half-wave tiles (31 and 32) take their
// halo sample instead of the neighbour across the boundary.
struct Edges {
    bool left;   // lane 32 in half-wave mode
    bool right;  // lane 31 in half-wave mode
};

template <bool HALF>
__device__ __forceinline__ float left_of(float old, float src, const Edges &e) {
    const float v = from_left(old, src);
    if constexpr (HALF) return e.left ? old : v;
    return v;
}
template <bool HALF>
__device__ __forceinline__ float right_of(float old, float src, const Edges &e) {
    const float v = from_right(old, src);
    if constexpr (HALF) return e.right ? old : v;
    return v;
}

// Quantised raw values (uint16, binary16) repeat along iso-depth lines so
// often that nearly every wavefront holds a pixel with a left-out neighbour:
// those kinds take the general aggregation everywhere, without the per-pixel
// test and wavefront vote that let the FP32 kinds skip it.  With no branch the compiler also shares
// a pair's equality test between the two pixels of the pair.
template <int KIND> constexpr bool kTieHeavy = KIND == KIND_U16 || KIND == KIND_F16;

// s[k+1] - s[k-1] at the lane's columns.
template <int KIND, int PX> __device__ __forceinline__ void make_hdiff(Row<PX> &o) {
#pragma unroll
    for (int k = 0; k < PX; ++k) {
        if constexpr (KIND == KIND_DISP)
            o.D[k] = o.z[k + 2] - o.z[k];
        else
            o.D[k] = (o.z[k] - o.z[k + 2]) * (o.s[k] * o.s[k + 2]);
    }
}

// A sample as the window holds it.  Strict rule: as it is (the masks say
// whether it counts).  Lenient rule: an invalid one is 0 for the mean, which
// multiplies it by the pair's reciprocal 0, and NaN for the median, so that
// one ordered compare with the centre leaves it out.
template <int KIND, int AGG, bool LEN>
__device__ __forceinline__ float sample(typename Raw<KIND>::T x) {
    if constexpr (!LEN) return Raw<KIND>::window(x);
    if constexpr (AGG == AGG_MEAN) return Raw<KIND>::value(x);
    return Raw<KIND>::ok(x) ? Raw<KIND>::window(x) : __builtin_nanf("");
}

// A row's values and validity, and for the 3-row filters its horizontal
// differences (FD needs only those of the middle row: make_middle).
template <int KIND, int AGG, int PX, bool HALF, bool FD, bool LEN>
__device__ __forceinline__ void finish_row(RawRow<KIND, PX> &raw, Row<PX> &o,
                                           const Edges &e, const Tail &tail) {
    if constexpr (PX > 1)
        if (tail.any) shift_down<PX>(raw.x, tail.skip);
    // lanes that take their outer neighbour from the halo sample
    constexpr Mask kLeft = HALF ? 0x100000001ull : 1ull, kRight = kLeft << (HALF ? 31 : 63);
    const float h = sample<KIND, AGG, LEN>(raw.h);
    const Mask okh = mask_of(Raw<KIND>::ok(raw.h));
#pragma unroll
    for (int k = 0; k < PX; ++k) {
        o.z[k + 1] = sample<KIND, AGG, LEN>(raw.x.v[k]);
        o.ok[k + 1] = mask_of(Raw<KIND>::ok(raw.x.v[k]));
    }
    o.z[0] = left_of<HALF>(h, o.z[PX], e);
    o.z[PX + 1] = right_of<HALF>(h, o.z[1], e);
    o.ok[0] = ((o.ok[PX] << 1) & ~kLeft) | (okh & kLeft);
    o.ok[PX + 1] = ((o.ok[1] >> 1) & ~kRight) | (okh & kRight);
#pragma unroll
    for (int k = 0; k < PX; ++k) o.hok[k] = o.ok[k] & o.ok[k + 1] & o.ok[k + 2];
    // the outer columns' reciprocals are formed again: one v_rcp each costs
    // less than the lane shift and the half-wave select
#pragma unroll
    for (int i = 0; i < PX + 2; ++i) o.s[i] = KIND == KIND_DISP ? o.z[i] : rcp(o.z[i]);
    if constexpr (!FD) make_hdiff<KIND, PX>(o);
}

// Means over pairs that count their candidates where they are formed: a pair
// that gives its pixels no candidate (equal values, or under the lenient rule
// an invalid one) gets the reciprocal 0, once for both pixels, and a mask
// from which its pixels count what they keep.  For data where such pairs are
// in nearly every wavefront; the other kinds blank slots in a rare branch.
// 1024 uneven u16 frames, FD-mean: 1.84 ms (4.05 TB/s of algorithmic bytes),
// against 1.91 ms with a test, a select and a count in every slot; with the
// batch kernel's scalar table loads, global stores (store_stream) and the
// scaled normal (normal_z) 1.75 ms, 4.27 TB/s.
template <int KIND, int AGG, bool LEN>
constexpr bool kPairMean = AGG == AGG_MEAN && (kTieHeavy<KIND> || LEN);

// 1 / (b - a), or 0 with the bit of `keep` clear if the pair is left out.
template <bool LEN>
__device__ __forceinline__ float pair_or_zero(float a, float b, Mask oka, Mask okb, Mask &keep) {
    keep = mask_of(a != b);
    if constexpr (LEN) keep &= oka & okb;
    const float r = rcp(b - a);
    const bool k = lane(keep);
    return k ? r : 0.f;
}

// Of these, strict means of quantised raw values count in vector registers:
// two distinct values differ by at least a known step (1 for uint16, 2^-24 for
// binary16), so the difference over that step, clamped to [0, 1], is 1 for a
// pair that counts and 0 for equal values.  The product with it, and the sums
// of it, are adds and multiplies at twice the rate of the compare, the select
// and the adds with carry that masks take: 64 x 480x640 FD-mean FP16, u16 49.0
// -> 46.8 us, binary16 50.5 -> 47.6 us; 1024 uneven u16 frames 1.78 -> 1.74 ms.
template <int KIND, int AGG, bool LEN>
constexpr bool kPairCount = kPairMean<KIND, AGG, LEN> && kTieHeavy<KIND> && !LEN;

template <int KIND>
__device__ __forceinline__ float pair_counted(float a, float b, float &count) {
    const float d = b - a;
    if constexpr (KIND == KIND_U16)
        asm("v_mul_f32_e64 %0, %1, %1 clamp" : "=v"(count) : "v"(d));
    else
        asm("v_mul_f32_e64 %0, |%1|, %2 clamp" : "=v"(count) : "v"(d), "v"(0x1p24f));
    return mul_legacy(rcp(d), count);  // inf * 0 = 0
}

// What only the middle row of the window needs, formed when a row becomes
// that (earlier it would hold registers): the horizontal pairs.
template <int KIND, int AGG, int PX, bool FD, bool LEN>
__device__ __forceinline__ void make_middle(Row<PX> &o) {
    float count[PX + 1];
#pragma unroll
    for (int i = 0; i <= PX; ++i) {
        if constexpr (kPairCount<KIND, AGG, LEN>)
            o.rE[i] = pair_counted<KIND>(o.z[i], o.z[i + 1], count[i]);
        else if constexpr (kPairMean<KIND, AGG, LEN>)
            o.rE[i] = pair_or_zero<LEN>(o.z[i], o.z[i + 1], o.ok[i], o.ok[i + 1], o.kE[i]);
        else
            o.rE[i] = rcp(o.z[i + 1] - o.z[i]);
    }
    if constexpr (kPairCount<KIND, AGG, LEN>) {
#pragma unroll
        for (int k = 0; k < PX; ++k) o.mid[k] = count[k] + count[k + 1];
    }
    if constexpr (FD) make_hdiff<KIND, PX>(o);
}

// Reciprocals of the vertical and diagonal pairs between an upper row and the
// row below it (lower minus upper).
template <int PX> struct Pairs {
    float rS[PX];       // (up k)   - (low k)
    float rSE[PX + 1];  // rSE[i]: (up col i-1) - (low col i)
    float rSW[PX + 1];  // rSW[i]: (up col i)   - (low col i-1)
    // kPairMean: which of them give candidates, and how many of the three
    // above a pixel of the lower row do
    Mask kS[PX], kSE[PX + 1], kSW[PX + 1];
    int top[PX];
    // kPairCount: how many candidates a pixel of the lower row gets from the
    // three above it, and one of the upper row from the three below
    float above[PX], under[PX];
};

template <int KIND, int AGG, bool LEN, int PX>
__device__ __forceinline__ void make_pairs(const Row<PX> &up, const Row<PX> &lo, Pairs<PX> &o) {
    if constexpr (kPairCount<KIND, AGG, LEN>) {
        float cS[PX], cSE[PX + 1], cSW[PX + 1];
#pragma unroll
        for (int k = 0; k < PX; ++k)
            o.rS[k] = pair_counted<KIND>(up.z[k + 1], lo.z[k + 1], cS[k]);
#pragma unroll
        for (int i = 0; i <= PX; ++i) {
            o.rSE[i] = pair_counted<KIND>(up.z[i], lo.z[i + 1], cSE[i]);
            o.rSW[i] = pair_counted<KIND>(up.z[i + 1], lo.z[i], cSW[i]);
        }
#pragma unroll
        for (int k = 0; k < PX; ++k) {
            o.above[k] = cS[k] + (cSE[k] + cSW[k + 1]);
            o.under[k] = cS[k] + (cSE[k + 1] + cSW[k]);
        }
    } else if constexpr (kPairMean<KIND, AGG, LEN>) {
#pragma unroll
        for (int k = 0; k < PX; ++k)
            o.rS[k] = pair_or_zero<LEN>(up.z[k + 1], lo.z[k + 1], up.ok[k + 1], lo.ok[k + 1],
                                        o.kS[k]);
#pragma unroll
        for (int i = 0; i <= PX; ++i) {
            o.rSE[i] = pair_or_zero<LEN>(up.z[i], lo.z[i + 1], up.ok[i], lo.ok[i + 1], o.kSE[i]);
            o.rSW[i] = pair_or_zero<LEN>(up.z[i + 1], lo.z[i], up.ok[i + 1], lo.ok[i], o.kSW[i]);
        }
#pragma unroll
        for (int k = 0; k < PX; ++k)
            o.top[k] = (lane(o.kS[k]) ? 1 : 0) + (lane(o.kSE[k]) ? 1 : 0) +
                       (lane(o.kSW[k + 1]) ? 1 : 0);
    } else {
#pragma unroll
        for (int k = 0; k < PX; ++k) o.rS[k] = rcp(lo.z[k + 1] - up.z[k + 1]);
#pragma unroll
        for (int i = 0; i <= PX; ++i) {
            o.rSE[i] = rcp(lo.z[i + 1] - up.z[i]);
            o.rSW[i] = rcp(lo.z[i] - up.z[i + 1]);
        }
    }
}

// Order statistics 3 and 4 (0-based) of 8 values in 16 instructions.  The
// median of 9 values in three sorted columns (l_i, m_i, h_i) is
// med3(max of the l_i, med3 of the m_i, min of the h_i); with the ninth value
// +inf it is x4 of the other eight, with -inf it is x3.  The two medians share
// the sorted columns (t0, t1, t2) and (t3, t4, t5), 3 instructions each, and
// the sorted pair (p, q) of t6, t7, whose column is (p, q, +inf) or
// (-inf, p, q).  Every output is one of the inputs, so ties and infinities
// come out exactly.  min, max and med3 issue at half the rate of adds and
// multiplies (4.3 against 2.4 cycles per wavefront and SIMD), and the median
// kernels are bound by issue: against the 24 of two merged sorted quads,
// 64 x 480x640 FP32 Sobel-median went from 63.8 to 60.4 us, the lenient rule
// from 102.3 to 98.6 us, one 2160x3840 u16 FD-median frame from 29.6 to
// 27.9 us.
__device__ __forceinline__ void middle_pair(const float (&t)[8], float &x3, float &x4) {
    const float p = vmin(t[6], t[7]), q = vmax(t[6], t[7]);
    const float l = vmax(vmin3(t[0], t[1], t[2]), vmin3(t[3], t[4], t[5]));  // largest low
    const float h = vmin(vmax3(t[0], t[1], t[2]), vmax3(t[3], t[4], t[5]));  // smallest high
    const float m1 = vmed3(t[0], t[1], t[2]), m2 = vmed3(t[3], t[4], t[5]);
    x3 = vmed3(l, vmed3(m1, m2, p), vmin(h, q));  // columns with (-inf, p, q)
    x4 = vmed3(vmax(l, p), vmed3(m1, m2, q), h);  // columns with (p, q, +inf)
}

// Output element stores.
template <int OUT> struct Out;
template <> struct Out<OUT_F32> {
    using T = float;
    __device__ static T cvt(float x) { return x; }
};
template <> struct Out<OUT_RGBN>;  // FP16 channels, stored by tile_row's packed branch
template <> struct Out<OUT_F16> {
    using T = _Float16;
    // Round the FP32 value to nearest even.  The value is pinned first so
    // that the compiler cannot fold the product that feeds it into a mixed-
    // precision multiply rounded once to FP16: whether it did would depend
    // on the kernel it inlines into, and the same pixel could then round
    // differently alone and in a batch.
    __device__ static T cvt(float x) {
        asm("" : "+v"(x));
        return (_Float16)x;
    }
};

template <> struct Out<OUT_RGBN> : Out<OUT_F16> {};

template <int PX> struct MaskWord;
template <> struct MaskWord<1> { using T = uint8_t; };
template <> struct MaskWord<2> { using T = uint16_t; };
template <> struct MaskWord<4> { using T = uint32_t; };

// Row r of the three-row window together with the pair reciprocals between
// it and row r + 1.
template <int PX> struct RowState {
    Row<PX> row;
    Pairs<PX> below;
};

// B + half times the median's double: x3 + x4, or 2 x3 if an odd number
// of values is kept.
__device__ __forceinline__ float median_pair(const float (&t)[8], bool odd, float half, float B) {
    float x3, x4;
    middle_pair(t, x3, x4);
    return fmaf(half, x3 + (odd ? x3 : x4), B);
}

// Candidates t_j = N_j w_j of the 8 slots (see the file header).  For
// disparity, t_j without its factor -d, which all slots share (a negative
// factor reverses the order, but the middle one or two stay the same).
// Called
// inside each branch of the aggregation so that the min/max network sees
// values produced in its own basic block (the compiler then knows they are
// canonical and inserts no quieting instructions).
template <int KIND>
__device__ __forceinline__ void candidates(const float (&Nj)[8], const float (&rj)[8], float zc,
                                           float (&t)[8]) {
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        if constexpr (KIND == KIND_DISP)
            t[j] = Nj[j] * rj[j];
        else
            t[j] = fmaf(Nj[j] * zc, rj[j], Nj[j]);
    }
}

// B + the median of the kept candidates; zj/zc decide which slots are left out.
// `general` pads left-out slots alternately +inf / -inf; otherwise all 8
// are kept.  With nothing kept, the four +inf and four -inf pads give
// -inf + inf = NaN, which the caller's norm test turns into the degenerate
// normal.
// A neighbour gives no candidate when its raw value equals the centre's
// (dZ = 0) or, under the lenient rule, when it is invalid.
template <bool LEN> __device__ __forceinline__ bool left_out(float zj, float zc) {
    if constexpr (LEN) return !__builtin_islessgreater(zj, zc);  // invalid: NaN
    return zj == zc;
}

template <int KIND, bool LEN>
__device__ __forceinline__ float median8(const float (&Nj)[8], const float (&rj)[8],
                                         const float (&zj)[8], float zc, float B, bool general) {
    float t[8];
    candidates<KIND>(Nj, rj, zc, t);
    const float half = KIND == KIND_DISP ? -0.5f * zc : 0.5f;
    if (!general) return median_pair(t, false, half, B);
    float pad = kInf;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const bool drop = left_out<LEN>(zj[j], zc);
        t[j] = drop ? pad : t[j];
        pad = drop ? -pad : pad;
    }
    return median_pair(t, pad < 0.f, half, B);  // odd number left out -> position 3
}

// Sum of the candidates of the 8 slots.  Opposite slots share their N_j up to
// the sign.  Depth: t_j = N_j z_j rho_j (z_j rho_j = 1 + z rho_j), so a slot
// whose reciprocal is 0 adds 0.  Disparity: without the factor -d.
template <int KIND>
__device__ __forceinline__ float slot_sum(float Gu, float Gv, const float (&rj)[8],
                                          const float (&zj)[8]) {
    // the diagonals' N are +-(G_u + G_v) and +-(G_u - G_v), formed first: along
    // a line of nearly equal depth the pair's sum is large and its N small, and
    // products with G_u and G_v apart would cancel: 20-60 % more rms error
    // against 64 bits on indoor depth and slanted surfaces, for 1 % of time
    const float Spp = Gu + Gv, Spm = Gu - Gv;
    if constexpr (KIND == KIND_DISP) {
        const float s = fmaf(Spm, rj[7] - rj[6], Spp * (rj[4] - rj[5]));
        return fmaf(Gu, rj[0] - rj[1], fmaf(Gv, rj[2] - rj[3], s));
    } else {
        const float q0 = fmaf(zj[0], rj[0], -(zj[1] * rj[1]));
        const float q1 = fmaf(zj[2], rj[2], -(zj[3] * rj[3]));
        const float q2 = fmaf(zj[4], rj[4], -(zj[5] * rj[5]));
        const float q3 = fmaf(zj[7], rj[7], -(zj[6] * rj[6]));
        return fmaf(Gu, q0, fmaf(Gv, q1, fmaf(Spm, q3, Spp * q2)));
    }
}

// B + the mean of the kept candidates, strict rule (lenient means take the pair
// form, kPairMean).  1/8 is exact and v_rcp_f32 returns it
// exactly for m = 8, so a pixel with nothing left out gets the same bits
// whichever path its wavefront takes.  With nothing kept the sum is 0 and
// 0 * (1/0) is NaN, which the caller's norm test turns into the degenerate
// normal.
template <int KIND>
__device__ __forceinline__ float finish_mean(float sum, float weight, float zc, float B) {
    if constexpr (KIND == KIND_DISP) return fmaf(-(sum * zc), weight, B);
    return fmaf(sum, weight, B);
}
template <int KIND>
__device__ __forceinline__ float mean8(float Gu, float Gv, const float (&rj)[8],
                                       const float (&zj)[8], float zc,
                                       float B, bool general) {
    if (!general) return finish_mean<KIND>(slot_sum<KIND>(Gu, Gv, rj, zj), 0.125f, zc, B);
    float r[8];
    int m = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const bool drop = left_out<false>(zj[j], zc);
        r[j] = drop ? 0.f : rj[j];
        m += drop ? 0 : 1;
    }
    return finish_mean<KIND>(slot_sum<KIND>(Gu, Gv, r, zj), rcp((float)m), zc, B);
}

// Outputs are written once and not read back by this kernel: nontemporal
// stores keep them from displacing the input rows that neighbouring tiles
// still read from the caches.  The pointers are cast to the global address
// space: the uneven batch reads its frames' addresses from memory, and stores
// through a generic pointer would be flat ones, with a 64-bit address formed
// per lane instead of a scalar base and a 32-bit offset.
// The vectors are only as aligned as their elements (rows of any width start
// anywhere): the GPU's memory instructions take any alignment.
#define SNE_GLOBAL __attribute__((address_space(1)))
template <typename V> __device__ __forceinline__ void store_stream(SNE_GLOBAL char *p, const V &v) {
    if constexpr (sizeof(V) == 16) {
        typedef unsigned U __attribute__((ext_vector_type(4), aligned(1)));
        __builtin_nontemporal_store(__builtin_bit_cast(U, v), (SNE_GLOBAL U *)p);
    } else if constexpr (sizeof(V) == 8) {
        typedef unsigned U __attribute__((ext_vector_type(2), aligned(1)));
        __builtin_nontemporal_store(__builtin_bit_cast(U, v), (SNE_GLOBAL U *)p);
    } else if constexpr (sizeof(V) == 4) {
        typedef unsigned U __attribute__((aligned(1)));
        __builtin_nontemporal_store(__builtin_bit_cast(U, v), (SNE_GLOBAL U *)p);
    } else if constexpr (sizeof(V) == 2) {
        typedef unsigned short U __attribute__((aligned(1)));
        __builtin_nontemporal_store(__builtin_bit_cast(U, v), (SNE_GLOBAL U *)p);
    } else {
        static_assert(sizeof(V) == 1, "store width");
        __builtin_nontemporal_store(__builtin_bit_cast(unsigned char, v),
                                    (SNE_GLOBAL unsigned char *)p);
    }
}
// The first sizeof(V) / sizeof(E) - skip elements of a vector, one by one
// (Tail).  The vector is taken as it was packed for the whole lanes: asking
// for its elements would make the compiler convert them one by one for those
// too.
template <typename E, typename V>
__device__ __forceinline__ void store_front(SNE_GLOBAL char *p, const V &v, int skip) {
    constexpr int N = (int)(sizeof(V) / sizeof(E));
    constexpr int W = (int)((sizeof(V) + 3) / 4), kPer = (int)(4 / sizeof(E));
    uint32_t w[W] = {};
    __builtin_memcpy(w, &v, sizeof(V));
#pragma unroll
    for (int i = 0; i < W; ++i) asm("" : "+v"(w[i]));
#pragma unroll
    for (int k = 0; k + 1 < N; ++k) {
        if (k + skip >= N) break;
        const uint32_t bits = w[k / kPer] >> (8 * sizeof(E) * (k % kPer));
        if constexpr (sizeof(E) == 4) store_stream(p + 4 * k, bits);
        else if constexpr (sizeof(E) == 2) store_stream(p + 2 * k, (uint16_t)bits);
        else store_stream(p + k, (uint8_t)bits);
    }
}
// A wave-uniform pointer as a base for store_stream.
__device__ __forceinline__ SNE_GLOBAL char *store_base(const void *p) {
    return (SNE_GLOBAL char *)const_cast<void *>(p);
}

// s_b - s_a of two samples (a before b along the line): for depth
// (z_a - z_b) s_a s_b, the form the named kernels use; for disparity d_b - d_a.
template <int KIND>
__device__ __forceinline__ float one_sided(float za, float zb, float sa, float sb) {
    if constexpr (KIND == KIND_DISP)
        return zb - za;
    else
        return (za - zb) * (sa * sb);
}

// One gradient line under the lenient rule: samples zm (minus side), z0
// (middle), zp (plus side) with the filtered values sm, s0, sp and the line's
// central difference `both` (sp - sm, formed as the strict path forms it).
// Returns the line's difference (0 if it has none) and sets `have`.
template <int KIND>
__device__ __forceinline__ float lenient_line(float zm, float z0, float zp, float sm, float s0,
                                              float sp, float both, Mask okm, Mask ok0, Mask okp,
                                              Mask &have) {
    float plus, minus;  // one-sided: 2 (sp - s0) and 2 (s0 - sm)
    if constexpr (KIND == KIND_DISP) {
        plus = 2.f * (zp - z0);
        minus = 2.f * (z0 - zm);
    } else {
        plus = 2.f * ((z0 - zp) * (s0 * sp));
        minus = 2.f * ((zm - z0) * (sm * s0));
    }
    have = (okm & okp) | (ok0 & (okm | okp));
    const bool two = lane(okm & okp), any = lane(have), up = lane(okp);
    const float one = up ? plus : minus;
    const float some = any ? one : 0.f;
    return two ? both : some;
}

// The lenient horizontal lines of a finished row.
template <int KIND, int PX> __device__ __forceinline__ void lenient_hlines(Row<PX> &o) {
#pragma unroll
    for (int k = 0; k < PX; ++k)
        o.Lh[k] = lenient_line<KIND>(o.z[k], o.z[k + 1], o.z[k + 2], o.s[k], o.s[k + 1],
                                     o.s[k + 2], o.D[k], o.ok[k], o.ok[k + 1], o.ok[k + 2],
                                     o.hh[k]);
}

// Lenient G from its lines (centre line c, side lines a and b, each 0 when
// missing): the strict combination of the available lines, rescaled to the
// full filter's weight.  With every line present it is the strict value.
__device__ __forceinline__ float lenient_combine(float c, Mask hc, float a, Mask ha, float b,
                                                 Mask hb, const GradW &w, Mask &have) {
    const float g = fmaf(w.wa, a + b, c);
    const Mask both = ha & hb, any = ha | hb;
    have = hc | any;
    const bool centre = lane(hc), two = lane(both), some = lane(any);
    const float with_side = some ? w.r[0] : w.r[1];
    const float with = two ? 1.f : with_side, without = two ? w.r[2] : w.r[3];
    return g * (centre ? with : without);
}

// n_z of column k of the middle row: B + Phi over the 8 slots.  `scale` is a
// factor that n_x and n_y still need (1 unless set).
template <int KIND, int AGG, bool LEN, bool GENERAL, int PX>
__device__ __forceinline__ float normal_z(int k, const FrameDesc &f, int col, float fv, float Gu,
                                          float Gv, float &scale, const Row<PX> &rp,
                                          const Row<PX> &rc,
                                          const Row<PX> &rn, const Pairs<PX> &pu,
                                          const Pairs<PX> &pd) {
    const int c = k + 1;
    const float zc = rc.z[c];
    const float fu = (float)(col + k) - f.u0;
    const float B = fmaf(fu, Gu, fv * Gv);
    // slots: E, W, S, N, SE, NW, SW, NE
    const float zj[8] = {rc.z[c + 1], rc.z[c - 1], rn.z[c], rp.z[c],
                         rn.z[c + 1], rp.z[c - 1], rn.z[c - 1], rp.z[c + 1]};
    const float rj[8] = {rc.rE[c], -rc.rE[c - 1], pd.rS[k], -pu.rS[k],
                         pd.rSE[c], -pu.rSE[k], pd.rSW[k], -pu.rSW[c]};
    if constexpr (kPairCount<KIND, AGG, LEN>) {
        // the vector times m instead of the sum divided by it (quantised
        // depth keeps it far from the ends of the FP32 range); m = 0 gives
        // the zero vector, hence the degenerate normal
        scale = (pu.above[k] + pd.under[k]) + rc.mid[k];
        return fmaf(scale, B, slot_sum<KIND>(Gu, Gv, rj, zj));
    } else if constexpr (kPairMean<KIND, AGG, LEN>) {
        int m = pu.top[k];
        m += lane(rc.kE[c]) ? 1 : 0;
        m += lane(rc.kE[c - 1]) ? 1 : 0;
        m += lane(pd.kS[k]) ? 1 : 0;
        m += lane(pd.kSE[c]) ? 1 : 0;
        m += lane(pd.kSW[k]) ? 1 : 0;
        const float sum = slot_sum<KIND>(Gu, Gv, rj, zj);
        if constexpr (kTieHeavy<KIND>) {
            scale = (float)m;  // as above
            return fmaf(scale, B, sum);
        }
        return finish_mean<KIND>(sum, rcp((float)m), zc, B);
    } else if constexpr (AGG == AGG_MEAN) {
        return mean8<KIND>(Gu, Gv, rj, zj, zc, B, GENERAL);
    } else {
        const float Spp = Gu + Gv, Spm = Gu - Gv;
        const float Nj[8] = {Gu, -Gu, Gv, -Gv, Spp, -Spp, -Spm, Spm};
        return median8<KIND, LEN>(Nj, rj, zj, zc, B, GENERAL);
    }
}

// Output row r of a tile from the window (prev, cur, next); `pend` holds the
// raw loads of row r + 1 on entry and those of row r + 1 + SNE_PREFETCH_ROWS
// on exit.
template <int KIND, int GK, int AGG, int OUT, int PX, bool HALF, bool LEN>
__device__ __forceinline__ void tile_row(const FrameDesc &f, const InBuf &ib, const InBuf &rgbb,
                                         int r, int rend, int col, int col_off, int halo_off,
                                         const Edges &e, const Tail &tail, const GradW &gw,
                                         RawRow<KIND, PX> &pend,
                                         const RowState<PX> &prev, RowState<PX> &cur,
                                         RowState<PX> &next) {
    constexpr bool FD = GK == GK_FD;
    constexpr bool LENR = LEN && GK != GK_CUSTOM;  // the lenient rule applies
    finish_row<KIND, AGG, PX, HALF, FD, LEN>(pend, next.row, e, tail);
    if constexpr (LENR && !FD) lenient_hlines<KIND, PX>(next.row);
    load_raw<KIND, PX>(ib, r + 1 + SNE_PREFETCH_ROWS, col_off, halo_off, pend);  // prefetch
    // packed output: this row's RGBX bytes, in flight while the row is
    // computed (a frame without colour has an empty resource: zeros)
    Vec<float, PX> rgbx;
    if constexpr (OUT == OUT_RGBN) {
        rgbx = buf_load<float, PX>(
            rgbb, (int)((unsigned)r * (unsigned)rgbb.pitch_bytes +
                        (unsigned)(col_off < kOOB ? (col - tail.skip) * 4 : kOOB)));
        if constexpr (PX > 1)
            if (tail.any) shift_down<PX>(rgbx, tail.skip);
    }
    make_middle<KIND, AGG, PX, FD, LEN>(cur.row);
    make_pairs<KIND, AGG, LEN, PX>(cur.row, next.row, cur.below);
    const Row<PX> &rp = prev.row, &rc = cur.row, &rn = next.row;
    const Pairs<PX> &pu = prev.below, &pd = cur.below;

    // vertical central differences of s at columns -1..PX
    float V[PX + 2];
#pragma unroll
    for (int i = 0; i < PX + 2; ++i) {
        if constexpr (FD) {
            if (i == 0 || i == PX + 1) { V[i] = 0.f; continue; }
        }
        if constexpr (KIND == KIND_DISP)
            V[i] = rn.z[i] - rp.z[i];
        else
            V[i] = (rp.z[i] - rn.z[i]) * (rp.s[i] * rn.s[i]);
    }

    // lenient rule: when a valid pixel of this row somewhere in the
    // wavefront lacks a full window, its vertical lines at columns 0..PX+1
    // (each used by three pixels; the horizontal ones come with the rows)
    bool lenient_path = false;
    float VL[PX + 2];
    Mask VH[PX + 2];
    if constexpr (LENR && !FD) {
        Mask need = 0;
#pragma unroll
        for (int k = 0; k < PX; ++k)
            need |= rc.ok[k + 1] & ~(rp.hok[k] & rc.hok[k] & rn.hok[k]);
        if (need != 0) {
            lenient_path = true;
#pragma unroll
            for (int i = 0; i < PX + 2; ++i)
                VL[i] = lenient_line<KIND>(rp.z[i], rc.z[i], rn.z[i], rp.s[i], rc.s[i], rn.s[i],
                                           V[i], rp.ok[i], rc.ok[i], rn.ok[i], VH[i]);
        }
    }

    // pixels that take the general aggregation whatever the vote below says
    bool general[PX];
#pragma unroll
    for (int k = 0; k < PX; ++k) general[k] = kTieHeavy<KIND> || kPairMean<KIND, AGG, LEN>;

    float Gu[PX], Gv[PX];
    Mask valid[PX];
#pragma unroll
    for (int k = 0; k < PX; ++k) {
        const int c = k + 1;
        valid[k] = rp.hok[k] & rc.hok[k] & rn.hok[k];
        if constexpr (FD) {
            Gu[k] = rc.D[k];
            Gv[k] = V[c];
        } else if constexpr (GK == GK_CUSTOM) {
            // any 3x3 K_x: per line k2 (s_+ - s_0) - k0 (s_0 - s_-) + ks s_0;
            // line a of K_y (column c + a - 1) is row a of K_x
            Gu[k] = 0.f;
            Gv[k] = 0.f;
#pragma unroll
            for (int a = 0; a < 3; ++a) {
                const Row<PX> &X = a == 0 ? rp : (a == 1 ? rc : rn);
                const float hp = one_sided<KIND>(X.z[c], X.z[c + 1], X.s[c], X.s[c + 1]);
                const float hm = one_sided<KIND>(X.z[c - 1], X.z[c], X.s[c - 1], X.s[c]);
                Gu[k] += fmaf(gw.k2[a], hp, fmaf(-gw.k0[a], hm, gw.ks[a] * X.s[c]));
                const int b = c + a - 1;
                const float vp = one_sided<KIND>(rc.z[b], rn.z[b], rc.s[b], rn.s[b]);
                const float vm = one_sided<KIND>(rp.z[b], rc.z[b], rp.s[b], rc.s[b]);
                Gv[k] += fmaf(gw.k2[a], vp, fmaf(-gw.k0[a], vm, gw.ks[a] * rc.s[b]));
            }
        } else {
            // the 3-row filter divided by its centre weight (wa = side /
            // centre): n' scales as a whole, the normal does not change
            Gu[k] = fmaf(gw.wa, rp.D[k] + rn.D[k], rc.D[k]);
            Gv[k] = fmaf(gw.wa, V[c - 1] + V[c + 1], V[c]);
        }
        // with every line present the lenient G is the strict one, bit for
        // bit, so pixels with a full window may take either path
        if constexpr (LENR && FD) {
            // FD has one line per direction: decided per column position,
            // nothing shared
            if ((rc.ok[c] & ~valid[k]) != 0) {
                general[k] = true;
                Mask hc, vc;
                Gu[k] = lenient_line<KIND>(rc.z[c - 1], rc.z[c], rc.z[c + 1], rc.s[c - 1],
                                           rc.s[c], rc.s[c + 1], rc.D[k], rc.ok[c - 1], rc.ok[c],
                                           rc.ok[c + 1], hc);
                Gv[k] = lenient_line<KIND>(rp.z[c], rc.z[c], rn.z[c], rp.s[c], rc.s[c], rn.s[c],
                                           V[c], rp.ok[c], rc.ok[c], rn.ok[c], vc);
                valid[k] = rc.ok[c] & hc & vc;
            }
        }
    }
    if constexpr (LENR && !FD) {
        if (lenient_path) {
#pragma unroll
            for (int k = 0; k < PX; ++k) {
                const int c = k + 1;
                Mask du, dv;
                Gu[k] = lenient_combine(rc.Lh[k], rc.hh[k], rp.Lh[k], rp.hh[k], rn.Lh[k],
                                        rn.hh[k], gw, du);
                Gv[k] = lenient_combine(VL[c], VH[c], VL[c - 1], VH[c - 1], VL[c + 1],
                                        VH[c + 1], gw, dv);
                valid[k] = rc.ok[c] & du & dv;
            }
        }
    }
    const float fv = (float)r - f.v0;
    float nz[PX];
    bool done = false;
    if constexpr (LENR && !FD && !kTieHeavy<KIND> && !kPairMean<KIND, AGG, LEN>) {
        // one branch for the row: no test of its pixels' ties
        if (lenient_path) {
            float unused;
#pragma unroll
            for (int k = 0; k < PX; ++k) {
                // values of their own: otherwise the compiler forms the
                // candidates ahead of the branch, for both sides of it, and
                // holds those of all pixels at once
                asm("" : "+v"(Gu[k]), "+v"(Gv[k]));
                nz[k] = normal_z<KIND, AGG, LEN, true, PX>(k, f, col, fv, Gu[k], Gv[k], unused, rp,
                                                           rc, rn, pu, pd);
            }
        }
        done = lenient_path;
    }
    if (!done) {
#pragma unroll
        for (int k = 0; k < PX; ++k) {
            // A slot is left out iff raw_j == raw, i.e. its pair reciprocal is
            // +-inf.  That is rare in FP32 data: pad only when a valid pixel of
            // this wavefront needs it (the choice is wave-uniform, and both paths
            // give the same result when nothing is left out).
            // (signs do not matter here: the raw pair values are used)
            // For the mean, a class test of the plain sum says the same in one
            // half-rate instruction instead of five, but a pixel with ties
            // then forms both sums: 64 x 480x640 FD-mean, FP16 output, 42.6
            // instead of 42.9 us on depth without ties (1-3 % in 48 forms), 57.0
            // instead of 51.1 on millimetres converted to metres (6 %, at most 13).
            if constexpr (!kTieHeavy<KIND> && !kPairMean<KIND, AGG, LEN>) {
                const int c = k + 1;
                const float rmax = vmax8abs(rc.rE[c], rc.rE[c - 1], pd.rS[k], pu.rS[k], pd.rSE[c],
                                            pu.rSE[k], pd.rSW[k], pu.rSW[c]);
                general[k] = general[k] || (mask_of(rmax == kInf) & valid[k]) != 0;
            }
            float scale = 1.f;
            if (general[k])
                nz[k] = normal_z<KIND, AGG, LEN, true, PX>(k, f, col, fv, Gu[k], Gv[k], scale, rp, rc,
                                                           rn, pu, pd);
            else
                nz[k] = normal_z<KIND, AGG, LEN, false, PX>(k, f, col, fv, Gu[k], Gv[k], scale, rp, rc,
                                                            rn, pu, pd);
            if constexpr (kTieHeavy<KIND> && kPairMean<KIND, AGG, LEN>) {
                Gu[k] *= scale;
                Gv[k] *= scale;
            }
        }
    }

    using OT = typename Out<OUT>::T;
    Vec<OT, PX> ox, oy, oz;
    bool mk[PX];
    float fz[PX];
    Mask deg[PX], any_deg = 0;
#pragma unroll
    for (int k = 0; k < PX; ++k) {
        const float nx = f.fx * Gu[k], ny = f.fy * Gv[k];
        const float n2 = fmaf(nx, nx, fmaf(ny, ny, nz[k] * nz[k]));
        // n2 is NaN where nothing was kept and 0 for a zero vector: there the
        // normal is (0, 0, -1), set below for the few rows that hold one
        const Mask pos = mask_of(n2 > 0.f);
        deg[k] = valid[k] & ~pos;
        any_deg |= deg[k];
        const bool keep = lane(valid[k] & pos);
        const float rs = __builtin_amdgcn_rsqf(n2);
        const float inv = keep ? rs : 0.f;
        ox.v[k] = Out<OUT>::cvt(neg_mul_or_zero(nx, inv));
        oy.v[k] = Out<OUT>::cvt(neg_mul_or_zero(ny, inv));
        fz[k] = mul_or_zero(nz[k], inv);
        mk[k] = lane(valid[k]);
    }
    if (any_deg != 0) {
#pragma unroll
        for (int k = 0; k < PX; ++k) {
            const bool d = lane(deg[k]);
            fz[k] = d ? -1.f : fz[k];
        }
    }
#pragma unroll
    for (int k = 0; k < PX; ++k) oz.v[k] = Out<OUT>::cvt(fz[k]);
    if constexpr (OUT == OUT_RGBN) {
        // one 16-byte pixel: R, G, B (bytes / 255), mask, n_x, n_y, n_z, 0
        typedef unsigned U4 __attribute__((ext_vector_type(4)));
        U4 px[PX];
#pragma unroll
        for (int k = 0; k < PX; ++k) {
            const unsigned c = __builtin_bit_cast(unsigned, rgbx.v[k]);
            const float s255 = 1.f / 255.f;
            const _Float16 R = Out<OUT_F16>::cvt((float)(c & 0xffu) * s255);
            const _Float16 G = Out<OUT_F16>::cvt((float)((c >> 8) & 0xffu) * s255);
            const _Float16 Bc = Out<OUT_F16>::cvt((float)((c >> 16) & 0xffu) * s255);
            const _Float16 M = mk[k] ? (_Float16)1.f : (_Float16)0.f;
            typedef _Float16 H8 __attribute__((ext_vector_type(8)));
            px[k] = __builtin_bit_cast(U4, H8{R, G, Bc, M, ox.v[k], oy.v[k], oz.v[k],
                                              (_Float16)0.f});
        }
        // A lane's pixels are 16 PX contiguous bytes, but one store
        // instruction would scatter 16-byte pieces 16 PX bytes apart (3.6
        // times slower at 4 columns).  Each wavefront turns its row around
        // through LDS, so that a store covers kLanes contiguous pixels.
        // Slots are swizzled by lane so that neither direction has bank
        // conflicts.  One wavefront uses each part: no barrier, only order.
        // 64 x 480x640 with colour (24 bytes a pixel): 89 us at 2 columns,
        // 5.3 TB/s, against 98 us at 1 column without the turn.
        constexpr int kLanes = HALF ? kWave / 2 : kWave;
        const int llane = (int)threadIdx.x & (kLanes - 1), c0 = col - llane * PX;
        const unsigned row = (unsigned)r * (unsigned)f.out_pitch;
        SNE_GLOBAL char *o = store_base(f.out);
        if constexpr (PX == 1) {
            if (col < f.W && r < rend) store_stream(o + (row + (unsigned)col) * 16u, px[0]);
        } else {
            __shared__ U4 turn[kBlock * PX];
            U4 *part = turn + ((int)threadIdx.x - llane) * PX;
            auto slot = [](int l, int k) { return l * PX + (k ^ ((l * PX / 16) & (PX - 1))); };
            asm volatile("" ::: "memory");
#pragma unroll
            for (int k = 0; k < PX; ++k) part[slot(llane, k)] = px[k];
            __builtin_amdgcn_wave_barrier();
            asm volatile("" ::: "memory");
#pragma unroll
            for (int j = 0; j < PX; ++j) {
                const int v = j * kLanes + llane;
                const U4 q = part[slot(v / PX, v % PX)];
                if (c0 + v < f.W && r < rend)
                    store_stream(o + (row + (unsigned)(c0 + v)) * 16u, q);
            }
        }
        if (f.mask) {
            typename MaskWord<PX>::T w = 0;
#pragma unroll
            for (int k = 0; k < PX; ++k) w |= (typename MaskWord<PX>::T)mk[k] << (8 * k);
            SNE_GLOBAL char *m =
                store_base(f.mask) + ((unsigned)r * (unsigned)f.mask_pitch + (unsigned)col);
            if (col + PX <= f.W && r < rend) store_stream(m, w);
            if constexpr (PX > 1)
                if (tail.any && tail.skip > 0 && r < rend) store_front<uint8_t>(m, w, tail.skip);
        }
    } else {
        // uniform plane bases + one 32-bit byte offset per lane (the host
        // keeps each plane below 4 GiB)
        SNE_GLOBAL char *o = store_base(f.out);
        const int64_t plane = f.out_plane * (int64_t)sizeof(OT);
        const unsigned off = ((unsigned)r * (unsigned)f.out_pitch + (unsigned)col) * sizeof(OT);
        const unsigned moff = (unsigned)r * (unsigned)f.mask_pitch + (unsigned)col;
        typename MaskWord<PX>::T w = 0;
        if (f.mask) {
#pragma unroll
            for (int k = 0; k < PX; ++k) w |= (typename MaskWord<PX>::T)mk[k] << (8 * k);
        }
        if (col + PX <= f.W && r < rend) {
            store_stream(o + off, ox);
            store_stream(o + plane + off, oy);
            store_stream(o + 2 * plane + off, oz);
            if (f.mask) store_stream(store_base(f.mask) + moff, w);
        }
        if constexpr (PX > 1)
            if (tail.any && tail.skip > 0 && r < rend) {
                store_front<OT>(o + off, ox, tail.skip);
                store_front<OT>(o + plane + off, oy, tail.skip);
                store_front<OT>(o + 2 * plane + off, oz, tail.skip);
                if (f.mask) store_front<uint8_t>(store_base(f.mask) + moff, w, tail.skip);
            }
    }
}

// One tile: columns [c0, c0 + 64 PX) x rows [r0, r0 + rows) of frame f, or
// in half-wave mode two tiles of 32 PX columns: lanes 0-31 take rows
// [r0, r0 + rows), lanes 32-63 rows [r0 + rows, r0 + 2 rows) of the same
// strip (the frame, hence the buffer resource, stays wave-uniform).  Rows
// past the frame read as 0 and are not stored.  The row loop is unrolled three
// times with the window's roles rotating, so no register state is copied.
template <int KIND, int GK, int AGG, int OUT, int PX, bool HALF, bool LEN>
__device__ __forceinline__ void run_tile(const FrameDesc &f, int c0, int r0, int rows,
                                         const GradW &kgw) {
    using T = typename Raw<KIND>::T;
    // The lenient rule selects among the rescaling factors per lane; left in
    // the kernel arguments, the select becomes one of their addresses and a
    // memory load per pixel.
    GradW gw = kgw;
    if constexpr (LEN)
        asm("" : "+s"(gw.r[0]), "+s"(gw.r[1]), "+s"(gw.r[2]), "+s"(gw.r[3]));
    constexpr int kLanes = HALF ? kWave / 2 : kWave;
    const int lane = threadIdx.x & (kWave - 1);
    const int llane = lane & (kLanes - 1);
    const int col = c0 + llane * PX;
    const int esz = (int)sizeof(T);
    const InBuf ib = make_inbuf(f.in, f.in_pitch, f.H, esz);
    InBuf rgbb{};
    if constexpr (OUT == OUT_RGBN) rgbb = make_inbuf(f.rgb, f.rgb ? f.rgb_pitch : 0, f.H, 1);
    // (a frame narrower than PX columns is never given PX columns per lane)
    const Tail tail{PX > 1 && c0 + kLanes * PX > f.W && f.W % PX != 0,
                    col < f.W ? max(col + PX - f.W, 0) : 0};
    const int col_off = col < f.W ? (col - tail.skip) * esz : kOOB;
    int hcol = -1;
    if (llane == 0) hcol = c0 - 1;
    if (llane == kLanes - 1) hcol = c0 + kLanes * PX;
    const int halo_off = (hcol >= 0 && hcol < f.W) ? hcol * esz : kOOB;
    const Edges e{HALF && lane == kLanes, HALF && lane == kLanes - 1};
    const int rb = HALF ? r0 + (lane >> 5) * rows : r0;  // first row of this lane's band
    const int rend = min(rb + rows, f.H);                // rows stored: [rb, rend)
    const int n = HALF ? rows : rend - rb;               // wave-uniform iterations

    RawRow<KIND, PX> p0;
    RowState<PX> A, B, C;
    load_raw<KIND, PX>(ib, rb - 1, col_off, halo_off, p0);
    finish_row<KIND, AGG, PX, HALF, GK == GK_FD, LEN>(p0, A.row, e, tail);
    load_raw<KIND, PX>(ib, rb, col_off, halo_off, p0);
    finish_row<KIND, AGG, PX, HALF, GK == GK_FD, LEN>(p0, B.row, e, tail);
    if constexpr (LEN && GK == GK_3ROW) {  // the lenient rule's shared horizontal lines
        lenient_hlines<KIND, PX>(A.row);
        lenient_hlines<KIND, PX>(B.row);
    }
    make_pairs<KIND, AGG, LEN, PX>(A.row, B.row, A.below);
    load_raw<KIND, PX>(ib, rb + 1, col_off, halo_off, p0);
#define SNE_ROW(I, P, X, Y, Z)                                                                  \
    tile_row<KIND, GK, AGG, OUT, PX, HALF, LEN>(f, ib, rgbb, rb + (I), rend, col, col_off, halo_off, \
                                                e, tail, gw, P, X, Y, Z)
#if SNE_PREFETCH_ROWS == 1
    for (int i = 0; i < n; i += 3) {
        SNE_ROW(i, p0, A, B, C);
        if (i + 1 >= n) break;
        SNE_ROW(i + 1, p0, B, C, A);
        if (i + 2 >= n) break;
        SNE_ROW(i + 2, p0, C, A, B);
    }
#else
    // two rows in flight: p0 and p1 alternate; the loop covers six rows (the
    // common period of the window roles and the two load buffers), so no
    // buffer is ever copied (a copy would wait for its load)
    RawRow<KIND, PX> p1;
    load_raw<KIND, PX>(ib, rb + 2, col_off, halo_off, p1);
    for (int i = 0; i < n; i += 6) {
        SNE_ROW(i, p0, A, B, C);
        if (i + 1 >= n) break;
        SNE_ROW(i + 1, p1, B, C, A);
        if (i + 2 >= n) break;
        SNE_ROW(i + 2, p0, C, A, B);
        if (i + 3 >= n) break;
        SNE_ROW(i + 3, p1, A, B, C);
        if (i + 4 >= n) break;
        SNE_ROW(i + 4, p0, B, C, A);
        if (i + 5 >= n) break;
        SNE_ROW(i + 5, p1, C, A, B);
    }
#endif
#undef SNE_ROW
}

// Blocks are handed to the 8 XCDs round-robin; renumber them so that XCD x
// works on a contiguous range of tiles (vertically adjacent tiles share halo
// rows through that XCD's L2).
__device__ __forceinline__ int xcd_block(int b, int nb) {
    const int x = b & 7, i = b >> 3;
    const int q = nb >> 3, rem = nb & 7;
    return x * q + min(x, rem) + i;
}

// Runs of G: XCD x takes runs of G consecutive blocks, the runs of the 8
// XCDs interleaved, so the blocks resident at any time still cover one
// window of the batch (the plain order's DRAM locality) while vertically
// adjacent tiles mostly meet in one XCD's L2 (their shared halo rows are
// fetched once).  Blocks of a partial last round of 8 G keep their order.
__device__ __forceinline__ int xcd_chunk(int b, int nb, int G) {
    const int full = nb / (8 * G) * (8 * G);
    if (b >= full) return b;
    const int x = b & 7, i = b >> 3;
    return (i / G) * (8 * G) + x * G + (i % G);
}

template <int KIND, int GK, int AGG, int OUT, int PX, bool HALF, bool LEN>
__global__ __launch_bounds__(kBlock) SNE_OCCUPANCY void sne_uniform_kernel(UniformArgs a) {
    const int b = a.xcd_remap == 1   ? xcd_block(blockIdx.x, gridDim.x)
                  : a.xcd_remap > 1 ? xcd_chunk(blockIdx.x, gridDim.x, a.xcd_remap)
                                    : (int)blockIdx.x;
    // wave-uniform by construction; readfirstlane lets the compiler keep the
    // frame's buffer resource in scalar registers
    const int tile = __builtin_amdgcn_readfirstlane(b * kWavesPerBlock + (int)(threadIdx.x >> 6));
    if (tile >= a.ntiles) return;
    const int per_frame = a.nbands * a.nstrips;
    const int frame = tile / per_frame;
    const int rem = tile - frame * per_frame;
    const int band = rem / a.nstrips;
    const int strip = rem - band * a.nstrips;
    FrameDesc f = a.f;
    using IT = typename Raw<KIND>::T;
    using OT = typename Out<OUT>::T;
    f.in = static_cast<const IT *>(a.f.in) + frame * a.in_fstride;
    f.out = static_cast<OT *>(a.f.out) + frame * a.out_fstride;
    if (f.mask) f.mask = a.f.mask + frame * a.mask_fstride;
    if constexpr (OUT == OUT_RGBN)
        if (f.rgb) f.rgb = static_cast<const char *>(a.f.rgb) + frame * a.rgb_fstride;
    // half-wave mode: a "band" is a pair of bands and a strip is 32 PX wide
    const int r0 = band * a.rows * (HALF ? 2 : 1);
    run_tile<KIND, GK, AGG, OUT, PX, HALF, LEN>(f, strip * (HALF ? kWave / 2 : kWave) * PX, r0,
                                                a.rows, a.gw);
}

// ------------------------------------------------ wide custom gradient filters
// A (2R+1)x(2R+1) custom K_x (R = 2, 3; K_y = K_x^T) reads R samples on each
// side, more than the three-row register window holds.  One block stages a
// 128 x 16 (64 x 16) output tile and its R-wide apron in LDS as (z, s) pairs (z = 0
// where invalid or outside the frame), then each thread takes 2 columns (1) by 4
// rows of pixels.  The taps are formed against one reference value z_r
// (s_r = 1 / z_r), the mean of the four middle pixels, which lie in the
// windows of all of them:
// sum_ab K_ab s_ab = sum_ab K_ab (s_ab - s_r) + (sum K) s_r, with
// s_ab - s_r = (z_r - z_ab) s_ab s_r from a raw-value difference (for
// disparity d_ab - d_r), so each sample's difference serves all 8 pixels
// (one pixel's sample as reference: 1.9e-7 rms of the 5x5 normals against 64
// bits, the mean 1.2e-7):
//   G = s_r (sum_ab K_ab (z_r - z_ab) s_ab + sum K)      (depth)
//   G = sum_ab K_ab (d_ab - d_r) + (sum K) d_r            (disparity)
// The neighbourhood of n_z stays the 8-connected one, and a pixel is kept iff
// its whole (2R+1)x(2R+1) window is inside the frame and valid.
// SEP: K_x = kc kr^T (a smoothing column times a derivative row, say); then
// each window row's two weighted sums serve every pixel of a column, so a
// pixel takes 2(2R+1) FMAs of row sums instead of 2(2R+1)^2 taps.  Its weights
// are held in vector registers: an FMA with a scalar operand issues at half
// rate.
// Bound by instruction issue.  Two columns per thread (CPT) share the
// reference's differences, the row minima and the pairs between them (6 instead
// of 8 reciprocals per pixel): 64 x 480x640 FP32 median, 5x5 product 73 us (98
// with one column), 7x7 product 87 (128), 5x5 general 79 (117).  A launch of
// few blocks takes as long as one thread: there one column per thread, half the
// tile, with the reference of the pair of columns, so that the bits stay the
// same (one frame, 5x5 product, FP32 median: 240x320 4.6 us, 6.1 with two
// columns, 480x640 5.5 against 6.4).  Tiles of 8 rows, 2 per thread, were no
// faster there (480x640 8.6 us with either at two columns).
// Blocks run in runs of kWideRun per XCD (xcd_chunk), so the tiles above and
// below a tile mostly share its apron rows through one L2.
constexpr int kWideRun = 16;

// A scalar weight as a vector register's value.
__device__ __forceinline__ float in_vgpr(float x) {
    float r;
    asm("v_mov_b32 %0, %1" : "=v"(r) : "s"(x));
    return r;
}

template <int KIND, int R, int AGG, int OUT, bool SEP, int CPT>
__global__ __launch_bounds__(kBlock) void sne_wide_kernel(WideArgs a) {
    constexpr int TW = kWave * CPT;                // tile width
    constexpr int N = 2 * R + 1, LW = TW + 2 * R, LH = kWideTH + 2 * R;
    constexpr int RPT = kWideTH / kWavesPerBlock;  // rows per thread
    constexpr int S = N + CPT - 1;                 // samples of a window row
    static_assert(RPT * kWavesPerBlock == kWideTH && (CPT == 1 || CPT == 2), "tile shape");
    static_assert(RPT >= 3 && RPT - 2 <= R && R >= 1, "the reference is in every window");
    static_assert((CPT == 1 || S % 2 == 0) && LW % 2 == 0, "16-byte LDS reads");
    __shared__ float4 T[LH * LW / 2];  // (z, s) of two columns
    using IT = typename Raw<KIND>::T;
    using OT = typename Out<OUT>::T;
    const int blk = xcd_chunk((int)blockIdx.x, (int)gridDim.x, kWideRun);
    if (blk >= a.nblocks) return;
    const int per_frame = a.ntx * a.nty;
    const int frame = blk / per_frame;
    const int rem = blk - frame * per_frame;
    const int ty = rem / a.ntx;
    const int x0 = (rem - ty * a.ntx) * TW, y0 = ty * kWideTH;
    FrameDesc f = a.f;
    f.in = static_cast<const IT *>(a.f.in) + frame * a.in_fstride;
    f.out = static_cast<OT *>(a.f.out) + frame * a.out_fstride;
    if (f.mask) f.mask = a.f.mask + frame * a.mask_fstride;
    const int esz = (int)sizeof(IT);
    const InBuf ib = make_inbuf(f.in, f.in_pitch, f.H, esz);
    const int lane = (int)threadIdx.x & (kWave - 1);
    const int wv = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));

    // stage pairs of columns (gx, gx + 1); samples outside the frame read as 0
    // (invalid).  A wavefront takes the first TW / 2 pairs of one row (of two
    // with CPT 1) at a time, and the apron pairs right of them go one to a
    // thread; all loads are issued before the first is used.
    constexpr int kPairs = TW / 2, kRows = kBlock / kPairs;  // rows per pass
    constexpr int kPasses = (LH + kRows - 1) / kRows;
    static_assert(LH * R <= kBlock, "one apron pair per thread");
    IT z0[kPasses + 1], z1[kPasses + 1];
    auto load_pair = [&](int row, int pair, IT &l, IT &r) {
        const int gy = y0 - R + row, gx = x0 - R + 2 * pair;
        const bool yin = gy >= 0 && gy < f.H;
        const int at = gy * ib.pitch_bytes + gx * esz;
        l = buf_load<IT, 1>(ib, yin && gx >= 0 && gx < f.W ? at : kOOB).v[0];
        r = buf_load<IT, 1>(ib, yin && gx + 1 >= 0 && gx + 1 < f.W ? at + esz : kOOB).v[0];
    };
    auto put_pair = [&](int row, int pair, IT l, IT r) {
        const float zl = Raw<KIND>::value(l), zr = Raw<KIND>::value(r);
        T[row * (LW / 2) + pair] = make_float4(zl, KIND == KIND_DISP ? zl : rcp(zl), zr,
                                               KIND == KIND_DISP ? zr : rcp(zr));
    };
    const int row0 = CPT == 2 ? wv : (int)threadIdx.x / kPairs;
    const int pair0 = (int)threadIdx.x & (kPairs - 1);
    const int arow = (int)threadIdx.x / R, apair = kPairs + (int)threadIdx.x % R;
    const bool apron = (int)threadIdx.x < LH * R;
#pragma unroll
    for (int i = 0; i < kPasses; ++i) load_pair(row0 + i * kRows, pair0, z0[i], z1[i]);
    if (apron) load_pair(arow, apair, z0[kPasses], z1[kPasses]);
#pragma unroll
    for (int i = 0; i < kPasses; ++i)
        if (LH % kRows == 0 || row0 + i * kRows < LH)
            put_pair(row0 + i * kRows, pair0, z0[i], z1[i]);
    if (apron) put_pair(arow, apair, z0[kPasses], z1[kPasses]);
    __syncthreads();

    const int top = wv * RPT;  // LDS row of pixel row 0's window top
    const int x = x0 + CPT * lane;
    // the first pair of the window; of that of the even column with CPT 1
    const float4 *base = T + top * (LW / 2) + lane / (2 / CPT);
    // the reference all window sums subtract: the mean of the four pixels in
    // the middle of 2 columns by 4 rows, each in the windows of all of these
    float near[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const float4 l = base[(1 + i + R) * (LW / 2) + R / 2];
        near[i][0] = R % 2 ? l.z : l.x;
        near[i][1] = R % 2 ? base[(1 + i + R) * (LW / 2) + R / 2 + 1].x : l.z;
    }
    const float rz = (0.25f * near[0][0] + 0.25f * near[0][1]) +
                     (0.25f * near[1][0] + 0.25f * near[1][1]);
    const float2 ref = make_float2(rz, KIND == KIND_DISP ? rz : rcp(rz));
    float kc[N], kr[N];
    if constexpr (SEP) {
#pragma unroll
        for (int b = 0; b < N; ++b) {
            kc[b] = in_vgpr(a.kc[b]);
            kr[b] = in_vgpr(a.kr[b]);
        }
    }
    float gu[RPT][CPT], gv[RPT][CPT], mn[RPT][CPT];
    float zk[RPT + 2][CPT + 2];  // the 3x3 neighbourhoods
    float rmin[2][CPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i)
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            gu[i][c] = 0.f;
            gv[i][c] = 0.f;
            mn[i][c] = kInf;
        }
    // window row ar feeds pixel row i as its filter row ar - i
#pragma unroll
    for (int ar = 0; ar < RPT + 2 * R; ++ar) {
        // one window row at a time: left alone, the scheduler reads them all
        // first and takes 136 registers
        __builtin_amdgcn_sched_barrier(0);
        float zv[S], d[S];
        const auto diff = [&](float z, float sv) {
            return KIND == KIND_DISP ? sv - ref.y : (ref.x - z) * sv;
        };
        if constexpr (CPT == 2) {
#pragma unroll
            for (int b = 0; b < S; b += 2) {
                const float4 t = base[ar * (LW / 2) + b / 2];
                zv[b] = t.x;
                zv[b + 1] = t.z;
                d[b] = diff(t.x, t.y);
                d[b + 1] = diff(t.z, t.w);
            }
        } else {
            const float2 *line = reinterpret_cast<const float2 *>(T) + (top + ar) * LW + lane;
#pragma unroll
            for (int b = 0; b < S; ++b) {
                zv[b] = line[b].x;
                d[b] = diff(line[b].x, line[b].y);
            }
        }
        if (ar >= R - 1 && ar <= R + RPT) {
#pragma unroll
            for (int c = 0; c < CPT + 2; ++c) zk[ar - (R - 1)][c] = zv[R - 1 + c];
        }
        // minima of the row's windows: zv[1..2R] is common to two
        float both = vmin3(zv[1], zv[2], zv[3]);
#pragma unroll
        for (int b = 4; b + 1 <= 2 * R; b += 2)
            if (b + 1 < 2 * R) both = vmin3(both, zv[b], zv[b + 1]);
        rmin[ar & 1][0] = vmin3(both, zv[0], zv[2 * R]);
        if constexpr (CPT == 2) rmin[ar & 1][1] = vmin3(both, zv[2 * R], zv[2 * R + 1]);
        if (ar & 1) {  // two rows at a time into the windows that hold them
#pragma unroll
            for (int i = 0; i < RPT; ++i)
#pragma unroll
                for (int c = 0; c < CPT; ++c) {
                    const bool h0 = ar - 1 >= i && ar - 1 <= i + 2 * R;
                    const bool h1 = ar >= i && ar <= i + 2 * R;
                    if (h0 && h1) mn[i][c] = vmin3(mn[i][c], rmin[0][c], rmin[1][c]);
                    else if (h0) mn[i][c] = vmin(mn[i][c], rmin[0][c]);
                    else if (h1) mn[i][c] = vmin(mn[i][c], rmin[1][c]);
                }
        }
        float hr[CPT], hc[CPT];  // SEP: sum_b kr[b] d[b], sum_b kc[b] d[b]
        if constexpr (SEP) {
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                hr[c] = 0.f;
                hc[c] = 0.f;
#pragma unroll
                for (int b = 0; b < N; ++b) {
                    hr[c] = fmaf(kr[b], d[b + c], hr[c]);
                    hc[c] = fmaf(kc[b], d[b + c], hc[c]);
                }
            }
        }
#pragma unroll
        for (int i = 0; i < RPT; ++i) {
            const int ka = ar - i;
            if (ka < 0 || ka > 2 * R) continue;
#pragma unroll
            for (int c = 0; c < CPT; ++c) {
                if constexpr (SEP) {
                    gu[i][c] = fmaf(kc[ka], hr[c], gu[i][c]);  // K_x row ka = kc[ka] kr
                    gv[i][c] = fmaf(kr[ka], hc[c], gv[i][c]);  // K_y row ka = kr[ka] kc
                } else {
#pragma unroll
                    for (int b = 0; b < N; ++b) {
                        gu[i][c] = fmaf(a.kx[ka * N + b], d[b + c], gu[i][c]);
                        gv[i][c] = fmaf(a.kx[b * N + ka], d[b + c], gv[i][c]);
                    }
                }
            }
        }
    }

    // the sums are finished here: sunk to the pixel that uses them, they would
    // keep every row's partial sums in registers
    Mask ok[RPT][CPT];
#pragma unroll
    for (int i = 0; i < RPT; ++i)
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            asm volatile("" : "+v"(gu[i][c]), "+v"(gv[i][c]));
            ok[i][c] = mask_of(mn[i][c] > 0.f);
        }

    // pair reciprocals (lower or right minus upper or left) between the kept
    // rows, the ones above pixel row i carried over from row i - 1
    float pS[CPT], pSE[CPT + 1], pSW[CPT + 1];
    auto vertical = [&](int u, float (&vS)[CPT], float (&vSE)[CPT + 1], float (&vSW)[CPT + 1]) {
#pragma unroll
        for (int c = 0; c < CPT; ++c) vS[c] = rcp(zk[u + 1][c + 1] - zk[u][c + 1]);
#pragma unroll
        for (int c = 0; c <= CPT; ++c) {
            vSE[c] = rcp(zk[u + 1][c + 1] - zk[u][c]);
            vSW[c] = rcp(zk[u + 1][c] - zk[u][c + 1]);
        }
    };
    vertical(0, pS, pSE, pSW);
#pragma unroll
    for (int i = 0; i < RPT; ++i) {
        const int y = y0 + top + i;
        float rE[CPT + 1], nS[CPT], nSE[CPT + 1], nSW[CPT + 1];
#pragma unroll
        for (int c = 0; c <= CPT; ++c) rE[c] = rcp(zk[i + 1][c + 1] - zk[i + 1][c]);
        vertical(i + 1, nS, nSE, nSW);
        const float fv = (float)y - f.v0;
        Vec<OT, CPT> ox, oy, oz;
        bool mk[CPT];
#pragma unroll
        for (int c = 0; c < CPT; ++c) {
            const float z0 = zk[i + 1][c + 1];
            float Gu, Gv;
            if constexpr (KIND == KIND_DISP) {
                Gu = fmaf(a.ksum, ref.y, gu[i][c]);
                Gv = fmaf(a.ksum, ref.y, gv[i][c]);
            } else {
                Gu = ref.y * (gu[i][c] + a.ksum);
                Gv = ref.y * (gv[i][c] + a.ksum);
            }
            const Mask valid = ok[i][c];
            // slots: E, W, S, N, SE, NW, SW, NE
            const float zj[8] = {zk[i + 1][c + 2], zk[i + 1][c],     zk[i + 2][c + 1],
                                 zk[i][c + 1],     zk[i + 2][c + 2], zk[i][c],
                                 zk[i + 2][c],     zk[i][c + 2]};
            const float rj[8] = {rE[c + 1],   -rE[c],  nS[c],  -pS[c],
                                 nSE[c + 1], -pSE[c], nSW[c], -pSW[c + 1]};
            const float fu = (float)(x + c) - f.u0;
            const float B = fmaf(fu, Gu, fv * Gv);
            bool general = true;
            if constexpr (!kTieHeavy<KIND>) {
                const float rmax = vmax8abs(rE[c + 1], rE[c], nS[c], pS[c], nSE[c + 1], pSE[c],
                                            nSW[c], pSW[c + 1]);
                general = (mask_of(rmax == kInf) & valid) != 0;
            }
            float nz;
            if constexpr (AGG == AGG_MEAN) {
                nz = mean8<KIND>(Gu, Gv, rj, zj, z0, B, general);
            } else {
                const float Spp = Gu + Gv, Spm = Gu - Gv;
                const float Nj[8] = {Gu, -Gu, Gv, -Gv, Spp, -Spp, -Spm, Spm};
                nz = median8<KIND, false>(Nj, rj, zj, z0, B, general);
            }
            const float nx = f.fx * Gu, ny = f.fy * Gv;
            const float n2 = fmaf(nx, nx, fmaf(ny, ny, nz * nz));
            const Mask pos = mask_of(n2 > 0.f);
            const bool keep = ::sne::lane(valid & pos), deg = ::sne::lane(valid & ~pos);
            const float rs = __builtin_amdgcn_rsqf(n2);
            const float inv = keep ? rs : 0.f;
            const float oz1 = mul_or_zero(nz, inv);
            ox.v[c] = Out<OUT>::cvt(neg_mul_or_zero(nx, inv));
            oy.v[c] = Out<OUT>::cvt(neg_mul_or_zero(ny, inv));
            oz.v[c] = Out<OUT>::cvt(deg ? -1.f : oz1);
            mk[c] = ::sne::lane(valid);
        }
#pragma unroll
        for (int c = 0; c < CPT; ++c) pS[c] = nS[c];
#pragma unroll
        for (int c = 0; c <= CPT; ++c) {
            pSE[c] = nSE[c];
            pSW[c] = nSW[c];
        }
        if (x < f.W && y < f.H) {
            SNE_GLOBAL char *o = store_base(f.out);
            const int64_t plane = f.out_plane * (int64_t)sizeof(OT);
            const unsigned off = ((unsigned)y * (unsigned)f.out_pitch + (unsigned)x) * sizeof(OT);
            SNE_GLOBAL char *m =
                store_base(f.mask) + ((unsigned)y * (unsigned)f.mask_pitch + (unsigned)x);
            if (CPT == 2 && x + 1 < f.W) {
                store_stream(o + off, ox);
                store_stream(o + plane + off, oy);
                store_stream(o + 2 * plane + off, oz);
                if (f.mask)
                    store_stream(m, (uint16_t)((mk[0] ? 1 : 0) | (mk[CPT - 1] ? 0x100 : 0)));
            } else {
                store_stream(o + off, ox.v[0]);
                store_stream(o + plane + off, oy.v[0]);
                store_stream(o + 2 * plane + off, oz.v[0]);
                if (f.mask) store_stream(m, (uint8_t)(mk[0] ? 1 : 0));
            }
        }
    }
}

// The batch tables are only read at wave-uniform addresses and do not change
// while the kernel runs (the queue heads apart, which are not read here):
// loads through the constant address space go to scalar registers directly,
// which keeps a frame's buffer resource and constants there (loaded through a
// generic pointer they would count as lane-varying, and each buffer load of
// the tile would become a loop over distinct resources).
template <typename T> __device__ __forceinline__ T uniform_load(const T *p) {
    static_assert(sizeof(T) % 4 == 0, "dword-sized table entries");
    struct Words {
        int w[sizeof(T) / 4];
    };
    typedef const __attribute__((address_space(4))) int CInt;
    CInt *c = (CInt *)p;
    Words v;
#pragma unroll
    for (int i = 0; i < (int)(sizeof(T) / 4); ++i) v.w[i] = c[i];
    return __builtin_bit_cast(T, v);
}

// Frame of a tile: the last f with tile_start[f] <= tile (tile_start is
// strictly increasing, tile_start[0] = 0).  The 64 lanes probe evenly spaced
// frames of the remaining range at once and a ballot keeps the segment that
// holds the tile, so 1024 frames take two dependent loads instead of the ten
// of a binary search.  Called with all lanes active.
__device__ __forceinline__ int find_frame(const int32_t *tile_start, int nframes, int tile) {
    const int lane = threadIdx.x & (kWave - 1);
    int lo = 0, hi = nframes - 1;  // the frame is in [lo, hi]; tile_start[lo] <= tile
    while (lo < hi) {
        const int step = (hi - lo + kWave) / kWave;  // ceil((hi - lo + 1) / 64)
        const int probe = lo + lane * step;
        const int32_t v = ((SNE_GLOBAL const int32_t *)tile_start)[min(probe, hi)];  // in bounds
        const bool le = probe <= hi && v <= tile;
        const uint64_t m = __builtin_amdgcn_ballot_w64(le);  // lanes 0..k, k >= 0
        const int k = 63 - __builtin_clzll(m);
        lo += k * step;
        hi = min(hi, lo + step - 1);
    }
    return lo;
}

// Persistent uneven batch.  A wavefront first takes `chunk` tiles at a time
// from the queue of its block's XCD, then from the other queues in turn,
// until all are drained.  The queues hold contiguous tile ranges, so
// neighbouring tiles (which share halo rows) mostly run on one XCD and meet
// in its L2, and the atomic increments are spread over eight addresses.
template <int KIND, int GK, int AGG, int OUT, int PX, bool HALF, bool LEN>
__global__ __launch_bounds__(kBlock) SNE_BATCH_OCCUPANCY void sne_batch_kernel(BatchArgs a) {
    const int lane = threadIdx.x & (kWave - 1);
    BatchHeader *head = static_cast<BatchHeader *>(a.table);
    const int nframes = uniform_load(&head->nframes);
    const int ntiles = uniform_load(&head->ntiles);
    const BatchTable t = batch_table(a.table, nframes);
    const int home = (int)(blockIdx.x % kQueues);
    for (int i = 0; i < kQueues; ++i) {
        const int q = (home + i) % kQueues;
        const int begin = (int)((int64_t)ntiles * q / kQueues);
        const int end = (int)((int64_t)ntiles * (q + 1) / kQueues);
        // The counters only grow: a queue seen exhausted by a plain load is
        // left without an atomic (a stale smaller value merely costs one),
        // so the waves of a grid larger than the batch leave after a few
        // reads instead of queueing eight atomics each on the same lines.
        int seen = 0;
        if (lane == 0)
            seen = __hip_atomic_load((SNE_GLOBAL int32_t *)&head->queue[q].next, __ATOMIC_RELAXED,
                                     __HIP_MEMORY_SCOPE_AGENT);
        if (__builtin_amdgcn_readfirstlane(seen) >= end - begin) continue;
        for (;;) {
            int taken = 0;
            if (lane == 0)
                taken = __hip_atomic_fetch_add((SNE_GLOBAL int32_t *)&head->queue[q].next, a.chunk,
                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            taken = __builtin_amdgcn_readfirstlane(taken);  // lane 0 is the first active lane
            const int first = begin + min(taken, end - begin);
            if (first >= end) break;
            const int last = min(first + a.chunk, end);
            for (int tile = first; tile < last; ++tile) {
                const int frame =
                    __builtin_amdgcn_readfirstlane(find_frame(t.tile_start, nframes, tile));
                FrameDesc f = uniform_load(t.frames + frame);
                const float4 K = uniform_load(a.ktable + f.k_index);
                f.fx = K.x;
                f.fy = K.y;
                f.u0 = K.z;
                f.v0 = K.w;
                const int local = tile - uniform_load(t.tile_start + frame);
                const int ns = uniform_load(t.nstrips + frame);
                const int band = local / ns;
                const int strip = local - band * ns;
                const int r0 = band * a.rows * (HALF ? 2 : 1);
                run_tile<KIND, GK, AGG, OUT, PX, HALF, LEN>(
                    f, strip * (HALF ? kWave / 2 : kWave) * PX, r0, a.rows, a.gw);
            }
        }
    }
}

template <int KIND, int GK, int AGG, int OUT, bool LEN>
hipError_t uniform_px(int px, const UniformArgs &a, int grid, hipStream_t s) {
    // px: columns per lane, + 100 for the half-wave mode
    switch (px) {
    case 1: hipLaunchKernelGGL((sne_uniform_kernel<KIND, GK, AGG, OUT, 1, false, LEN>), dim3(grid), dim3(kBlock), 0, s, a); break;
    case 2: hipLaunchKernelGGL((sne_uniform_kernel<KIND, GK, AGG, OUT, 2, false, LEN>), dim3(grid), dim3(kBlock), 0, s, a); break;
    case 4: hipLaunchKernelGGL((sne_uniform_kernel<KIND, GK, AGG, OUT, 4, false, LEN>), dim3(grid), dim3(kBlock), 0, s, a); break;
    case 101: hipLaunchKernelGGL((sne_uniform_kernel<KIND, GK, AGG, OUT, 1, true, LEN>), dim3(grid), dim3(kBlock), 0, s, a); break;
    case 102: hipLaunchKernelGGL((sne_uniform_kernel<KIND, GK, AGG, OUT, 2, true, LEN>), dim3(grid), dim3(kBlock), 0, s, a); break;
    case 104: hipLaunchKernelGGL((sne_uniform_kernel<KIND, GK, AGG, OUT, 4, true, LEN>), dim3(grid), dim3(kBlock), 0, s, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int KIND, int GK, int AGG, int OUT, bool LEN>
hipError_t batch_px(int px, const BatchArgs &a, int grid, hipStream_t s) {
    // px: columns per lane, + 100 for the half-wave mode
    switch (px) {
    case 1: hipLaunchKernelGGL((sne_batch_kernel<KIND, GK, AGG, OUT, 1, false, LEN>), dim3(grid), dim3(kBlock), 0, s, a); break;
    case 2: hipLaunchKernelGGL((sne_batch_kernel<KIND, GK, AGG, OUT, 2, false, LEN>), dim3(grid), dim3(kBlock), 0, s, a); break;
    case 4: hipLaunchKernelGGL((sne_batch_kernel<KIND, GK, AGG, OUT, 4, false, LEN>), dim3(grid), dim3(kBlock), 0, s, a); break;
    case 101: hipLaunchKernelGGL((sne_batch_kernel<KIND, GK, AGG, OUT, 1, true, LEN>), dim3(grid), dim3(kBlock), 0, s, a); break;
    case 102: hipLaunchKernelGGL((sne_batch_kernel<KIND, GK, AGG, OUT, 2, true, LEN>), dim3(grid), dim3(kBlock), 0, s, a); break;
    case 104: hipLaunchKernelGGL((sne_batch_kernel<KIND, GK, AGG, OUT, 4, true, LEN>), dim3(grid), dim3(kBlock), 0, s, a); break;
    default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

template <int KIND, int GK, int AGG, int OUT, bool LEN>
hipError_t occupancy_px(int px, int *blocks) {
    const void *f = nullptr;
    switch (px) {
    case 1: f = reinterpret_cast<const void *>(&sne_batch_kernel<KIND, GK, AGG, OUT, 1, false, LEN>); break;
    case 2: f = reinterpret_cast<const void *>(&sne_batch_kernel<KIND, GK, AGG, OUT, 2, false, LEN>); break;
    case 4: f = reinterpret_cast<const void *>(&sne_batch_kernel<KIND, GK, AGG, OUT, 4, false, LEN>); break;
    case 101: f = reinterpret_cast<const void *>(&sne_batch_kernel<KIND, GK, AGG, OUT, 1, true, LEN>); break;
    case 102: f = reinterpret_cast<const void *>(&sne_batch_kernel<KIND, GK, AGG, OUT, 2, true, LEN>); break;
    case 104: f = reinterpret_cast<const void *>(&sne_batch_kernel<KIND, GK, AGG, OUT, 4, true, LEN>); break;
    default: return hipErrorInvalidValue;
    }
    return hipOccupancyMaxActiveBlocksPerMultiprocessor(blocks, f, kBlock, 0);
}

// Dispatch on the runtime variant: filter class, aggregation, output type
// and rule, then the tile's column class.  FN is uniform_px, batch_px or
// occupancy_px; ARGS... are their arguments after px.
#define SNE_DISPATCH_LEN(FN, KIND, GK, AGG, OUT, v, ...)                                   \
    (((v).kind & kLenientFlag) ? FN<KIND, GK, AGG, OUT, true>((v).px, __VA_ARGS__)         \
                              : FN<KIND, GK, AGG, OUT, false>((v).px, __VA_ARGS__))
#define SNE_DISPATCH_OUT(FN, KIND, GK, AGG, v, ...)                                        \
    ((v).out == OUT_F32 ? SNE_DISPATCH_LEN(FN, KIND, GK, AGG, OUT_F32, v, __VA_ARGS__)     \
                        : SNE_DISPATCH_LEN(FN, KIND, GK, AGG, OUT_F16, v, __VA_ARGS__))
#define SNE_DISPATCH_AGG(FN, KIND, GK, v, ...)                                             \
    ((v).agg == AGG_MEAN ? SNE_DISPATCH_OUT(FN, KIND, GK, AGG_MEAN, v, __VA_ARGS__)        \
                         : SNE_DISPATCH_OUT(FN, KIND, GK, AGG_MEDIAN, v, __VA_ARGS__))
#define SNE_DISPATCH(FN, KIND, v, ...)                                                     \
    ((v).grad == 0 ? SNE_DISPATCH_AGG(FN, KIND, GK_FD, v, __VA_ARGS__)                     \
                   : SNE_DISPATCH_AGG(FN, KIND, GK_3ROW, v, __VA_ARGS__))

#define SNE_DISPATCH_RGBN_AGG(FN, KIND, GK, v, ...)                                        \
    ((v).agg == AGG_MEAN ? SNE_DISPATCH_LEN(FN, KIND, GK, AGG_MEAN, OUT_RGBN, v, __VA_ARGS__)  \
                         : SNE_DISPATCH_LEN(FN, KIND, GK, AGG_MEDIAN, OUT_RGBN, v, __VA_ARGS__))

template <int KIND>
hipError_t uniform_variant(const Variant &v, const UniformArgs &a, int grid, hipStream_t s) {
    if (v.out == OUT_RGBN)  // the packed output exists for single frames and uniform batches
        return (v.grad == 0 ? SNE_DISPATCH_RGBN_AGG(uniform_px, KIND, GK_FD, v, a, grid, s)
                            : SNE_DISPATCH_RGBN_AGG(uniform_px, KIND, GK_3ROW, v, a, grid, s));
    if (v.grad == kGradCustom) {  // custom kernels: single frames and uniform batches, strict
        if (v.agg == AGG_MEAN)
            return v.out == OUT_F32
                       ? uniform_px<KIND, GK_CUSTOM, AGG_MEAN, OUT_F32, false>(v.px, a, grid, s)
                       : uniform_px<KIND, GK_CUSTOM, AGG_MEAN, OUT_F16, false>(v.px, a, grid, s);
        return v.out == OUT_F32
                   ? uniform_px<KIND, GK_CUSTOM, AGG_MEDIAN, OUT_F32, false>(v.px, a, grid, s)
                   : uniform_px<KIND, GK_CUSTOM, AGG_MEDIAN, OUT_F16, false>(v.px, a, grid, s);
    }
    return SNE_DISPATCH(uniform_px, KIND, v, a, grid, s);
}
template <int KIND, int R, bool SEP, int CPT>
hipError_t wide_cols(const Variant &v, const WideArgs &a, hipStream_t s) {
    const dim3 grid((unsigned)a.nblocks), block(kBlock);
    if (v.agg == AGG_MEAN) {
        if (v.out == OUT_F32)
            hipLaunchKernelGGL((sne_wide_kernel<KIND, R, AGG_MEAN, OUT_F32, SEP, CPT>), grid,
                               block, 0, s, a);
        else
            hipLaunchKernelGGL((sne_wide_kernel<KIND, R, AGG_MEAN, OUT_F16, SEP, CPT>), grid,
                               block, 0, s, a);
    } else {
        if (v.out == OUT_F32)
            hipLaunchKernelGGL((sne_wide_kernel<KIND, R, AGG_MEDIAN, OUT_F32, SEP, CPT>), grid,
                               block, 0, s, a);
        else
            hipLaunchKernelGGL((sne_wide_kernel<KIND, R, AGG_MEDIAN, OUT_F16, SEP, CPT>), grid,
                               block, 0, s, a);
    }
    return hipGetLastError();
}
template <int KIND, int R, bool SEP>
hipError_t wide_r(const Variant &v, const WideArgs &a, hipStream_t s) {
    return a.cols == 1 ? wide_cols<KIND, R, SEP, 1>(v, a, s) : wide_cols<KIND, R, SEP, 2>(v, a, s);
}
template <int KIND>
hipError_t wide_variant(const Variant &v, const WideArgs &a, hipStream_t s) {
    if (a.R == 2)
        return a.separable ? wide_r<KIND, 2, true>(v, a, s) : wide_r<KIND, 2, false>(v, a, s);
    if (a.R == 3)
        return a.separable ? wide_r<KIND, 3, true>(v, a, s) : wide_r<KIND, 3, false>(v, a, s);
    return hipErrorInvalidValue;
}
template <int KIND>
hipError_t batch_variant(const Variant &v, const BatchArgs &a, int grid, hipStream_t s) {
    return SNE_DISPATCH(batch_px, KIND, v, a, grid, s);
}
template <int KIND> hipError_t occupancy_variant(const Variant &v, int *blocks) {
    return SNE_DISPATCH(occupancy_px, KIND, v, blocks);
}

}  // namespace

#if SNE_KIND == 0
#define SNE_SUFFIX f32
#elif SNE_KIND == 1
#define SNE_SUFFIX u16
#elif SNE_KIND == 2
#define SNE_SUFFIX f16
#else
#define SNE_SUFFIX disp
#endif
#define SNE_CAT2(a, b) a##b
#define SNE_CAT(a, b) SNE_CAT2(a, b)

hipError_t SNE_CAT(launch_uniform_, SNE_SUFFIX)(const Variant &v, const UniformArgs &a, int grid,
                                                hipStream_t s) {
    return uniform_variant<SNE_KIND>(v, a, grid, s);
}

hipError_t SNE_CAT(launch_wide_, SNE_SUFFIX)(const Variant &v, const WideArgs &a, hipStream_t s) {
    return wide_variant<SNE_KIND>(v, a, s);
}

hipError_t SNE_CAT(launch_batch_, SNE_SUFFIX)(const Variant &v, const BatchArgs &a, int grid,
                                              hipStream_t s) {
    return batch_variant<SNE_KIND>(v, a, grid, s);
}

hipError_t SNE_CAT(occupancy_batch_, SNE_SUFFIX)(const Variant &v, int *blocks) {
    return occupancy_variant<SNE_KIND>(v, blocks);
}

}  // namespace sne
