// bs_split_dev.h -- device code of sums of Gauss points over targets on the
// matrix cores at the 16-bit rate, as accurate as the binary32 contraction
// where the scaled values stay in binary16's range (the host decides).
//
// Positions are relative to the centre c of the targets' block and scaled by
// a power of two xs, strengths by ws.  With x' = x - c, p' = p - c, a Gauss
// point's term is s W x (x' - p'), s = |x' - p'|^-3, so
//   v(x) = (sum s W) x x' - sum s (W x p'),
// two contractions:
//   |x' - p'|^2 = |x'|^2 + |p'|^2 - 2 x'.p'
//     on v_mfma_f32_16x16x32_bf16, every binary32 factor written as the sum
//     of three bfloat16 pieces (8 + 8 + 8 bits: exact): first the products
//     with a middle or low piece (seven of the nine of each coordinate; the
//     ninth is below 2^-32 of the term) and the middle and low pieces of
//     |p'|^2 and |x'|^2, then the products of the high pieces on top.  (All in
//     one instruction, which the 32 inner slots would hold, the small
//     products round the result to 1.25 x 2^-24 rms, binary32 FMAs to 0.78;
//     the two-ring velocities' error against FP64 rises from 6.0e-8 to 6.6e-8.)
//   sum s [W, W x p']
//     on v_mfma_f32_16x16x32_f16 over 32 points: s and the six components
//     written as two binary16 pieces each (11 + 11 bits and the second one's
//     sign: 23 bits, binary32 has 24), the 12 component pieces as rows, the
//     two pieces of s one after the other, the smaller first.  The instruction
//     rounds after every eight points, at the magnitude of what it adds to
//     (rms 0.58 units in the last place, unbiased), so the 32 points' sum
//     starts from zero and is added to the running sum in binary32.
// The output lanes of the first product are the operand lanes of the second
// (lane: target l % 16, points 4 (l / 16) + j of two tiles), so s passes
// between them in registers.  Per 1024 pairs the matrix pipe takes 192
// cycles where the binary32 instructions take 384 nominal; a pair costs a
// v_rsq_f32 and five vector instructions, three of them shared by two pairs'
// pieces.
#pragma once

#include "bs_mlp_dev.h" // bf16x8

#include <hip/hip_runtime.h>

namespace bsk {

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

// Upper 16 bits of hi and of lo, as one register (lo in the low half).
__device__ __forceinline__ unsigned pack_hi16(unsigned hi, unsigned lo)
{
    return __builtin_amdgcn_perm(hi, lo, 0x07060302u);
}

// v = h + m + l exactly, each with at most eight significant bits (bfloat16
// values in the upper halves).
__device__ __forceinline__ void bf16_pieces(float v, unsigned &h, unsigned &m, unsigned &l)
{
    h = __float_as_uint(v) & 0xffff0000u;
    const float r = v - __uint_as_float(h);
    m = __float_as_uint(r) & 0xffff0000u;
    l = __float_as_uint(r - __uint_as_float(m));
}

// (a, b) = h + l with binary16 pieces (22 bits).
__device__ __forceinline__ void f16_pieces(float a, float b, f16x2 &h, f16x2 &l)
{
    const f16x2 p = {(_Float16)a, (_Float16)b};
    unsigned u = __builtin_bit_cast(unsigned, p);
    asm("" : "+v"(u)); // (as in split_cubes)
    h = __builtin_bit_cast(f16x2, u);
    float ra = fmaf(a, 1.f, -(float)h.x), rb = fmaf(b, 1.f, -(float)h.y);
    asm("" : "+v"(ra), "+v"(rb));
    l = (f16x2){(_Float16)ra, (_Float16)rb};
}

// Operands of 32 Gauss points (a unit: two tiles of 16) in LDS.
// a1[tile][piece][i]: (x, y, z, |p'|^2) of the piece (high, middle, low) of
// point i; a2[q][row][jj]: component piece `row` of point 16 (jj / 4) + 4 q +
// jj % 4; rows 0-5 the high pieces of [W, W x p'] components (0 1 2 3 then 4
// 5 at 8 9), see split_row.
constexpr int kSplitRows = 12;
struct SplitUnit {
    u32x2 a1[2][3][16];
    _Float16 a2[4][kSplitRows][8];
};

// Stored row of matrix row r: rows 0-3 high pieces of components 0-3, 4-7
// their low pieces, 8 9 high and 12 13 low pieces of components 4 5 (so that
// the high and low sums of a component meet in neighbouring lane groups);
// the other rows are not used and read a stored one.
__device__ __forceinline__ int split_row(int r)
{
    return r < 10 ? r : r == 12 ? 10 : r == 13 ? 11 : 8;
}

// Operands of point i (0 .. 31) of a unit: offset (px, py, pz) from the
// centre, scaled by xs; strength (wx, wy, wz), scaled by ws.  A slot without
// a point passes ok = false (any finite offset): its terms are zero.
__device__ __forceinline__ void split_store(SplitUnit &U, int i, float px, float py, float pz, float wx, float wy,
                                            float wz, bool ok)
{
    float n2 = (px * px + py * py) + pz * pz;
    n2 = ok ? n2 : 1e30f;
    wx = ok ? wx : 0.f;
    wy = ok ? wy : 0.f;
    wz = ok ? wz : 0.f;
    unsigned h[4], m[4], l[4];
    bf16_pieces(px, h[0], m[0], l[0]);
    bf16_pieces(py, h[1], m[1], l[1]);
    bf16_pieces(pz, h[2], m[2], l[2]);
    bf16_pieces(n2, h[3], m[3], l[3]);
    const int tile = i >> 4, r = i & 15;
    U.a1[tile][0][r] = (u32x2){pack_hi16(h[1], h[0]), pack_hi16(h[3], h[2])};
    U.a1[tile][1][r] = (u32x2){pack_hi16(m[1], m[0]), pack_hi16(m[3], m[2])};
    U.a1[tile][2][r] = (u32x2){pack_hi16(l[1], l[0]), pack_hi16(l[3], l[2])};
    const float c[6] = {wx, wy, wz, wy * pz - wz * py, wz * px - wx * pz, wx * py - wy * px};
    _Float16(*o)[8] = U.a2[r >> 2];
    const int jj = 4 * tile + (r & 3);
#pragma unroll
    for (int k = 0; k < 6; k += 2) {
        f16x2 ch, cl;
        f16_pieces(c[k], c[k + 1], ch, cl);
#pragma unroll
        for (int e = 0; e < 2; ++e) {
            o[k < 4 ? k + e : k + 4 + e][jj] = ch[e];
            o[k < 4 ? k + 4 + e : k + 6 + e][jj] = cl[e];
        }
    }
}

// The lane's target operand of the first product: the high pieces' products
// (hi) and all others (lo).
struct SplitTarget {
    bf16x8 lo, hi;
};

// |x' - p'|^2 of four points of a tile and the lane's target (A from
// split_load1).
__device__ __forceinline__ f32x4 split_d2(const bf16x8 &A, const SplitTarget &B)
{
    const f32x4 z = {0.f, 0.f, 0.f, 0.f};
    const f32x4 lo = __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, B.lo, z, 0, 0, 0);
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(A, B.hi, lo, 0, 0, 0);
}

// The lane's operand of the first product for tile `tile` of a unit: inner
// slots 8 q .. 8 q + 7 of point i16.  Lane groups q = 0: high and middle
// pieces; 1: the same with ones in place of |p'|^2; 2: high, low; 3: middle
// (a one in place of |p'|^2), low.  The target operand holds the pieces they
// are multiplied by (split_target); the ones take |x'|^2.
__device__ __forceinline__ bf16x8 split_load1(const SplitUnit &U, int tile, int q, int i16)
{
    const u32x2 a = U.a1[tile][q == 3 ? 1 : 0][i16], b = U.a1[tile][q < 2 ? 1 : 2][i16];
    const unsigned ka = (q & 1) ? 0xffffu : 0xffffffffu, va = (q & 1) ? 0x3f800000u : 0u;
    const unsigned kb = q == 1 ? 0xffffu : 0xffffffffu, vb = q == 1 ? 0x3f800000u : 0u;
    const u32x4 v = {a.x, (a.y & ka) | va, b.x, (b.y & kb) | vb};
    return __builtin_bit_cast(bf16x8, v);
}

__device__ __forceinline__ f16x8 split_load2(const SplitUnit &U, int q, int row)
{
    return *reinterpret_cast<const f16x8 *>(&U.a2[q][row][0]);
}

// The lane's target operand: with t = -2 x' and x2 = |x'|^2 (pieces h, m, l)
// lane group 0 of the products holds (h, 1, h, 1), 1 (m, x2 h, m, x2 m), 2
// (l, 0, h, 1), 3 (l, x2 l, m, 0); the first half of group 0 and x2 h belong
// to the high pieces' instruction.
__device__ __forceinline__ SplitTarget split_target(float x, float y, float z, float x2, int q)
{
    unsigned h[4], m[4], l[4];
    bf16_pieces(-2.f * x, h[0], m[0], l[0]);
    bf16_pieces(-2.f * y, h[1], m[1], l[1]);
    bf16_pieces(-2.f * z, h[2], m[2], l[2]);
    bf16_pieces(x2, h[3], m[3], l[3]);
    const unsigned one = 0x3f800000u;
    unsigned a[4], b[4];
#pragma unroll
    for (int c = 0; c < 3; ++c) {
        a[c] = q == 0 ? 0u : q == 1 ? m[c] : l[c];
        b[c] = (q & 1) ? m[c] : h[c];
    }
    a[3] = q == 3 ? l[3] : 0u;
    b[3] = q == 1 ? m[3] : q == 3 ? 0u : one;
    const u32x4 v = {pack_hi16(a[1], a[0]), pack_hi16(a[3], a[2]), pack_hi16(b[1], b[0]), pack_hi16(b[3], b[2])};
    const u32x4 w = {q == 0 ? pack_hi16(h[1], h[0]) : 0u,
                     q == 0 ? pack_hi16(one, h[2]) : q == 1 ? pack_hi16(h[3], 0u) : 0u, 0u, 0u};
    SplitTarget t;
    t.lo = __builtin_bit_cast(bf16x8, v);
    t.hi = __builtin_bit_cast(bf16x8, w);
    return t;
}

// s = iv^3 of eight pairs as binary16 pieces h + l.
__device__ __forceinline__ void split_cubes(const float (&iv)[8], f16x8 &h, f16x8 &l)
{
    u32x4 hp, lp;
#pragma unroll
    for (int k = 0; k < 4; ++k) {
        const float i0 = iv[2 * k], i1 = iv[2 * k + 1];
        const float q0 = i0 * i0, q1 = i1 * i1;
        // (the empty statements keep the packed pair as the operand of the
        // residuals and the residuals in binary32 until they are packed:
        // v_mul, v_cvt_pk_f16_f32 and v_fma_mix_f32 issue in 3 to 5 cycles;
        // the compiler would merge the conversions into v_fma_mixlo /
        // mixhi_f16, which take 9 to 11)
        f16x2 p = {(_Float16)(i0 * q0), (_Float16)(i1 * q1)};
        unsigned u = __builtin_bit_cast(unsigned, p);
        asm("" : "+v"(u));
        p = __builtin_bit_cast(f16x2, u);
        float r0 = fmaf(i0, q0, -(float)p.x), r1 = fmaf(i1, q1, -(float)p.y);
        asm("" : "+v"(r0), "+v"(r1));
        const f16x2 r = {(_Float16)r0, (_Float16)r1};
        hp[k] = u;
        lp[k] = __builtin_bit_cast(unsigned, r);
    }
    h = __builtin_bit_cast(f16x8, hp);
    l = __builtin_bit_cast(f16x8, lp);
}

// The six sums of four target tiles (D[nt]: matrix rows 4 q + j of target
// l % 16 of tile nt), high and low pieces added, as six registers per lane:
//   y[2 P + j] (j < 2): component j of target tile 2 P + q in lane groups
//     q = 0, 1 and component 4 + j of tile 2 P + q - 2 in groups 2, 3;
//   y[4 + j] (j < 2): component 2 + j of target tile q.
__device__ __forceinline__ void split_gather(const f32x4 *D, float (&y)[6])
{
    float t[2][4];
#pragma unroll
    for (int P = 0; P < 2; ++P)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(D[2 * P][j]),
                                                             __float_as_uint(D[2 * P + 1][j]), false, false);
            t[P][j] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
        }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
        y[j] = t[0][j];
        y[2 + j] = t[1][j];
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(t[0][2 + j]), __float_as_uint(t[1][2 + j]),
                                                         false, false);
        y[4 + j] = __uint_as_float(sw[0]);
    }
}

// Where split_gather leaves component c of target `node` (0 .. 63): register
// and lane.
__device__ __forceinline__ int split_slot(int c, int node, int &lane)
{
    const int nt = node >> 4, i = node & 15, P = nt >> 1, hb = nt & 1;
    lane = c < 2 ? 16 * hb + i : c < 4 ? 16 * nt + i : 32 + 16 * hb + i;
    return c < 2 ? 2 * P + c : c < 4 ? 2 + c : 2 * P + c - 4;
}

} // namespace bsk
