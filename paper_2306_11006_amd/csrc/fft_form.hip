// fft_form.hip -- the blind rotation with its products by a double-precision
// transform whose rounding is proven exact, on gfx950.
//
// A CMux step (ArctyrEX Fig. 1 loop body) adds sum_r D_r * a_{r,c'} to each
// accumulator component c' in Z_{2^32}[X]/(X^N+1).  Here every product is
// taken in C[X]/(X^M - i), M = N/2: the map a -> sum_{j<M} (a_j + i a_{j+M})
// X^j is a ring isomorphism from R[X]/(X^N+1), and X^M - i splits into M
// linear factors, so a transform of M complex points turns a product into M
// complex multiplications.
//
// Exactness.  Each key coefficient is split into two signed 16-bit halves,
// K = k0 + 2^16 k1 (mod 2^32), with a transform each; the two sums
// sum_r D_r k_{h,r} are integers, recovered by rounding and recombined mod
// 2^32 (k1's sum only matters mod 2^16).  The rounding is right when the
// error of every coefficient is below 1/2.  With u = 2^-53, R = 2l digit
// polynomials of |digit| <= d, |k| <= 2^15 and m = log2 M stages:
//  * a forward butterfly (a + wb by two fused multiply-adds per part, 2a
//    minus that; w rounded to 53 bits) has an error of at most 5u times the
//    2-norm of its outputs, an inverse one (sum, difference times conj(w))
//    4u, so a transform's relative 2-norm error is at most 5mu;
//  * the 2R fused multiply-adds of a pointwise sum add at most 2 sqrt(2) R u
//    sum_r |D_r| |K_r| per point;
//  * ||D_r o K_r||_2 <= max|K_r| ||D_r||_2 <= (sqrt(2) M 2^15)(sqrt(2) M d)
//    (the same product bounds the other order), and the inverse transform
//    divides 2-norms by sqrt(M); a coefficient's error is at most the 2-norm
//    of the error vector.
// Together a coefficient is off by less than
//   E = 2 R M^1.5 d 2^15 (15 m + 2 sqrt(2) R) u:
// 0.005 at the default set (N = 1024, Bg = 2^7, l = 3), 0.08 at the large
// one (N = 2048, Bg = 2^10, l = 2).  A context uses this kernel when E is at
// most 1/4 (fft_error_bound), for any key and any input, so the results are
// the integers of the other kernels, bit for bit.
//
// Work split.  One workgroup per bootstrap.  A step has four phases between
// barriers: (0) every thread rotates, subtracts and takes the digits of its
// coefficients; (1) a wave per digit polynomial (per two at N = 512 and 256;
// two waves at N = 2048) runs a whole forward transform, PPL = 8 points per
// lane (4 at N = 256); (2) a thread per point sums the 2l products for the
// four outputs (component, key half); (3) a wave per output runs the inverse
// transform, rounds and adds into the accumulator.  A wave's transform is
// three register passes with two exchanges through its own row of LDS, which
// need no barrier (N = 256: see quad_forward); rows are padded or swizzled so
// that every 16 lanes of a 16-byte access fall in distinct banks (a
// conflict-free exchange of 8 KB takes 140 cycles, three quarters of it the
// write; an unswizzled one 360).
//
// What bounds it: at N = 1024 a step takes 8,300 cycles for one bootstrap and
// 15,300 for two.  The VALU issues 3,798 wave instructions of it per bootstrap
// (3,100 are the transforms' and sums' f64 work, 4.4 to 5.1 cycles each on a
// SIMD), the LDS is active 3,460 cycles, and the key's 192 KB come through the
// CU's vector cache at 64 bytes a cycle behind them; since the waves leave a
// barrier together and run the same phase, VALU and LDS time mostly add up.
// Default set (n = 630, l = 3): 2.2 ms for one bootstrap and 2.7 for 256,
// against 2.8 to 8.5 ms for the int8 kernels and 10.3 for the modular
// transform; 8.0 ms for 1024, against 17.9 and 31.6.  Large set (n = 742,
// N = 2048, l = 2): 4.0 ms for one, 32.5 ms for 2000.
#include "internal.hpp"

#include <cmath>
#include <type_traits>
#include <vector>

namespace cggi {

namespace {

typedef double d2 __attribute__((ext_vector_type(2)));

// A transform of M = N/2 points is H transforms of MS points, one per wave:
// at N = 2048 (H = 2) those of the even and the odd coefficients, E and O,
// both at the roots Y of Y^MS = i, which the pointwise phase combines into
// the points E(X^2) +- X O(X^2) as it reads them (and splits its sums the
// same way).  Index bits of an MS-point transform, from the top: a (RB bits,
// the registers of pass 1), b (RB bits, pass 2), c (LAST bits, the stages of
// pass 3, whose registers are b's low BS bits and c).
template <int N> struct FCfg {
    static constexpr int M = N / 2;
    static constexpr int H = N == 2048 ? 2 : 1;
    static constexpr int MS = M / H;
    static constexpr int LOGM = __builtin_ctz(MS);
    static constexpr bool QUAD = N == 256;       // (see quad_forward)
    static constexpr int RB = QUAD ? 2 : 3;
    static constexpr int PPL = 1 << RB;          // points per lane
    static constexpr int LPF = MS / PPL;         // lanes per transform
    static constexpr int FPW = 64 / LPF;         // transforms per wave
    static constexpr int LAST = LOGM - 2 * RB;
    static constexpr int BS = RB - LAST;
    static constexpr int NTW = 1 << (RB - 1);    // twiddles per lane and pass
    // bootstrap workgroup: a thread per point of an MS-point transform
    static constexpr int THREADS = MS, WAVES = MS / 64;
    static constexpr int TW2 = NTW, TW3 = NTW + PPL * NTW; // table offsets
    static constexpr int TWX = TW3 + LPF * NTW;  // H = 2: [MS] values X
    static constexpr int TW4 = TW3 + 16 * NTW;   // QUAD: [LPF]
    static constexpr bool PAD = !QUAD && LAST == 3; // padded rows (see fslot)
    // slots of an LDS row
    static constexpr int ROW = QUAD ? MS + 8 : PAD ? MS + MS / 8 : MS;
    // a lane's transform among its wave's, and its place in it
    static __device__ __forceinline__ int tf(int lane)
    {
        return QUAD ? lane >> 3 & 1 : lane / LPF;
    }
    static __device__ __forceinline__ int tlane(int lane)
    {
        return QUAD ? lane >> 4 << 3 | (lane & 7) : lane % LPF;
    }
};

// Slot of index (a, b, c) in a transform's exchange row, such that every 16
// lanes of a 16-byte access fall in distinct banks.  For 512 points one pad
// slot per 8 does that and leaves each access one lane base plus an
// immediate; the shorter transforms swizzle.
template <int N> __device__ __forceinline__ int fslot(int a, int b, int c)
{
    using C = FCfg<N>;
    if constexpr (C::PAD)
        return a * 72 + b * 9 + c;
    constexpr int AM = (1 << (4 - C::LAST)) - 1;
    return (a << (C::RB + C::LAST)) | ((b ^ (a & AM)) << C::LAST) |
           (c ^ (b >> C::BS));
}

// Order memory operations of one wave's lanes on LDS (they complete in
// order; this only keeps the compiler from moving them).
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

__device__ __forceinline__ void fft_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// (a, b) -> (a + wb, a - wb), w times i when ROT.
template <bool ROT>
__device__ __forceinline__ void bf_fwd(d2 &a, d2 &b, d2 w)
{
    d2 p;
    if (!ROT) {
        p.x = fma(-w.y, b.y, fma(w.x, b.x, a.x));
        p.y = fma(w.y, b.x, fma(w.x, b.y, a.y));
    } else {
        p.x = fma(-w.y, b.x, fma(-w.x, b.y, a.x));
        p.y = fma(-w.y, b.y, fma(w.x, b.x, a.y));
    }
    b.x = fma(2.0, a.x, -p.x);
    b.y = fma(2.0, a.y, -p.y);
    a = p;
}

// (a, b) -> (a + b, (a - b) conj(w)), w times i when ROT.
template <bool ROT>
__device__ __forceinline__ void bf_inv(d2 &a, d2 &b, d2 w)
{
    const d2 d = {a.x - b.x, a.y - b.y};
    a.x += b.x;
    a.y += b.y;
    const double re = fma(d.x, w.x, d.y * w.y);
    const double im = fma(d.y, w.x, -(d.x * w.y));
    if (!ROT) {
        b.x = re;
        b.y = im;
    } else {
        b.x = im;
        b.y = -re;
    }
}

// NS stages over the low NS bits of the register index (the bits above them
// select independent blocks with their own twiddles).  The node of a block
// after bits beta_0.. has the twiddle of its first 2^(t-1) siblings times
// i^beta_(t-1), so stage t of a block reads tw[(1 << t) / 2 + ..] only.
template <int PPL, int NS, bool INV>
__device__ __forceinline__ void reg_stages(d2 (&v)[PPL], const d2 *tw)
{
    constexpr int BLK = 1 << NS, PER = BLK / 2;   // twiddles per block
#pragma unroll
    for (int blk = 0; blk < PPL / BLK; ++blk)
#pragma unroll
        for (int tt = 0; tt < NS; ++tt) {
            const int t = INV ? NS - 1 - tt : tt;
            const int half = BLK >> (t + 1);      // distance of a butterfly
            const d2 *wt = tw + blk * PER + (t == 0 ? 0 : (1 << (t - 1)));
#pragma unroll
            for (int g = 0; g < (1 << t); ++g) {  // bits beta_0 .. beta_(t-1)
                // beta_0 is g's top bit; siblings in order of beta_0 + 2
                // beta_1 + .. over the first t - 1 bits
                int rev = 0;
                for (int q = 0; q + 1 < t; ++q)
                    rev |= ((g >> (t - 1 - q)) & 1) << q;
                const bool rot = t > 0 && (g & 1);
#pragma unroll
                for (int k = 0; k < half; ++k) {
                    d2 &x = v[blk * BLK + g * 2 * half + k];
                    d2 &y = v[blk * BLK + g * 2 * half + k + half];
                    if (INV) {
                        if (rot)
                            bf_inv<true>(x, y, wt[rev]);
                        else
                            bf_inv<false>(x, y, wt[rev]);
                    } else {
                        if (rot)
                            bf_fwd<true>(x, y, wt[rev]);
                        else
                            bf_fwd<false>(x, y, wt[rev]);
                    }
                }
            }
        }
}

// The inverse's last pass: the stages of the root (X^(2^NS) = i after the
// deeper ones), whose twiddles are the same in every lane.  A difference is
// turned by 1 - i tan instead of cos - i sin, two operations a butterfly less
// (six), and the cosines are left to the caller's next multiplication
// (root_scale); two halves that meet carry the same one or, at the last
// stage's odd positions, a ratio of cosines for the multiply-add to take in.
// A stage's error is at most 3u of its outputs' 2-norm, u each from the
// difference, the tangent or ratio and the result, and the few u of
// root_scale fit in what the bound above grants beyond that.
template <int NS> __device__ __forceinline__ void root_stages(d2 (&v)[1 << NS])
{
    constexpr double TAN16 = 0.19891236737965800691;    // tan(pi/16)
    constexpr double TAN516 = 1.4966057626654890177;    // tan(5 pi/16)
    constexpr double TAN8 = 0.41421356237309504882;     // tan(pi/8)
    constexpr double RATIO = 0.56645449735052153656;  // cos(5 pi/16)/cos(pi/16)
    auto turn = [](d2 &x, d2 &y, double t, bool rot) {
        const d2 d = {x.x - y.x, x.y - y.y};
        x += y;
        const d2 r = {fma(t, d.y, d.x), fma(-t, d.x, d.y)};
        y = rot ? d2{r.y, -r.x} : r;
    };
    if constexpr (NS == 3)
#pragma unroll
        for (int g = 0; g < 4; ++g)
            turn(v[2 * g], v[2 * g + 1], g >> 1 ? TAN516 : TAN16, g & 1);
    constexpr int Q = 1 << (NS - 2);
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int k = 0; k < Q; ++k)
            turn(v[2 * Q * g + k], v[2 * Q * g + Q + k], TAN8, g);
#pragma unroll
    for (int k = 0; k < 2 * Q; ++k) {
        d2 &x = v[k], &y = v[k + 2 * Q];
        const double rho = NS == 3 && (k & 1) ? RATIO : 1.0;
        const d2 d = {fma(-rho, y.x, x.x), fma(-rho, y.y, x.y)};
        x = {fma(rho, y.x, x.x), fma(rho, y.y, x.y)};
        y = {d.x + d.y, d.y - d.x};
    }
}

// The factor root_stages leaves out of register k.
template <int NS> constexpr double root_scale(int k)
{
    constexpr double COS16 = 0.98078528040323044913;    // cos(pi/16)
    constexpr double COS8 = 0.92387953251128675613;     // cos(pi/8)
    constexpr double COS4 = 0.70710678118654752440;     // cos(pi/4)
    return (NS == 3 && (k & 1) ? COS16 : 1.0) *
           (k >> (NS - 2) & 1 ? COS8 : 1.0) * (k >> (NS - 1) & 1 ? COS4 : 1.0);
}

// A lane's twiddles: pass 1 (the same for every lane), 2 and 3.
template <int N> struct Tw {
    d2 w1[FCfg<N>::NTW], w2[FCfg<N>::NTW], w3[FCfg<N>::NTW];
    d2 w4;                          // QUAD
    __device__ __forceinline__ void load(const double *__restrict__ t, int lf)
    {
        using C = FCfg<N>;
        const d2 *t2 = reinterpret_cast<const d2 *>(t);
#pragma unroll
        for (int k = 0; k < C::NTW; ++k) {
            w1[k] = t2[k];
            w2[k] = t2[C::TW2 + (lf >> C::LAST) * C::NTW + k];
            w3[k] = t2[C::TW3 + (C::QUAD ? lf & 15 : lf) * C::NTW + k];
        }
        if constexpr (C::QUAD) {
            w4 = t2[C::TW4 + lf];
            asm volatile("" : "+v"(w4.x), "+v"(w4.y));
        }
        // arrived before any loop: a use inside one would otherwise wait for
        // every load the loop has in flight
#pragma unroll
        for (int k = 0; k < C::NTW; ++k) {
            asm volatile("" : "+v"(w2[k].x), "+v"(w2[k].y));
            asm volatile("" : "+v"(w3[k].x), "+v"(w3[k].y));
        }
    }
};

// Swap the points' register bits 1 and 0 with lane bits 5 (W32) and 4 (W16).
template <bool W32, bool W16>
__device__ __forceinline__ void swap_lanes(d2 (&v)[4])
{
    typedef uint32_t u4 __attribute__((ext_vector_type(4)));
    u4 w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k)
        w[k] = __builtin_bit_cast(u4, v[k]);
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        if constexpr (W32)
#pragma unroll
            for (int k = 0; k < 2; ++k) {
                const auto r = __builtin_amdgcn_permlane32_swap(
                    w[k][d], w[k + 2][d], false, false);
                w[k][d] = r[0];
                w[k + 2][d] = r[1];
            }
        if constexpr (W16)
#pragma unroll
            for (int k = 0; k < 4; k += 2) {
                const auto r = __builtin_amdgcn_permlane16_swap(
                    w[k][d], w[k + 1][d], false, false);
                w[k][d] = r[0];
                w[k + 1][d] = r[1];
            }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k)
        v[k] = __builtin_bit_cast(d2, w[k]);
}

// The transforms of N = 256, 128 points on 32 lanes of four.  Index bits n6
// .. n0 become result bits b0 .. b6, the top one first: registers n6 n5,
// lane bits 5 4 2 1 0 n4 .. n0 (bit 3 is the transform); two stages, n4 n3
// swapped into the registers, two stages, an exchange through LDS that
// leaves n2 n1 in the registers, n0 on lane bit 5 and b0 .. b3 on bits 4 2 1
// 0, two stages, n0 swapped in, one stage.  The 8-point lanes of the longer
// transforms would leave one busy wave per phase, whose chain of f64
// instructions (5 cycles each for a lone wave) and exchanges was most of a
// step: 0.278 -> 0.213 ms for 128 steps of one bootstrap (l = 2), 2.79 ->
// 2.35 ms for 8192.  Slot of (b0 .. b3, n2 n1 n0) in
// the exchange row: 8 consecutive lanes fall in distinct banks of one half
// for either side, and the wave's other row (an odd multiple of 8 slots
// away) in the other half.
__device__ __forceinline__ int qslot(int b, int n)
{
    return b << 3 | (n ^ (b & 7));
}

template <class F>
__device__ __forceinline__ void quad_forward(d2 (&v)[4], d2 *row, int lf,
                                             const Tw<256> &tw, F mid)
{
    reg_stages<4, 2, false>(v, tw.w1);
    swap_lanes<true, true>(v);
    mid(0);
    reg_stages<4, 2, false>(v, tw.w2);
    wave_sync();
#pragma unroll
    for (int k = 0; k < 4; ++k)
        row[qslot(lf >> 3 << 2 | k, lf & 7)] = v[k];
    mid(1);
    wave_sync();
#pragma unroll
    for (int k = 0; k < 4; ++k)
        v[k] = row[qslot(lf & 15, k << 1 | lf >> 4)];
    reg_stages<4, 2, false>(v, tw.w3);
    swap_lanes<true, false>(v);
    bf_fwd<false>(v[0], v[2], tw.w4);
    bf_fwd<true>(v[1], v[3], tw.w4);
    wave_sync();
}

template <class F>
__device__ __forceinline__ void quad_inverse(d2 (&v)[4], d2 *row, int lf,
                                             const Tw<256> &tw, F mid)
{
    bf_inv<false>(v[0], v[2], tw.w4);
    bf_inv<true>(v[1], v[3], tw.w4);
    swap_lanes<true, false>(v);
    reg_stages<4, 2, true>(v, tw.w3);
    wave_sync();
#pragma unroll
    for (int k = 0; k < 4; ++k)
        row[qslot(lf & 15, k << 1 | lf >> 4)] = v[k];
    mid(0);
    wave_sync();
#pragma unroll
    for (int k = 0; k < 4; ++k)
        v[k] = row[qslot(lf >> 3 << 2 | k, lf & 7)];
    reg_stages<4, 2, true>(v, tw.w2);
    mid(1);
    swap_lanes<true, true>(v);
    root_stages<2>(v);
    wave_sync();
}

// Forward transform of the lane's points v (register index a, lane (b, c)),
// through the transform's own LDS row; on return the registers are pass 3's
// (b's low bits, c) on lane (a, b's high bits).
// mid(0) and mid(1) run after the writes of the two exchanges.
template <int N, class F>
__device__ __forceinline__ void fft_forward(d2 (&v)[FCfg<N>::PPL], d2 *row,
                                            int lf, const Tw<N> &tw, F mid)
{
    using C = FCfg<N>;
    if constexpr (C::QUAD) {
        quad_forward(v, row, lf, tw, mid);
        return;
    } else {
    constexpr int CM = (1 << C::LAST) - 1, LM = (1 << C::BS) - 1;
    reg_stages<C::PPL, C::RB, false>(v, tw.w1);
    wave_sync();
#pragma unroll
    for (int k = 0; k < C::PPL; ++k)
        row[fslot<N>(k, lf >> C::LAST, lf & CM)] = v[k];
    mid(0);
    wave_sync();
#pragma unroll
    for (int k = 0; k < C::PPL; ++k)
        v[k] = row[fslot<N>(lf >> C::LAST, k, lf & CM)];
    reg_stages<C::PPL, C::RB, false>(v, tw.w2);
    wave_sync();
#pragma unroll
    for (int k = 0; k < C::PPL; ++k)
        row[fslot<N>(lf >> C::LAST, k, lf & CM)] = v[k];
    mid(1);
    wave_sync();
#pragma unroll
    for (int k = 0; k < C::PPL; ++k)
        v[k] = row[fslot<N>(lf >> C::LAST,
                            ((lf & CM) << C::BS) | ((k >> C::LAST) & LM),
                            k & CM)];
    reg_stages<C::PPL, C::LAST, false>(v, tw.w3);
    wave_sync();
    }
}

// The inverse of fft_forward, unscaled; ROOT: but for root_scale.
template <int N, bool ROOT, class F>
__device__ __forceinline__ void fft_inverse(d2 (&v)[FCfg<N>::PPL], d2 *row,
                                            int lf, const Tw<N> &tw, F mid)
{
    using C = FCfg<N>;
    if constexpr (C::QUAD) {
        quad_inverse(v, row, lf, tw, mid);
        return;
    } else {
    constexpr int CM = (1 << C::LAST) - 1, LM = (1 << C::BS) - 1;
    reg_stages<C::PPL, C::LAST, true>(v, tw.w3);
    wave_sync();
#pragma unroll
    for (int k = 0; k < C::PPL; ++k)
        row[fslot<N>(lf >> C::LAST,
                     ((lf & CM) << C::BS) | ((k >> C::LAST) & LM), k & CM)] =
            v[k];
    mid(0);
    wave_sync();
#pragma unroll
    for (int k = 0; k < C::PPL; ++k)
        v[k] = row[fslot<N>(lf >> C::LAST, k, lf & CM)];
    reg_stages<C::PPL, C::RB, true>(v, tw.w2);
    wave_sync();
#pragma unroll
    for (int k = 0; k < C::PPL; ++k)
        row[fslot<N>(lf >> C::LAST, k, lf & CM)] = v[k];
    mid(1);
    wave_sync();
#pragma unroll
    for (int k = 0; k < C::PPL; ++k)
        v[k] = row[fslot<N>(k, lf >> C::LAST, lf & CM)];
    if constexpr (ROOT)
        root_stages<C::RB>(v);
    else
        reg_stages<C::PPL, C::RB, true>(v, tw.w1);
    wave_sync();
    }
}

// bsk [n][2l][2][N] -> transforms [n][2l][4][M] of the key halves times 1/M
// (a power of two: exact), output o = 2 c' + h; points [H][MS] as a
// transform leaves them: register k of lane f at k LPF + f; for H = 2 first
// the MS values at X, then those at -X.  One wave per workgroup, FPW
// polynomials each.
template <int N>
__global__ __launch_bounds__(64) void k_fft_key(
    const uint32_t *__restrict__ bsk, const double *__restrict__ tab,
    double *__restrict__ out, int npoly)
{
    using C = FCfg<N>;
    constexpr int H = C::H;
    __shared__ __align__(16) double rows[C::FPW * C::ROW * 2];
    const int lane = threadIdx.x, lf = C::tlane(lane), f = C::tf(lane);
    Tw<N> tw;
    tw.load(tab, lf);
    // polynomial index (i * 2l + r) * 4 + o
    const int p = min((int)blockIdx.x * C::FPW + f, npoly - 1);
    const int h = p & 1;
    const uint32_t *src = bsk + (size_t)(p >> 1) * N;
    auto half = [&](uint32_t x) -> double {
        const int lo = (int16_t)(x & 0xFFFFu);
        return h ? (double)(int16_t)((x - (uint32_t)lo) >> 16) : (double)lo;
    };
    d2 v[H][C::PPL];
    d2 *row = reinterpret_cast<d2 *>(rows) + f * C::ROW;
#pragma unroll
    for (int q = 0; q < H; ++q) {
#pragma unroll
        for (int k = 0; k < C::PPL; ++k) {
            const int j = H * (k * C::LPF + lf) + q;
            v[q][k].x = half(src[j]);
            v[q][k].y = half(src[j + C::M]);
        }
        fft_forward<N>(v[q], row, lf, tw, [](int) {});
    }
    d2 *dst = reinterpret_cast<d2 *>(out) + (size_t)p * C::M;
#pragma unroll
    for (int k = 0; k < C::PPL; ++k) {
        const double s = 1.0 / C::M;
        const int j = k * C::LPF + lf;
        if constexpr (H == 2)
            bf_fwd<false>(v[0][k], v[H - 1][k],
                          reinterpret_cast<const d2 *>(tab)[C::TWX + j]);
#pragma unroll
        for (int q = 0; q < H; ++q)
            dst[q * C::MS + j] = d2{v[q][k].x * s, v[q][k].y * s};
    }
}

__device__ __forceinline__ uint32_t fft_modswitch(uint32_t u, int log2_2n)
{
    return (u + (1u << (31 - log2_2n))) >> (32 - log2_2n);
}

// LDS: rows [max(2l, 4)][H][ROW] complex, accumulator [2][N] (H = 2: the even
// coefficients of a component, then its odd ones).
template <int N> size_t fft_smem_n(int l)
{
    const int rows = 2 * l > 4 ? 2 * l : 4;
    return (size_t)rows * FCfg<N>::H * FCfg<N>::ROW * 16 + (size_t)2 * N * 4;
}

size_t fft_smem(int N, int l)
{
    return N == 256    ? fft_smem_n<256>(l)
           : N == 512  ? fft_smem_n<512>(l)
           : N == 1024 ? fft_smem_n<1024>(l)
                       : fft_smem_n<2048>(l);
}

// The bootstraps [*from, *to) a launch of NB per workgroup takes of a batch
// of `count`.  pair_width > 0: the batch is split between a launch of two
// per workgroup, which takes whole rounds of pair_width and a last one of
// more than half, and a launch of one per workgroup for the rest.
__device__ __forceinline__ void fft_share(int NB, int count, int pair_width,
                                          int *from, int *to)
{
    *from = 0;
    *to = count;
    if (pair_width > 0) {
        const int rest = count % pair_width;
        const int cut = 2 * rest > pair_width ? count : count - rest;
        *(NB == 2 ? to : from) = cut;
    }
}

// NB: bootstraps per workgroup (they share the key values).  L (gadget
// levels) is a compile-time constant for the sets in use, 0 reads it at run
// time.  A thread reads the key values of its slot (H points) KR digit rows
// at a time, a batch ahead of their use (the first batch before the
// barrier); KR = 2L holds the whole column, read during the transforms.  (L =
// 0 that read each row where it is used waited for every one: 200 steps of
// 1024 bootstraps at N = 512, l = 4 took 4.12 ms, 2.02 a row ahead; the int8
// kernels 2.98.)
// WPE: waves per SIMD the registers are budgeted for.
template <int N, int NB, int L, int KR, int WPE>
__global__ __launch_bounds__(FCfg<N>::THREADS)
__attribute__((amdgpu_waves_per_eu(WPE)))
void k_bootstrap_fft(
    const double *__restrict__ key, const double *__restrict__ tab,
    const uint32_t *__restrict__ in, const uint32_t *__restrict__ testv,
    uint32_t *__restrict__ out, int B, const int32_t *__restrict__ d_count,
    int pair_width, int n, int beta, int l_rt)
{
    using C = FCfg<N>;
    constexpr int M = C::M, PPL = C::PPL, LPF = C::LPF, FPW = C::FPW;
    constexpr int ROW = C::ROW, H = C::H, MS = C::MS;
    constexpr int T = C::THREADS;
    constexpr int LOG2_2N = __builtin_ctz(2 * N);
    // The inverse's last pass by root_stages where its chain of instructions
    // is what a step waits for: one bootstrap of the default set 2.22 -> 2.17
    // ms, 256 of them 2.67 -> 2.62, 512 toy ones 0.293 -> 0.286.  With two
    // transforms per SIMD in the inverse phase it gains nothing (4096: 31.8 ->
    // 32.1 ms) or loses (one bootstrap at N = 2048: 3.94 -> 4.11 ms).
    constexpr bool ROOT = H == 1 && NB == 1;
    const int l = L ? L : l_rt;
    const int R = 2 * l;
    const int RB = (R > 4 ? R : 4) * H;          // rows of a bootstrap
    extern __shared__ __align__(16) unsigned char smem[];
    d2 *rows = reinterpret_cast<d2 *>(smem);     // [NB][RB][ROW]
    uint32_t *acc = reinterpret_cast<uint32_t *>(rows + NB * RB * ROW);
    // accumulator word of coefficient t of a component
    auto aidx = [](int t) { return H == 2 ? (t & 1) * M + (t >> 1) : t; };

    const int count = d_count ? min(B, *d_count) : B;
    int from, to;
    fft_share(NB, count, pair_width, &from, &to);
    const int g0 = from + blockIdx.x * NB;
    if (g0 >= to)
        return;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lf = C::tlane(lane), f = C::tf(lane);
    // (a last workgroup with fewer than NB bootstraps repeats its last one)
    const uint32_t *ct[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
        ct[b] = in + (size_t)min(g0 + b, to - 1) * (n + 1);

    // ACC = (0, X^(2N - b~) * v)
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        const int e = (2 * N - (int)fft_modswitch(ct[b][n], LOG2_2N)) &
                      (2 * N - 1);
#pragma unroll
        for (int q = 0; q < N / T; ++q) {
            const int m = tid + q * T;
            uint32_t v = testv ? testv[m] : (1u << 29);
            int t = m + e;
            if (t >= 2 * N) {
                t -= 2 * N;
            } else if (t >= N) {
                t -= N;
                v = 0u - v;
            }
            acc[2 * N * b + aidx(t)] = 0u;
            acc[2 * N * b + N + aidx(t)] = v;
        }
    }
    Tw<N> tw;
    tw.load(tab, lf);

    const uint32_t round_off = (beta * l < 32) ? (1u << (31 - beta * l)) : 0u;
    // the digits' rounding offset, and their top bits: with those flipped a
    // signed bit-field extract gives the digit in [-Bg/2, Bg/2)
    uint32_t dig_off = round_off, dig_flip = 0;
    for (int p = 1; p <= l; ++p) {
        dig_off += (1u << (beta - 1)) << (32 - p * beta);
        dig_flip |= (1u << (beta - 1)) << (32 - p * beta);
    }
    // X of this thread's slot (H = 2)
    d2 xs = {0.0, 0.0};
    if constexpr (H == 2) {
        xs = reinterpret_cast<const d2 *>(tab)[C::TWX + tid];
        asm volatile("" : "+v"(xs.x), "+v"(xs.y));
    }
    // key values in flight: batch bt covers rows KR bt .. of the slot
    constexpr bool AHEAD = L > 0 && KR == 2 * L;
    constexpr int NBT = L ? 2 * L / KR : 1;
    constexpr int KB = AHEAD ? 1 : 2, KL = KR * 4 * H;
    d2 kb[KB][KL];
    const d2 *key2 = reinterpret_cast<const d2 *>(key);
    auto key_issue = [&](int i, int bt, d2 (&dst)[KL], int q0, int q1) {
        // buffer loads: the row's offset is scalar and the lane's offset the
        // same for every row, so a load takes no vector address arithmetic
        const __amdgpu_buffer_rsrc_t rsrc = __builtin_amdgcn_make_buffer_rsrc(
            const_cast<d2 *>(key2 + (size_t)i * R * 4 * M), 0, R * 4 * M * 16,
            0x00020000);
#pragma unroll
        for (int q = q0; q < q1; ++q)
            dst[q] = __builtin_bit_cast(
                d2, __builtin_amdgcn_raw_buffer_load_b128(
                        rsrc, tid * 16, (bt * KL + q) * MS * 16, 0));
        __builtin_amdgcn_sched_barrier(0);
    };
    // forward transforms run on the last waves, inverse ones on the first
    const int nf = NB * R * H, ni = NB * 4 * H;
    const int fw = wave - (C::WAVES * FPW > nf ? C::WAVES - (nf + FPW - 1) / FPW
                                               : 0);

    // The step loop, over the steps with a nonzero rotation (X^0 ACC - ACC
    // = 0 decomposes to all-zero digits).  AHEAD has one copy per role so
    // that each reads its keys at fixed places: waves without a forward
    // transform (role 1) in phase (1), those without an inverse one (role 3)
    // a step ahead in phase (3), those with both between forward passes
    // (role 2; with eight waves of both, role 4, half of them between the
    // previous step's inverse passes, or the vector cache's 64 bytes a cycle
    // would hold up phase (1)).
    auto steps = [&](auto role_c) {
    constexpr int ROLE = decltype(role_c)::value;   // 0: any wave
    uint32_t ev[NB] = {};           // rotations of 64 steps, one per lane
    unsigned long long live = 0;    // those still to come, nonzero ones
    int i0 = -64;                   // first step of the 64
    auto next = [&]() -> int {
        while (!live) {
            i0 += 64;
            if (i0 >= n)
                return n;
            uint32_t any = 0;
#pragma unroll
            for (int b = 0; b < NB; ++b) {
                ev[b] = fft_modswitch(ct[b][min(i0 + lane, n)], LOG2_2N);
                any |= ev[b];
            }
            live = __ballot(any != 0 && i0 + lane < n);
        }
        const int b = __builtin_ctzll(live);
        live &= live - 1;
        return i0 + b;
    };
    int i = next();
    if constexpr (ROLE >= 3)
        if (i < n)
            key_issue(i, 0, kb[0], 0, ROLE == 3 ? KL : KL / 2);
    while (i < n) {
        int e[NB];
#pragma unroll
        for (int b = 0; b < NB; ++b)
            e[b] = __builtin_amdgcn_readlane(ev[b], i & 63);
        const int i_nxt = next();
        fft_barrier();   // ACC of the previous step complete
        // (0) digits of X^e ACC - ACC: those of coefficients j and j + M of
        // polynomial r side by side in dword j / H of row (r, j mod H),
        // whose transform's wave alone reads them
        {
            constexpr int ITEMS = NB * 2 * H;
            uint32_t x[ITEMS][2], y[ITEMS][2];
            // item it: bootstrap and component it / H, coefficients j, j + M
            auto coef = [&](int it) { return H * tid + it % H; };
#pragma unroll
            for (int it = 0; it < ITEMS; ++it)
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const int t = coef(it) + q * M;
                    const uint32_t *ac = acc + it / H * N;
                    x[it][q] = ac[aidx((t - e[it / (2 * H)]) & (N - 1))];
                    y[it][q] = ac[aidx(t)];
                }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int it = 0; it < ITEMS; ++it) {
                const int b = it / (2 * H), c = it / H % 2;
                uint32_t w[2];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    // all ones where the rotated index wrapped (bit N)
                    const uint32_t mk = (uint32_t)__builtin_amdgcn_sbfe(
                        coef(it) + q * M - e[b], LOG2_2N - 1, 1);
                    w[q] = ((x[it][q] ^ mk) + (dig_off - y[it][q] - mk)) ^
                           dig_flip;
                }
                uint32_t *dr =
                    reinterpret_cast<uint32_t *>(
                        rows + (b * RB + c * l * H + it % H) * ROW) + tid;
#pragma unroll
                for (int p = 0; p < (L ? L : l); ++p) {
                    const int sh = 32 - (p + 1) * beta;
                    const uint32_t d0 = __builtin_amdgcn_sbfe(w[0], sh, beta);
                    const uint32_t d1 = __builtin_amdgcn_sbfe(w[1], sh, beta);
                    dr[p * H * ROW * 4] =
                        __builtin_amdgcn_perm(d1, d0, 0x05040100);
                }
            }
        }
        fft_barrier();
        // (1) their transforms
        if constexpr (ROLE == 1)
            key_issue(i, 0, kb[0], 0, KL);
        auto forward = [&](int t0, auto mid) {
            // surplus lanes repeat the last polynomial's work (the same
            // stores of the same values)
            const int pol = FPW == 1 ? t0 : min(t0 + f, nf - 1);
            const int rh = R * H;
            d2 *row = rows + (NB == 1 ? pol : pol / rh * RB + pol % rh) * ROW;
            const uint32_t *dr = reinterpret_cast<const uint32_t *>(row) + lf;
            uint32_t dg[PPL];
#pragma unroll
            for (int k = 0; k < PPL; ++k)
                dg[k] = dr[k * LPF];
            d2 v[PPL];
#pragma unroll
            for (int k = 0; k < PPL; ++k) {
                v[k].x = (double)(int16_t)dg[k];
                v[k].y = (double)((int32_t)dg[k] >> 16);
            }
            fft_forward<N>(v, row, lf, tw, mid);
#pragma unroll
            for (int k = 0; k < PPL; ++k)
                row[k * LPF + lf] = v[k];
        };
        if constexpr (ROLE == 2 || ROLE == 4) {
            forward(fw, [&](int m) {
                key_issue(i, 0, kb[0],
                          ROLE == 2 ? m * KL / 2 : (m + 2) * KL / 4,
                          ROLE == 2 ? (m + 1) * KL / 2 : (m + 3) * KL / 4);
            });
            for (int t0 = fw + C::WAVES; t0 < nf; t0 += C::WAVES)
                forward(t0, [](int) {});
        } else if constexpr (ROLE == 3) {
            forward(fw, [](int) {});
        } else if constexpr (ROLE == 0) {
            for (int t0 = fw * FPW; t0 >= 0 && t0 < nf; t0 += C::WAVES * FPW)
                forward(t0, [](int) {});
        }
        if constexpr (!AHEAD)
            key_issue(i, 0, kb[0], 0, KL);
        fft_barrier();
        // (2) the four outputs' sums over the digit polynomials, in place
        // (a thread reads its point of every row before it writes it)
        auto mac = [](d2 &s, d2 x, d2 k) {
            s.x = fma(x.x, k.x, fma(-x.y, k.y, s.x));
            s.y = fma(x.x, k.y, fma(x.y, k.x, s.y));
        };
        // a row's points in the thread's slot
        auto points = [&](int row, d2 (&x)[H]) {
#pragma unroll
            for (int q = 0; q < H; ++q)
                x[q] = rows[(row + q) * ROW + tid];
            if constexpr (H == 2)
                bf_fwd<false>(x[0], x[H - 1], xs);
        };
        d2 s[NB][4][H] = {};
        if constexpr (L > 0) {
#pragma unroll
            for (int bt = 0; bt < NBT; ++bt) {
                if (bt + 1 < NBT)
                    key_issue(i, bt + 1, kb[(bt + 1) % KB], 0, KL);
#pragma unroll
                for (int rr = 0; rr < KR; ++rr)
#pragma unroll
                    for (int b = 0; b < NB; ++b) {
                        d2 x[H];
                        points(b * RB + (bt * KR + rr) * H, x);
#pragma unroll
                        for (int o = 0; o < 4; ++o)
#pragma unroll
                            for (int q = 0; q < H; ++q)
                                mac(s[b][o][q], x[q],
                                    kb[bt % KB][(rr * 4 + o) * H + q]);
                    }
            }
        } else {
            // R is even
            auto sum_row = [&](int r, const d2 (&k)[KL]) {
#pragma unroll
                for (int b = 0; b < NB; ++b) {
                    d2 x[H];
                    points(b * RB + r * H, x);
#pragma unroll
                    for (int o = 0; o < 4; ++o)
#pragma unroll
                        for (int q = 0; q < H; ++q)
                            mac(s[b][o][q], x[q], k[o * H + q]);
                }
            };
            int r = 0;
            for (; r + 2 < R; r += 2) {
                key_issue(i, r + 1, kb[1], 0, KL);
                sum_row(r, kb[0]);
                key_issue(i, r + 2, kb[0], 0, KL);
                sum_row(r + 1, kb[1]);
            }
            key_issue(i, r + 1, kb[1], 0, KL);
            sum_row(r, kb[0]);
            sum_row(r + 1, kb[1]);
        }
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int o = 0; o < 4; ++o) {
                if constexpr (H == 2)
                    bf_inv<false>(s[b][o][0], s[b][o][H - 1], xs);
#pragma unroll
                for (int q = 0; q < H; ++q)
                    rows[(b * RB + o * H + q) * ROW + tid] = s[b][o][q];
            }
        fft_barrier();
        // (3) inverse transforms; the sums are integers below 2^51, so
        // adding 1.5 * 2^52 leaves them rounded in the low mantissa bits
        if constexpr (ROLE == 3)
            key_issue(min(i_nxt, n - 1), 0, kb[0], 0, KL);
        for (int t0 = wave * FPW; ROLE != 3 && t0 < ni;
             t0 += C::WAVES * FPW) {
            // bootstrap, output, parity
            const int boq = FPW == 1 ? t0 : t0 + f;
            if (FPW > 1 && boq >= ni)
                break;
            const int b = NB == 1 ? 0 : boq / (4 * H), oq = boq - b * 4 * H;
            d2 *row = rows + (b * RB + oq) * ROW;
            d2 v[PPL];
#pragma unroll
            for (int k = 0; k < PPL; ++k)
                v[k] = row[k * LPF + lf];
            fft_inverse<N, ROOT>(v, row, lf, tw, [&](int m) {
                if constexpr (ROLE == 4)
                    key_issue(min(i_nxt, n - 1), 0, kb[0], m * KL / 4,
                              (m + 1) * KL / 4);
            });
            const int o = oq / H;
            uint32_t *ao = acc + (2 * b + (o >> 1)) * N + oq % H * M + lf;
            const int hs = 16 * (o & 1);
#pragma unroll
            for (int k = 0; k < PPL; ++k) {
                const double magic = 6755399441055744.0;
                const double sc = ROOT ? root_scale<C::RB>(k) : 1.0;
                const uint32_t re =
                    (uint32_t)__double_as_longlong(fma(v[k].x, sc, magic)) << hs;
                const uint32_t im =
                    (uint32_t)__double_as_longlong(fma(v[k].y, sc, magic)) << hs;
                __hip_atomic_fetch_add(ao + k * LPF, re, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
                __hip_atomic_fetch_add(ao + k * LPF + MS, im, __ATOMIC_RELAXED,
                                       __HIP_MEMORY_SCOPE_WORKGROUP);
            }
            if (ROLE)
                t0 = ni;
        }
        i = i_nxt;
    }
    };
    if constexpr (AHEAD) {
        if constexpr (NB * 2 * L * H >= C::WAVES && NB * 4 * H >= C::WAVES)
            steps(std::integral_constant<int, 4>{});
        else if (fw < 0)
            steps(std::integral_constant<int, 1>{});
        else if (wave < ni)
            steps(std::integral_constant<int, 2>{});
        else
            steps(std::integral_constant<int, 3>{});
    } else {
        steps(std::integral_constant<int, 0>{});
    }
    __syncthreads();

    // sample extraction of coefficient 0
#pragma unroll
    for (int b = 0; b < NB; ++b) {
        if (g0 + b >= to)
            break;
        uint32_t *o = out + (size_t)(g0 + b) * (N + 1);
        const uint32_t *ac = acc + 2 * N * b;
        for (int j = tid; j <= N; j += T) {
            uint32_t v;
            if (j == 0)
                v = ac[0];
            else if (j < N)
                v = 0u - ac[aidx(N - j)];
            else
                v = ac[N];
            o[j] = v;
        }
    }
}

// Twiddle table: for a pass that starts at stage s in the node of prefix rho
// (the earlier bits, first bit lowest), stage t's distinct twiddles
// exp(i pi (phi / 2^t + sum_q beta_q 2^(q - t))), phi = (1/4 + rho) / 2^s,
// over the bits beta_0 .. beta_(t-2) (the next bit multiplies by i).
void push_twiddles(std::vector<double> &t, unsigned rho, int s, int ns)
{
    const long double pi = acosl(-1.0L);
    const long double phi = (0.25L + rho) / (long double)(1u << s);
    for (int st = 0; st < ns; ++st) {
        const int cnt = st < 2 ? 1 : 1 << (st - 1);
        for (int b = 0; b < cnt; ++b) {
            const long double x =
                pi * (phi + (long double)b) / (long double)(1 << st);
            t.push_back((double)cosl(x));
            t.push_back((double)sinl(x));
        }
    }
}

unsigned rev_bits(unsigned x, int bits)
{
    unsigned r = 0;
    for (int i = 0; i < bits; ++i)
        r |= ((x >> i) & 1u) << (bits - 1 - i);
    return r;
}

template <int N> std::vector<double> fft_table()
{
    using C = FCfg<N>;
    std::vector<double> t;
    push_twiddles(t, 0, 0, C::RB);
    for (int a = 0; a < C::PPL; ++a)
        push_twiddles(t, rev_bits(a, C::RB), C::RB, C::RB);
    if constexpr (C::QUAD) {
        for (int b = 0; b < 16; ++b)
            push_twiddles(t, rev_bits(b, 4), 4, 2);
        for (int f = 0; f < C::LPF; ++f)   // b0 .. b4, b5 = 0
            push_twiddles(t, rev_bits((f & 15) << 2 | f >> 4 << 1, 6), 6, 1);
    } else {
        for (int f = 0; f < C::LPF; ++f)
            for (int bl = 0; bl < (1 << C::BS); ++bl) {
                // prefix (a, b), b = (lane's low bits, bl)
                const unsigned pre = ((unsigned)f << C::BS) | (unsigned)bl;
                push_twiddles(t, rev_bits(pre, 2 * C::RB), 2 * C::RB, C::LAST);
            }
    }
    if (C::H == 2)
        for (int j = 0; j < C::MS; ++j) {
            // the root of register j / LPF of lane j mod LPF
            const unsigned pre = (unsigned)(j % C::LPF * C::PPL + j / C::LPF);
            push_twiddles(t, rev_bits(pre, C::LOGM), C::LOGM, 1);
        }
    return t;
}

// Rows of a key batch (L > 0): the whole column at N = 1024, and at N = 2048
// where it fits the registers; two rows elsewhere.  Two waves per SIMD: 256
// registers.
template <int N> constexpr int FKR(int L)
{
    return N == 1024 || (N == 2048 && L == 2) ? 2 * L : 2;
}
constexpr int FWPE = 2;

// Two bootstraps per workgroup (N = 1024, l = 2 or 3, LDS permitting).
template <int N> constexpr bool FPAIR(int L) { return N == 1024 && L > 0; }

template <int N, int NB, int L, int KR> int fft_attr1()
{
    CGGI_HIP_TRY(hipFuncSetAttribute(
        reinterpret_cast<const void *>(&k_bootstrap_fft<N, NB, L, KR, FWPE>),
        hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024));
    return CGGI_OK;
}

template <int N, int L> int fft_attr()
{
    constexpr int KR = L ? FKR<N>(L) : 1;
    int rc = fft_attr1<N, 1, L, KR>();
    if constexpr (FPAIR<N>(L))
        if (!rc)
            rc = fft_attr1<N, 2, L, KR>();
    return rc;
}

template <int N> int fft_key_t(Ctx *c, const uint32_t *bsk, hipStream_t s)
{
    using C = FCfg<N>;
    const Shape &sh = c->sh;
    // made once; the upload below reads it after this function has returned
    static const std::vector<double> host_tab = fft_table<N>();
    const int npoly = sh.n * 2 * sh.l * 4;
    const size_t words = (size_t)npoly * C::M * 2;
    const size_t tab = host_tab.size() * sizeof(double);
    if (hipMalloc(&c->bsk_fft, words * sizeof(double) + tab) != hipSuccess) {
        // the context then serves its forms with their own kernels
        (void)hipGetLastError();
        c->bsk_fft = nullptr;
        return CGGI_OK;
    }
    c->fft_tw = c->bsk_fft + words;
    CGGI_HIP_TRY(hipMemcpyAsync(c->fft_tw, host_tab.data(), tab,
                                hipMemcpyHostToDevice, s));
    hipLaunchKernelGGL(k_fft_key<N>, dim3((npoly + C::FPW - 1) / C::FPW),
                       dim3(64), 0, s, bsk, c->fft_tw, c->bsk_fft, npoly);
    CGGI_HIP_TRY(hipGetLastError());
    return sh.l == 3   ? fft_attr<N, 3>()
           : sh.l == 2 ? fft_attr<N, 2>()
                       : fft_attr<N, 0>();
}

template <int N, int L>
int fft_launch_l(const Ctx *c, const uint32_t *in, const uint32_t *testv,
                 uint32_t *out, int B, const int32_t *d_count, hipStream_t s)
{
    const Shape &sh = c->sh;
    constexpr int KR = L ? FKR<N>(L) : 1;
    const size_t smem = fft_smem(N, sh.l);
    int pair_width = 0, grid = B;
    if constexpr (FPAIR<N>(L)) {
        // Batches wider than the chip: two bootstraps per workgroup in
        // rounds of twice the CUs, one per workgroup for a rest of at most
        // half a round (and for every narrower batch: a step of two takes
        // 1.8 times a step of one).  A count read on the device is split
        // there, so both are launched; the one with no share exits at once.
        pair_width = 2 * c->cus;
        grid = B < c->cus ? B : c->cus;
        const int rest = B % pair_width;
        const bool pairs = B > c->cus;
        const bool ones = d_count || (rest && rest <= c->cus);
        if (pairs) {
            hipLaunchKernelGGL((k_bootstrap_fft<N, 2, L, KR, FWPE>),
                               dim3((B + 1) / 2), dim3(FCfg<N>::THREADS),
                               2 * smem, s, c->bsk_fft, c->fft_tw, in, testv,
                               out, B, d_count, pair_width, sh.n, sh.beta,
                               sh.l);
            CGGI_HIP_TRY(hipGetLastError());
        }
        if (!ones)
            return CGGI_OK;
    }
    hipLaunchKernelGGL((k_bootstrap_fft<N, 1, L, KR, FWPE>), dim3(grid),
                       dim3(FCfg<N>::THREADS), smem, s, c->bsk_fft,
                       c->fft_tw, in, testv, out, B, d_count, pair_width, sh.n,
                       sh.beta, sh.l);
    CGGI_HIP_TRY(hipGetLastError());
    return CGGI_OK;
}

template <int N>
int fft_launch(const Ctx *c, const uint32_t *in, const uint32_t *testv,
               uint32_t *out, int B, const int32_t *d_count, hipStream_t s)
{
    return c->sh.l == 3
               ? fft_launch_l<N, 3>(c, in, testv, out, B, d_count, s)
           : c->sh.l == 2
               ? fft_launch_l<N, 2>(c, in, testv, out, B, d_count, s)
               : fft_launch_l<N, 0>(c, in, testv, out, B, d_count, s);
}

} // namespace

double fft_error_bound(const Shape &sh)
{
    const double M = sh.N / 2, m = sh.log2N - 1, R = 2.0 * sh.l;
    return 2.0 * R * M * std::sqrt(M) * std::ldexp(1.0, sh.beta - 1) *
           32768.0 * (15.0 * m + 2.0 * std::sqrt(2.0) * R) *
           std::ldexp(1.0, -53);
}

// Widest INT8 batch on this kernel.  At Bg up to 2^7 an int8 GEMM has one
// digit row per level, and at the small rings its throughput kernels match or
// beat the transforms once they fill the chip.  64 steps, int8 against this
// kernel: N = 256, l = 3: 0.388 and 0.301 ms for 1500 bootstraps, 0.413 and
// 0.464 for 2048, 2.50 and 2.83 for 16384; l = 1: 0.202 and 0.155 for 512,
// 0.146 and 0.170 for 1024; N = 512, l = 3: 0.855 and 0.786 for 1500, 0.992
// and 1.030 for 2048; l = 1: 0.246 and 0.172 for 256, 0.313 and 0.382 for
// 1024.  With two digit rows per level (Bg past 2^7), more levels at N = 512
// or a larger ring, this kernel is the faster one at every width.
int fft_int8_width(const Shape &sh, int cus)
{
    if (sh.S != 1 || sh.N > 512 || (sh.N == 512 && sh.l > 3))
        return INT32_MAX;
    return sh.l > 1 ? 6 * cus : sh.N == 512 ? cus : 2 * cus;
}

int fft_make_key(Ctx *c, const uint32_t *bsk, hipStream_t s)
{
    if (fft_error_bound(c->sh) > 0.25 || c->sh.beta > 16 ||
        fft_smem(c->sh.N, c->sh.l) > 160 * 1024)
        return CGGI_OK;                  // not available at these parameters
    switch (c->sh.N) {
    case 256: return fft_key_t<256>(c, bsk, s);
    case 512: return fft_key_t<512>(c, bsk, s);
    case 1024: return fft_key_t<1024>(c, bsk, s);
    default: return fft_key_t<2048>(c, bsk, s);
    }
}

int fft_bootstrap(const Ctx *c, const uint32_t *in, const uint32_t *testv,
                  uint32_t *out, int B, const int32_t *d_count, hipStream_t s)
{
    switch (c->sh.N) {
    case 256: return fft_launch<256>(c, in, testv, out, B, d_count, s);
    case 512: return fft_launch<512>(c, in, testv, out, B, d_count, s);
    case 1024: return fft_launch<1024>(c, in, testv, out, B, d_count, s);
    default: return fft_launch<2048>(c, in, testv, out, B, d_count, s);
    }
}

} // namespace cggi
