// keyswitch.hip -- LWE key switching N -> n on gfx950 (ArctyrEX Fig. 1,
// final step), plus the fused post-step of a gate level.
//
//   out = (0, .., 0, b') - sum_{j < N} sum_{p < t} ksk[j][p][d_{j,p}]
//   d_{j,p} = ((a'_j + 2^(31 - t*gamma)) >> (32 - (p+1)*gamma)) & (2^gamma-1)
//
// Work split: a workgroup owns KS_GATES ciphertexts and runs KS_JSPLIT
// wavefronts on each, every one summing the rows of a contiguous range of
// j; the partial sums meet in LDS.  The 64 lanes of a wavefront own the n+1
// output columns (NCH chunks of 64), so every gathered key row is read as
// coalesced 256-byte segments.  The digits are wave-uniform: each lane
// loads one a'_j of a 64-wide chunk, the wave broadcasts them one by one
// with readlane, and the digit, row address and loop control stay in scalar
// registers.  Rows of up to KS_PCH levels are fetched before any of them is
// used, so many loads are in flight per wave.  The key-switching key (tens
// of MB) is shared by every wave and stays in L2 / Infinity Cache; the
// ciphertexts of one workgroup walk j in step, so their gathers of the same
// (j, p) rows also share the L1.
//
// For key-switch bases up to 2^4 the sum is computed instead as an int8
// GEMM on v_mfma_i32_32x32x32_i8 (k_ks_mfma): with the one-hot digit matrix
// A[g][(j, p, h)] = (d_{g,j,p} == h) and the key as four signed int8 limbs,
// sum_{j,p} ksk[j][p][d_{g,j,p}][c] = sum_k A[g][k] * ksk[k][c].  The key
// (tens of MB) is then streamed once per 32 RT ciphertexts (RT = 2 or 4) instead
// of being gathered row by row for every ciphertext.
#include "internal.hpp"

#include <algorithm>

namespace cggi {

namespace {

constexpr int KS_GATES = 4;    // ciphertexts per workgroup
constexpr int KS_JSPLIT = 2;   // wavefronts per ciphertext (j ranges)
constexpr int KS_PCH = 4;      // key-switch levels fetched together
constexpr int KS_THREADS = 64 * KS_GATES * KS_JSPLIT;

// Source of the big ciphertext of item `it`:
//   plain batch: src = in + it*(N+1)
//   gate level : gate `it` reads ws_big[slot] (+ ws_big[slot+1] and +1/8
//                on the body for MUX), writes wires[out]
struct KsLevel {
    const cggi_gate_t *gates;
    const int32_t *slot;      // first bootstrap slot of each gate, -1 if none
    const uint32_t *big;      // [2G][N+1]
    uint32_t *wires;          // [W][n+1]
    int W;
};

// Source(s) and destination of item `it`; false if it produces nothing.
template <bool LEVEL>
__device__ __forceinline__ bool ks_item(int it, int B, const uint32_t *in,
                                        uint32_t *out, const KsLevel &lv,
                                        int n, int N, const uint32_t *&src0,
                                        const uint32_t *&src1, uint32_t *&dst)
{
    src0 = src1 = nullptr;
    dst = nullptr;
    if (it >= B)
        return false;
    if (LEVEL) {
        const cggi_gate_t gt = lv.gates[it];
        const int s = lv.slot[it];
        if (s < 0 || gt.out < 0 || gt.out >= lv.W)
            return false;
        src0 = lv.big + (size_t)s * (N + 1);
        if (gt.op == CGGI_MUX)
            src1 = lv.big + (size_t)(s + 1) * (N + 1);
        dst = lv.wires + (size_t)gt.out * (n + 1);
    } else {
        src0 = in + (size_t)it * (N + 1);
        dst = out + (size_t)it * (n + 1);
    }
    return true;
}

template <int NCH, bool LEVEL>
__global__ __launch_bounds__(KS_THREADS) void k_keyswitch(
    const uint32_t *__restrict__ ksk, const uint32_t *__restrict__ in,
    uint32_t *__restrict__ out, int B, KsLevel lv, int n, int N, int gamma,
    int t)
{
    __shared__ uint32_t part[KS_GATES][KS_JSPLIT - 1][64 * NCH];
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int gsub = wave / KS_JSPLIT, jpart = wave % KS_JSPLIT;
    const int it = blockIdx.x * KS_GATES + gsub;
    const uint32_t *src0, *src1;
    uint32_t *dst;
    const bool live = ks_item<LEVEL>(it, B, in, out, lv, n, N, src0, src1, dst);
    const int base = 1 << gamma;
    const uint32_t round_off = (t * gamma < 32) ? 1u << (31 - t * gamma) : 0u;
    const size_t rowlen = (size_t)n + 1;

    uint32_t acc[NCH];
#pragma unroll
    for (int k = 0; k < NCH; ++k)
        acc[k] = 0u;
    if (live) {
        if (jpart == 0) {
            uint32_t body = src0[N];
            if (src1)
                body += src1[N] + (1u << 29);
#pragma unroll
            for (int k = 0; k < NCH; ++k)
                if (lane + 64 * k == n)
                    acc[k] = body;
        }
        const int jlen = N / KS_JSPLIT;
        for (int j0 = jpart * jlen; j0 < (jpart + 1) * jlen; j0 += 64) {
            uint32_t a = src0[j0 + lane];
            if (src1)
                a += src1[j0 + lane];
            a += round_off;
            for (int jj = 0; jj < 64; ++jj) {
                const uint32_t u = __builtin_amdgcn_readlane(a, jj);
                const uint32_t *rows =
                    ksk + (size_t)(j0 + jj) * t * base * rowlen;
                for (int p0 = 0; p0 < t; p0 += KS_PCH) {
                    uint32_t v[KS_PCH][NCH];
#pragma unroll
                    for (int pp = 0; pp < KS_PCH; ++pp) {
                        const int p = p0 + pp;
                        if (p < t) {
                            uint32_t d = (u >> (32 - (p + 1) * gamma)) &
                                         (base - 1);
                            const uint32_t *row =
                                rows + ((size_t)p * base + d) * rowlen;
#pragma unroll
                            for (int k = 0; k < NCH; ++k) {
                                int col = lane + 64 * k;
                                v[pp][k] = col <= n ? row[col] : 0u;
                            }
                        } else {
#pragma unroll
                            for (int k = 0; k < NCH; ++k)
                                v[pp][k] = 0u;
                        }
                    }
#pragma unroll
                    for (int pp = 0; pp < KS_PCH; ++pp)
#pragma unroll
                        for (int k = 0; k < NCH; ++k)
                            acc[k] -= v[pp][k];
                }
            }
        }
    }
    if (jpart > 0) {
#pragma unroll
        for (int k = 0; k < NCH; ++k)
            part[gsub][jpart - 1][lane + 64 * k] = acc[k];
    }
    __syncthreads();
    if (jpart == 0 && live) {
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            int col = lane + 64 * k;
            uint32_t x = acc[k];
            for (int q = 0; q < KS_JSPLIT - 1; ++q)
                x += part[gsub][q][col];
            if (col <= n)
                dst[col] = x;
        }
    }
}

// ---- key switching as an int8 GEMM ----------------------------------------
// K runs over (j, slot), slot = p * 2^gamma + h padded to KSJ * 32 per j, so
// one MFMA K-step of 32 covers one slot block of one j.  Operand layouts of
// v_mfma_i32_32x32x32_i8: lane l holds 16 consecutive k (k = 16 (l >> 5) +
// byte) of row l & 31 (A: ciphertext) or column l & 31 (B: key column).
typedef int ks_v4i __attribute__((ext_vector_type(4)));
typedef int ks_v16i __attribute__((ext_vector_type(16)));

constexpr int KSM_THREADS = 512;   // eight waves

// ksk [N][t][2^gamma][n+1] -> limb blocks [NT][N][KSJ][4][64 lanes][16 B]:
// byte e of lane l in block (nt, j, sj, q) is limb q of
// ksk[j][p][h][32 nt + (l & 31)] for slot 32 sj + 16 (l >> 5) + e = p 2^gamma
// + h, zero where p >= t or the column is past n.  Limbs are signed:
// v = sum_q 2^(8q) v_q with v_q in [-128, 127].  A wave per (nt, j, sj): a lane
// reads its 16 key words once (32 columns side by side) and writes its 16
// bytes of each limb; a thread per dword, which read every word for each limb,
// took 143 us at the default set and 657 us at the large one, this 53 and 182.
__global__ __launch_bounds__(256) void k_ksk_to_i8(
    const uint32_t *__restrict__ ksk, uint32_t *__restrict__ out, int n,
    int N, int t, int gamma, int ksj, int nt_tiles)
{
    const int lane = threadIdx.x & 63;
    const int blk = __builtin_amdgcn_readfirstlane(
        (int)(blockIdx.x * 4 + (threadIdx.x >> 6)));
    if (blk >= nt_tiles * N * ksj)
        return;
    const int base = 1 << gamma;
    const int sj = blk % ksj, j = blk / ksj % N, nt = blk / ksj / N;
    const int col = 32 * nt + (lane & 31), kh = lane >> 5;
    const uint32_t *row = ksk + (size_t)j * t * base * (n + 1) + col;
    uint32_t w[4][4];                // [limb][dword of four slots]
#pragma unroll
    for (int e4 = 0; e4 < 4; ++e4) {
        uint32_t v[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            const int slot = 32 * sj + 16 * kh + 4 * e4 + e;   // p 2^gamma + h
            const bool in = slot < t * base && col <= n;
            // the low three limbs plus 128 are the bytes of v + 0x808080
            v[e] = ((in ? row[(size_t)slot * (n + 1)] : 0u) + 0x808080u) ^
                   0x808080u;
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            w[q][e4] = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                w[q][e4] |= (v[e] >> (8 * q) & 0xFFu) << (8 * e);
        }
    }
    uint4 *dst = reinterpret_cast<uint4 *>(out) + (size_t)blk * 256 + lane;
#pragma unroll
    for (int q = 0; q < 4; ++q)
        dst[q * 64] = make_uint4(w[q][0], w[q][1], w[q][2], w[q][3]);
}

// out rows = (0, .., 0, b'): the GEMM then subtracts into them.
template <bool LEVEL>
__global__ __launch_bounds__(256) void k_ks_init(const uint32_t *__restrict__ in,
                                                 uint32_t *__restrict__ out,
                                                 int B, KsLevel lv, int n, int N)
{
    const size_t total = (size_t)B * (n + 1);
    for (size_t idx = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
         idx < total; idx += (size_t)gridDim.x * blockDim.x) {
        const int it = (int)(idx / (n + 1)), col = (int)(idx % (n + 1));
        const uint32_t *src0, *src1;
        uint32_t *dst;
        if (!ks_item<LEVEL>(it, B, in, out, lv, n, N, src0, src1, dst))
            continue;
        uint32_t v = 0;
        if (col == n) {
            v = src0[N];
            if (src1)
                v += src1[N] + (1u << 29);
        }
        dst[col] = v;
    }
}

// One workgroup of eight waves: 32 RT ciphertexts (RT row tiles) x one range
// of j x 8 UW column units, UW = 8 / RT per wave; a unit is one limb of a
// 32-column tile, so a wave holds RT x UW = 8 accumulators.
//  * The one-hot digits (A) are the same for every column: each thread builds
//    the slots of one (ciphertext, j) of a chunk of 512 / (32 RT) j, and the
//    waves read them from LDS, double-buffered by chunk (one barrier per
//    chunk).
//  * A wave reads its key blocks (B) from L2 PF K-steps ahead, UW KB per
//    eight MFMAs.  With RT = 4 that is 32 bytes a cycle and CU, half the
//    vector cache's rate; 64 ciphertexts with one tile per wave and the
//    digits built by every wave ran at that rate: 185 -> 103 us for 1024
//    default ciphertexts, 2.75 -> 1.13 ms for 16,384 (2.4 POP/s of int8
//    work, near what the matrix cores sustain at the power limit), 0.68 ->
//    0.46 ms for 1024 large ones.
//  * The recombined limb sums are subtracted from the output rows with device
//    atomics (mod 2^32, so the order of the j ranges does not matter); with
//    RT = 4 a tile's two waves add theirs in LDS first.
// KSJ: K-steps per j as a constant (the chunk's loop unrolls and the loads in
// flight can be counted), 0 any number, -1 any number at base 2 (two levels
// per dword of slots).
template <int RT, bool LEVEL, int KSJ>
__global__ __launch_bounds__(KSM_THREADS) void k_ks_mfma(
    const int8_t *__restrict__ kski8, const uint32_t *__restrict__ in,
    uint32_t *__restrict__ out, int B, KsLevel lv, int n, int N, int gamma,
    int t, int ksj_rt, int nt_tiles, int jchunk)
{
    constexpr bool BASE2 = KSJ < 0;
    const int ksj = KSJ > 0 ? KSJ : ksj_rt;
    constexpr int UW = 8 / RT, ROWS = 32 * RT, CJ = KSM_THREADS / ROWS;
    // pad slots per j: the 16 / CJ rows x CJ j that 16 lanes build at once
    // then fall in distinct banks
    constexpr int PADJ = 16 / CJ;
    extern __shared__ __align__(16) unsigned char ks_smem[];
    __shared__ uint32_t *dst_l[ROWS];
    // A: [buffer][chunk j][K-step of j][row tile][kappa half][32 rows][16 B],
    // PADJ slots after each j
    ks_v4i *al = reinterpret_cast<ks_v4i *>(ks_smem);
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int unit = (blockIdx.y * 8 + wave) * UW;
    const int nt = unit >> 2, q0 = unit & 3;
    const int j0 = blockIdx.z * jchunk;
    const int JC = min(N, j0 + jchunk) - j0;      // a multiple of CJ
    const int base = 1 << gamma;
    const uint32_t round_off = (t * gamma < 32) ? 1u << (31 - t * gamma) : 0u;

    // this thread's ciphertext and j of a chunk
    const int row = threadIdx.x / CJ, jj = threadIdx.x % CJ;
    const uint32_t *src0, *src1;
    uint32_t *dst;
    const bool live = ks_item<LEVEL>(blockIdx.x * ROWS + row, B, in, out, lv, n,
                                     N, src0, src1, dst);
    if (jj == 0)
        dst_l[row] = dst;
    // (always loads, from row 0 where there is no ciphertext: a load under a
    // condition would make the wait for it one for every load in flight)
    const bool second = LEVEL && src1;
    if (!live)
        src0 = LEVEL ? lv.big : in;
    if (!second)
        src1 = src0;
    struct Pair {
        uint32_t a, b;
    };
    auto load_u = [&](int c) -> Pair {
        const int j = j0 + min(c * CJ, JC - CJ) + jj;
        return {src0[j], LEVEL ? src1[j] : 0u};
    };
    // the slots of this thread's (ciphertext, j), without branches
    auto build = [&](int buf, Pair uu) {
        const uint32_t u = uu.a + (second ? uu.b : 0u) + round_off;
        ks_v4i *d = al + (buf * CJ + jj) * (ksj * RT * 64 + PADJ) +
                    (row >> 5) * 64 + (row & 31);
        for (int sj = 0; sj < ksj; ++sj) {
#pragma unroll
            for (int kh = 0; kh < 2; ++kh) {
                ks_v4i a;
#pragma unroll
                for (int w = 0; w < 4; ++w) {
                    const int slot0 = 32 * sj + 16 * kh + 4 * w;
                    uint32_t word = 0;
                    if (!BASE2) {
                        const int p = slot0 >> gamma;
                        const uint32_t dg =
                            (u >> ((32 - (p + 1) * gamma) & 31)) &
                            (uint32_t)(base - 1);
                        const uint32_t rel =
                            dg - (uint32_t)(slot0 & (base - 1));
                        word = (rel < 4u ? 1u << (8 * (rel & 3)) : 0u) &
                               (uint32_t)((p - t) >> 31);
                    } else {
#pragma unroll
                        for (int hp = 0; hp < 2; ++hp) {
                            const int p = (slot0 >> 1) + hp;
                            const uint32_t dg = (u >> ((31 - p) & 31)) & 1u;
                            word |= (1u << (8 * (2 * hp + (int)dg))) &
                                    (uint32_t)((p - t) >> 31);
                        }
                    }
                    a[w] = (int)word;
                }
                d[sj * RT * 64 + kh * 32] = a;
            }
        }
    };

    const int S = JC * ksj, SC = CJ * ksj;   // K-steps: all, of a chunk
    const int nchunk = JC / CJ;
    // (waves past the last tile repeat tile 0 and drop it)
    const bool on = nt < nt_tiles;
    const int8_t *bp = kski8 + ((size_t)(on ? nt : 0) * N + j0) * ksj * 4096 +
                       q0 * 1024 + lane * 16;
    auto loadb = [&](int s, ks_v4i (&b)[UW]) {
        // (past the end the last step's blocks, unused)
        const int8_t *p = bp + (size_t)min(s, S - 1) * 4096;
#pragma unroll
        for (int q = 0; q < UW; ++q)
            b[q] = *reinterpret_cast<const ks_v4i *>(p + q * 1024);
    };
    ks_v16i acc[RT][UW];
#pragma unroll
    for (int mt = 0; mt < RT; ++mt)
#pragma unroll
        for (int q = 0; q < UW; ++q)
            acc[mt][q] = ks_v16i{};
    constexpr int PF = RT == 4 ? 4 : 2;      // K-steps of key blocks in flight
    ks_v4i bq[PF][UW];
    build(0, load_u(0));
    Pair u_nxt = load_u(1);
#pragma unroll
    for (int k = 0; k < PF; ++k)
        loadb(k, bq[k]);
    __syncthreads();
    for (int c = 0; c < nchunk; ++c) {
        build((c + 1) & 1, u_nxt);      // (after the last chunk: unused)
        u_nxt = load_u(c + 2);
        // A of the chunk's K-steps, read one ahead
        const ks_v4i *as = al + (c & 1) * CJ * (ksj * RT * 64 + PADJ) + lane;
        int sj = 0;
        ks_v4i av[2][RT];
        auto loada = [&](ks_v4i (&a)[RT]) {
#pragma unroll
            for (int mt = 0; mt < RT; ++mt)
                a[mt] = as[mt * 64];
            as += RT * 64;
            if (++sj == ksj) {
                sj = 0;
                as += PADJ;
            }
        };
        loada(av[0]);
        // SC is a multiple of PF: CJ is
        constexpr int UNROLL = KSJ > 0 ? CJ * KSJ / PF : 1;
#pragma unroll(UNROLL)
        for (int s = 0; s < (KSJ > 0 ? CJ * KSJ : SC); s += PF) {
#pragma unroll
            for (int k = 0; k < PF; ++k) {
                // (past the chunk's end: the next buffer's words, unused)
                loada(av[(k + 1) & 1]);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int mt = 0; mt < RT; ++mt)
#pragma unroll
                    for (int q = 0; q < UW; ++q)
                        acc[mt][q] = __builtin_amdgcn_mfma_i32_32x32x32_i8(
                            av[k & 1][mt], bq[k][q], acc[mt][q], 0, 0, 0);
                loadb(c * SC + s + k + PF, bq[k]);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        __syncthreads();
    }

    // recombine the wave's limbs; with two waves per tile the second hands
    // its sums over
    uint32_t x[RT][16];
#pragma unroll
    for (int mt = 0; mt < RT; ++mt)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            uint32_t y = 0;
#pragma unroll
            for (int q = 0; q < UW; ++q)
                y += (uint32_t)acc[mt][q][v] << (8 * q);
            x[mt][v] = y << (8 * q0);
        }
    if constexpr (UW == 2) {
        uint32_t *part = reinterpret_cast<uint32_t *>(ks_smem) +
                         (wave >> 1) * RT * 16 * 64 + lane;
        if (q0 != 0)
#pragma unroll
            for (int mt = 0; mt < RT; ++mt)
#pragma unroll
                for (int v = 0; v < 16; ++v)
                    part[(mt * 16 + v) * 64] = x[mt][v];
        __syncthreads();
        if (q0 != 0)
            return;
#pragma unroll
        for (int mt = 0; mt < RT; ++mt)
#pragma unroll
            for (int v = 0; v < 16; ++v)
                x[mt][v] += part[(mt * 16 + v) * 64];
    }
    const int col = 32 * nt + (lane & 31), kh = lane >> 5;
    if (!on || col > n)
        return;
#pragma unroll
    for (int mt = 0; mt < RT; ++mt)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
            uint32_t *o = dst_l[32 * mt + 8 * (v >> 2) + 4 * kh + (v & 3)];
            if (o)
                atomicSub(o + col, x[mt][v]);
        }
}

// Dynamic LDS of k_ks_mfma: two chunks of one-hot digits, or the hand-over
// of limb sums.
size_t ks_mfma_smem(int RT, int ksj)
{
    // (and the K-step read past the last chunk's end)
    const size_t a = (size_t)2 * (KSM_THREADS * ksj * 32 + 16 * 16) +
                     (size_t)RT * 64 * 16;
    const size_t h = RT == 4 ? (size_t)4 * RT * 16 * 64 * 4 : 0;
    return a > h ? a : h;
}

template <int RT, bool LEVEL>
int ks_mfma_launch(const Ctx *c, const uint32_t *in, uint32_t *out, int B,
                   KsLevel lv, hipStream_t s)
{
    const Shape &sh = c->sh;
    constexpr int ROWS = 32 * RT;
    const int nt_tiles = (sh.n + 1 + 31) / 32;
    const int ng = (nt_tiles * 4 * RT + 63) / 64;
    const int mg = (B + ROWS - 1) / ROWS;
    // Split j into kc ranges.  The workgroups run in rounds of one per CU,
    // and a workgroup costs about its j range plus 24 j (its start and its
    // atomic fold; 4, 10 and 24 compared over widths: 24 takes 107 us at
    // 1100 default ciphertexts where 10 takes 119, and 1-3% less at 1024
    // large ones, the others are alike), so take the split with the least
    // rounds x (j range + 24), the fewest ranges among equals; ranges are
    // multiples of 16 j (whole chunks).
    int jchunk = sh.N;
    long best = -1;
    for (int jc = sh.N; jc >= 16; jc -= 16) {
        const int kk = (sh.N + jc - 1) / jc;
        const long rounds = ((long)mg * ng * kk + c->cus - 1) / c->cus;
        const long cost = rounds * (jc + 24);
        if (best < 0 || cost < best) {
            best = cost;
            jchunk = jc;
        }
    }
    const int kc = (sh.N + jchunk - 1) / jchunk;
    auto fn = sh.gamma == 1    ? &k_ks_mfma<RT, LEVEL, -1>
              : c->ks_ksj == 1 ? &k_ks_mfma<RT, LEVEL, 1>
              : c->ks_ksj == 2 ? &k_ks_mfma<RT, LEVEL, 2>
                               : &k_ks_mfma<RT, LEVEL, 0>;
    hipLaunchKernelGGL(fn, dim3(mg, ng, kc), dim3(KSM_THREADS),
                       ks_mfma_smem(RT, c->ks_ksj), s, c->ksk_i8, in, out, B,
                       lv, sh.n, sh.N, sh.gamma, sh.t, c->ks_ksj, nt_tiles,
                       jchunk);
    CGGI_HIP_TRY(hipGetLastError());
    return CGGI_OK;
}

template <bool LEVEL>
int ks_mfma_dispatch(const Ctx *c, const uint32_t *in, uint32_t *out, int B,
                     KsLevel lv, hipStream_t s)
{
    const Shape &sh = c->sh;
    const size_t total = (size_t)B * (sh.n + 1);
    const int init_blocks = (int)std::min<size_t>((total + 255) / 256, 65536);
    hipLaunchKernelGGL(k_ks_init<LEVEL>, dim3(init_blocks), dim3(256), 0, s,
                       in, out, B, lv, sh.n, sh.N);
    CGGI_HIP_TRY(hipGetLastError());
    // Four row tiles past 64 ciphertexts, where two would read the key again.
    // From 49 on already where a long j range at few slot blocks per j hides
    // the empty tiles: 64 ciphertexts at n = 630, N = 1024 take 23.8 us in four
    // tiles and 27.8 in two with one block, 34.3 and 37.6 with two, but 77.2
    // and 70.5 with four blocks; at n = 742, N = 2048 38.8 and 42.1 with one,
    // 86.0 and 83.0 with two; at N = 256 14.7 and 11.9 with one.
    const bool four = B > 64 || (B > 48 && sh.N >= 1024 &&
                                 sh.N * c->ks_ksj <= 2048);
    return four ? ks_mfma_launch<4, LEVEL>(c, in, out, B, lv, s)
                : ks_mfma_launch<2, LEVEL>(c, in, out, B, lv, s);
}

template <bool LEVEL>
int ks_dispatch(const Ctx *c, const uint32_t *in, uint32_t *out, int B,
                KsLevel lv, hipStream_t s)
{
    if (c->ksk_i8)
        return ks_mfma_dispatch<LEVEL>(c, in, out, B, lv, s);
    const Shape &sh = c->sh;
    int nch = (sh.n + 1 + 63) / 64;
    dim3 grid((B + KS_GATES - 1) / KS_GATES), block(KS_THREADS);
#define KS_CASE(K)                                                           \
    case K:                                                                  \
        hipLaunchKernelGGL((k_keyswitch<K, LEVEL>), grid, block, 0, s,       \
                           c->ksk, in, out, B, lv, sh.n, sh.N, sh.gamma,     \
                           sh.t);                                            \
        break;
    switch (nch) {
        KS_CASE(1) KS_CASE(2) KS_CASE(3) KS_CASE(4) KS_CASE(5) KS_CASE(6)
        KS_CASE(7) KS_CASE(8) KS_CASE(9) KS_CASE(10) KS_CASE(11) KS_CASE(12)
        KS_CASE(13) KS_CASE(14) KS_CASE(15) KS_CASE(16)
    default:
        return set_error(CGGI_E_PARAM, "key switch: n + 1 > 1024");
    }
#undef KS_CASE
    CGGI_HIP_TRY(hipGetLastError());
    return CGGI_OK;
}

} // namespace

template <int KSJ> static int ks_mfma_attrs()
{
    const void *fn[4] = {
        reinterpret_cast<const void *>(&k_ks_mfma<2, false, KSJ>),
        reinterpret_cast<const void *>(&k_ks_mfma<2, true, KSJ>),
        reinterpret_cast<const void *>(&k_ks_mfma<4, false, KSJ>),
        reinterpret_cast<const void *>(&k_ks_mfma<4, true, KSJ>)};
    for (const void *f : fn)
        CGGI_HIP_TRY(hipFuncSetAttribute(
            f, hipFuncAttributeMaxDynamicSharedMemorySize,
            (int)ks_mfma_smem(4, 4)));
    return CGGI_OK;
}

int keyswitch_make_key(Ctx *c, hipStream_t s)
{
    const Shape &sh = c->sh;
    if (sh.gamma > 4)
        return CGGI_OK;             // large bases keep the row gather
    const int nt_tiles = (sh.n + 1 + 31) / 32;
    const int ksj = (sh.t * (1 << sh.gamma) + 31) / 32;
    const size_t bytes = (size_t)nt_tiles * sh.N * ksj * 4 * 1024;
    if (hipMalloc(&c->ksk_i8, bytes) != hipSuccess) {
        c->ksk_i8 = nullptr;
        return set_error(CGGI_E_NOMEM, "hipMalloc of the int8 key-switching "
                                       "key failed");
    }
    c->ks_ksj = ksj;
    int rc = sh.gamma == 1 ? ks_mfma_attrs<-1>()
             : ksj == 1    ? ks_mfma_attrs<1>()
             : ksj == 2    ? ks_mfma_attrs<2>()
                           : ks_mfma_attrs<0>();
    if (rc)
        return rc;
    hipLaunchKernelGGL(k_ksk_to_i8, dim3((nt_tiles * sh.N * ksj + 3) / 4),
                       dim3(256), 0, s, c->ksk,
                       reinterpret_cast<uint32_t *>(c->ksk_i8), sh.n, sh.N,
                       sh.t, sh.gamma, ksj, nt_tiles);
    CGGI_HIP_TRY(hipGetLastError());
    return CGGI_OK;
}

int keyswitch_launch(const Ctx *c, const uint32_t *in, uint32_t *out, int B,
                     hipStream_t s)
{
    KsLevel lv{};
    return ks_dispatch<false>(c, in, out, B, lv, s);
}

int keyswitch_level(const Ctx *c, const cggi_gate_t *gates,
                    const int32_t *slot, const uint32_t *big,
                    uint32_t *wires, int G, int W, hipStream_t s)
{
    KsLevel lv{gates, slot, big, wires, W};
    return ks_dispatch<true>(c, nullptr, nullptr, G, lv, s);
}

} // namespace cggi
