// SSD forward in fp32 arithmetic for any (P, N) within the library limits, on v_mfma_f32_32x32x2_f32
// (paper, background section on SSD: matrix work inside chunks, a linear recurrence between chunks;
// Theorem 1: the mixed streams feed one plain SSM).  fp32 io, and bf16 io at the sizes the bf16 MFMA
// kernels do not take.
//
// The result does not depend on the chunk length, so the kernels walk their own steps of 64 tokens:
// the work inside a step grows with its length, the states between steps never leave registers.
//   mix_ops_kernel    (batch, step, group): routes 64 tokens, mixes their B and C rows in fp32 and
//                     writes them, and the masked products G = C B^T, in the register layout of the
//                     operands the chain reads.  Shared by the heads of the group.
//   chain_f32_kernel  (batch, segment, head, 32 channels): walks the steps of a segment with the state in
//                     accumulator registers.  A wave owns 32 of the N state columns; its accumulator rows
//                     n = 8a + 4kg + b of channel p are at the same time the B operand of the readout
//                     contraction, so the state passes through neither LDS nor memory.
//                       Y[i][p]   = sum_n (exp(cs_i) C[i][n]) S[n][p]  +  sum_{j<=i} M[i][j] x[j][p]
//                       S[n][p]  <- exp(cs_last) S[n][p] + sum_j B[j][n] (dt_j exp(cs_last - cs_j) x[j][p])
//                       M[i][j]   = G[i][j] dt_j exp(cs_i - cs_j)
//                     The readout is split over the state columns, the 12 blocks of M over the waves, and
//                     the four partial Y tiles are added in a fixed order: 76 MFMAs per wave and step
//                     (N = 128) whatever the wave.  Where a tile has several waves (N <= 64) each keeps a part of the sum
//                     over j of S (SPLIT).
// Where batch x heads x slices alone would leave compute units idle, a sequence is walked as several
// segments: one launch sums each segment's own contribution to the state (state part only), and a
// segment of the output launch starts from the sum of those in front of it (the recurrence is linear
// in the state).
//
// Bound: no single unit.  On the 130M-shaped layer (two sequences of 2048 tokens: operands 12 us, contributions 30, output
// 66, 101 for the call) the f32 matrix pipe, 64 cycles an MFMA, is busy 44 % of the output launch and 39 % of the other
// by the counters; the rest is the waits between the dependent phases of a step and its two barriers, with two
// workgroups on a compute unit.
#include "common.hpp"
#include "mfma_util.hpp"

#include <atomic>
#include <type_traits>

namespace swimba {

constexpr int CF_STEP = 64;            // tokens per step
constexpr int CF_MIX_THREADS = 512;
constexpr int CF_XS = CF_STEP + 4;     // row stride of the transposed x tile (floats)
constexpr int CF_YS = 36;              // row stride of the partial Y tiles (floats)
constexpr int CF_GBLK = 12;            // 4-column blocks of the masked 64 x 64 product: 4 of tile row 0, 8 of tile row 1

typedef float __attribute__((ext_vector_type(4))) cf_f32x4_t;

__device__ __forceinline__ f32x16_t mfma_f32(float a, float b, f32x16_t c)
{
    return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// four consecutive elements as fp32
__device__ __forceinline__ float4 load4(const float *p) { return *reinterpret_cast<const float4 *>(p); }
__device__ __forceinline__ float4 load4(const bf16 *p)
{
    const uint2 u = *reinterpret_cast<const uint2 *>(p);
    return make_float4(bf_lo(u.x), bf_hi(u.x), bf_lo(u.y), bf_hi(u.y));
}

// Operand arrays, per (batch, step, group), N padded to NT tiles of 32 columns.  IT, QN and GB are 2, 8 and 12, and
// less for sequences of at most 32 tokens, which the chain walks by one tile row: 16 tokens take 8 KB a group, not 28.
//   cop (IT, NT, 4, 64, 4) [I][nt][a][lane][b] = C[32 I + lane%32][32 nt + 8a + 4(lane/32) + b]
//   bop (NT, QN, 64, 4)    [nt][q][lane][b]    = B[8q + 4(lane/32) + b][32 nt + lane%32]
//   gop (GB, 64, 4)        [blk][lane][b]      = (j <= i) C[i] . B[j], blk < 4: i = lane%32, q = blk, else i = 32 + lane%32,
//                          q = blk - 4; j = 8q + 4(lane/32) + b
// Of a step that is not full the rows of C and G without a token are not written: they meet no other row.
struct ChainOps {
    int IT, QN, GB;
};
__host__ __device__ inline ChainOps chain_ops(int L)
{
    const int q = (L + 7) / 8;
    return L > 32 ? ChainOps{2, 8, CF_GBLK} : ChainOps{1, q, q};
}

// PARTS = 4: four workgroups share a step, each with 16 of its tokens as rows of C and of G; it mixes the B rows
// that these meet, so B is read 2.5 times, by compute units that would have none of the steps.
// gpb groups per workgroup: its tokens are routed once for all of them.  QF: quads of a lane in flight, four where two
// workgroups share a compute unit, eight where one has it to itself.
template <typename T, int PARTS, int QF>
__global__ void __launch_bounds__(CF_MIX_THREADS, QF == 4 ? 4 : 2)
mix_ops_kernel(const T *__restrict__ Be, const T *__restrict__ Ce, const T *__restrict__ logits,
               int32_t *__restrict__ idx_out, float *__restrict__ w_out, const float *__restrict__ w_sel,
               float *__restrict__ cop, float *__restrict__ bop, float *__restrict__ gop, Shape s, int NT, int gpb)
{
    extern __shared__ __align__(16) unsigned char smem_raw[];
    const int K = s.K, NP = 32 * NT, RS = NP + 4;        // row stride of the mixed rows
    int32_t *s_idx = reinterpret_cast<int32_t *>(smem_raw);                 // [64][K]
    float *s_w = reinterpret_cast<float *>(s_idx + CF_STEP * K);             // [64][K]
    float *s_B = s_w + CF_STEP * K;                                          // [64][RS]
    float *s_C = s_B + CF_STEP * RS;                                         // [64][RS]
    constexpr int R = CF_STEP / PARTS;                   // rows of C and G in this workgroup
    const int part = blockIdx.x % PARTS, r0 = part * R, item = blockIdx.x / PARTS, gblocks = s.G / gpb;
    const int g_begin = (item % gblocks) * gpb;
    const int c = (item / gblocks) % s.nc;
    const int b = item / (gblocks * s.nc);
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int valid = min(CF_STEP, s.L - c * CF_STEP);
    const bool one_row = s.L <= 32;                      // of tiles (chain_ops)
    if (one_row && r0 >= valid) return;
    const int64_t tok0 = (int64_t)b * s.L + (int64_t)c * CF_STEP;
    const bool sel = (w_sel != nullptr);
    const ChainOps ops = chain_ops(s.L);

    // the step's logits, one piece of memory, pass through LDS where they do not fit registers
    const int ES = s.E | 1;                              // row stride
    if (!sel && s.E > ROUTE_FEW) {
        for (int i = tid; i < valid * s.E; i += CF_MIX_THREADS) s_B[i / s.E * ES + i % s.E] = to_float(logits[tok0 * s.E + i]);
        __syncthreads();
    }
    if (tid < valid) {
        const int64_t t = tok0 + tid;
        int32_t *ix = s_idx + tid * K;
        float *wx = s_w + tid * K;
        if (sel) {
            for (int r = 0; r < K; ++r) { ix[r] = r; wx[r] = w_sel[t * K + r]; }
        } else {
            const T *gl = logits + t * s.E;
            const float *row = s_B + tid * ES;
            if (s.E <= 8) route_few<8>([&](int e) { return to_float(gl[e]); }, s.E, K, ix, wx);
            else if (s.E <= ROUTE_FEW) route_few<ROUTE_FEW>([&](int e) { return to_float(gl[e]); }, s.E, K, ix, wx);
            else route_many([&](int e) { return row[e]; }, s.E, K, ix, wx);
            if (g_begin == 0 && tid >= r0 && tid < r0 + R)
                for (int r = 0; r < K; ++r) { idx_out[t * K + r] = ix[r]; w_out[t * K + r] = wx[r]; }
        }
    }
    __syncthreads();

    const int rowsE = sel ? K : s.E;
    const int64_t estride = (int64_t)s.G * s.N, tokstride = rowsE * estride;
    const bool vec = (s.N % 4 == 0);
    const int rowsC = max(0, min(valid - r0, R)), rowsB = rowsC > 0 ? min(valid, r0 + R) : 0;
    const int QPR = NP / 4, units = (rowsC + rowsB) * QPR;
    for (int g = g_begin; g < g_begin + gpb; ++g) {
        // ---- mixed rows: a lane takes quads of 4 columns of one stream, QF at a time; C rows [r0, r0 + R), then the B
        // ---- rows up to the last of them ----
        const T *Bg = Be + (tok0 * rowsE * s.G + g) * s.N;
        const T *Cg = Ce + (tok0 * rowsE * s.G + g) * s.N;
        for (int u0 = 0; u0 < units; u0 += QF * CF_MIX_THREADS) {
            float4 am[QF];
#pragma unroll
            for (int m = 0; m < QF; ++m) am[m] = make_float4(0.f, 0.f, 0.f, 0.f);
            for (int r = 0; r < K; ++r) {
                float4 v[QF];
                float ww[QF];
#pragma unroll
                for (int m = 0; m < QF; ++m) {
                    if (u0 + m * CF_MIX_THREADS >= units) continue;          // uniform
                    const int u = min(u0 + m * CF_MIX_THREADS + tid, units - 1);
                    const int rr = u / QPR, n = (u % QPR) * 4, j = rr < rowsC ? r0 + rr : rr - rowsC;
                    const T *src = (rr < rowsC ? Cg : Bg) + j * tokstride + s_idx[j * K + r] * estride;
                    ww[m] = s_w[j * K + r];
                    if (vec) {
                        v[m] = load4(src + min(n, s.N - 4));
                    } else {
                        float t[4];
#pragma unroll
                        for (int q = 0; q < 4; ++q) t[q] = to_float(src[min(n + q, s.N - 1)]);
                        v[m] = make_float4(t[0], t[1], t[2], t[3]);
                    }
                }
#pragma unroll
                for (int m = 0; m < QF; ++m) {
                    if (u0 + m * CF_MIX_THREADS >= units) continue;
                    am[m].x += ww[m] * v[m].x; am[m].y += ww[m] * v[m].y; am[m].z += ww[m] * v[m].z; am[m].w += ww[m] * v[m].w;
                }
            }
#pragma unroll
            for (int m = 0; m < QF; ++m) {
                const int u = u0 + m * CF_MIX_THREADS + tid;
                if (u < units) {
                    const int rr = u / QPR, n = (u % QPR) * 4;
                    float *f = reinterpret_cast<float *>(&am[m]);
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (n + q >= s.N) f[q] = 0.f;                   // padding columns
                    *reinterpret_cast<float4 *>((rr < rowsC ? s_C + (r0 + rr) * RS : s_B + (rr - rowsC) * RS) + n) = am[m];
                }
            }
        }
        __syncthreads();

        const int64_t bcg = ((int64_t)b * s.nc + c) * s.G + g;
        float4 *co = reinterpret_cast<float4 *>(cop) + bcg * (ops.IT * NT * 4 * 64);
        float4 *bo = reinterpret_cast<float4 *>(bop) + bcg * (NT * ops.QN * 64);
        float4 *go = reinterpret_cast<float4 *>(gop) + bcg * (ops.GB * 64);
        // ---- G^T[j][i] = B[j] . C[i] in 16 x 16 tiles (v_mfma_f32_16x16x4_f32): lane (i = lane%16, kq = lane/16) ends
        // ---- with four consecutive j of one i, which is a float4 of gop.  Tiles right of the diagonal are zero.  Rows past
        // ---- the end hold what LDS held: their entries are masked (j > i) or belong to no token. ----
        {
            const int l16 = lane & 15, kq = lane >> 4;
            const int t_begin = PARTS == 1 ? 0 : part < 2 ? 2 * part : 4 * part - 4;
            const int t_end = PARTS == 1 ? 12 : part < 2 ? t_begin + 2 : t_begin + 4;
            for (int t = t_begin + wave; t < t_end; t += CF_MIX_THREADS / 64) {
                // tile rows 0, 1 have columns J = 0, 1; rows 2, 3 columns 0..3
                const int I = t < 4 ? t >> 1 : 2 + ((t - 4) >> 2), J = t < 4 ? t & 1 : (t - 4) & 3;
                if (16 * I >= valid || (one_row && 16 * J >= valid)) continue;
                cf_f32x4_t acc = {0.f, 0.f, 0.f, 0.f};
                if (J <= I) {
                    const float *br = s_B + (16 * J + l16) * RS + 4 * kq, *cr = s_C + (16 * I + l16) * RS + 4 * kq;
                    for (int k = 0; k < NP; k += 16) {
                        const float4 av = *reinterpret_cast<const float4 *>(br + k);
                        const float4 bv = *reinterpret_cast<const float4 *>(cr + k);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av.x, bv.x, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av.y, bv.y, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av.z, bv.z, acc, 0, 0, 0);
                        acc = __builtin_amdgcn_mfma_f32_16x16x4f32(av.w, bv.w, acc, 0, 0, 0);
                    }
                }
                const int i = 16 * I + l16, j0 = 16 * J + 4 * kq;
#pragma unroll
                for (int q = 0; q < 4; ++q)
                    if (j0 + q > i) acc[q] = 0.f;
                const int blk = (i >> 5) * 4 + (j0 >> 3);
                if (blk < ops.GB) go[blk * 64 + ((j0 >> 2) & 1) * 32 + (i & 31)] = make_float4(acc[0], acc[1], acc[2], acc[3]);
            }
        }
        for (int u = tid; u < rowsC * NT * 8; u += CF_MIX_THREADS) {
            const int row = r0 + u % rowsC, v = u / rowsC, kg = v & 1, a = (v >> 1) & 3, nt = v >> 3;
            co[(((row >> 5) * NT + nt) * 4 + a) * 64 + kg * 32 + (row & 31)] =
                *reinterpret_cast<const float4 *>(s_C + row * RS + 32 * nt + 8 * a + 4 * kg);
        }
        const int QS = one_row ? (rowsC + 7) / 8 : R / 8;    // blocks of eight B rows in this workgroup
        for (int u = tid; u < NT * QS * 64; u += CF_MIX_THREADS) {
            const int ln = u & 63, q = r0 / 8 + (u >> 6) % QS, nt = (u >> 6) / QS, row = 8 * q + 4 * (ln >> 5);
            const float *src = s_B + row * RS + 32 * nt + (ln & 31);
            // rows past the end are multiplied by zeros of x: they have to be finite
            bo[(nt * ops.QN + q) * 64 + ln] = make_float4(row < valid ? src[0] : 0.f, row + 1 < valid ? src[RS] : 0.f,
                                                          row + 2 < valid ? src[2 * RS] : 0.f, row + 3 < valid ? src[3 * RS] : 0.f);
        }
        __syncthreads();                                     // the next group's rows
    }
}

// NTW: 32-column state tiles per wave (N <= 128 * NTW).  ROWT: 32-token tile rows of a step (1: sequences of at most
// 32 tokens).  OUT: y (and h_final); otherwise the state part only:
// the segment's own contribution to the state (from zero) into hseg, its total decay (log2) into aseg; with an h_final
// it is segment 0's copy of h0 for the output launch, whose own h_final is the caller's h0.
// SPLIT: waves that share a state tile where there are two or four waves to a tile (N <= 64, 32).  Each adds what its part of
// a step's tokens contributes to a state of its own and reads it out; the readouts meet with the other partial sums of Y, the
// states at the end.  N = 16: 36 MFMAs a wave and step for 76, four heads of 256 tokens 28.8 -> 23.7 us, 48 of 1000 tokens
// 58.4 -> 50.5; N = 64: 60 MFMAs, 48 of 1000 tokens 66.2 -> 58.3.
template <typename T, int NTW, bool OUT, int ROWT, int SPLIT>
__global__ void __launch_bounds__(256, NTW == 1 ? (ROWT == 1 ? 3 : 2) : 1)
chain_f32_kernel(const T *__restrict__ x, const T *__restrict__ dt, const float *__restrict__ A,
                 const float *__restrict__ D, const float *__restrict__ cop, const float *__restrict__ bop,
                 const float *__restrict__ gop, const float *h0, float *h_final,
                 float *__restrict__ hseg, float *__restrict__ aseg, T *__restrict__ y, Shape s, int NT, int nslice,
                 int nrun, int nseg, int steps_per_seg, int total, int nblocks)
{
    constexpr int QT = 4 * ROWT;                                 // 8-token blocks of a step
    constexpr int QW = QT / SPLIT;                               // that the wave adds to its state
    static_assert(OUT || ROWT == 2, "segments are of whole steps");
    static_assert(SPLIT == 1 || NTW == 1, "waves share a tile");
    __shared__ __align__(16) float s_x[2][32 * CF_XS];           // x^T of a step: [channel][token]
    __shared__ __align__(16) float s_cs[2][CF_STEP], s_dt[2][CF_STEP], s_c[2][CF_STEP];
    __shared__ int s_odd;                                        // an x or dt is not finite
    __shared__ __align__(16) float s_y[OUT ? 4 : 1][OUT ? 32 * ROWT * CF_YS : 1];   // partial Y per wave: [token][channel]

    // (batch, segment, head, slice), neighbours (heads of one group) on one XCD: they read the same operands
    const int lid = xcd_logical_id(blockIdx.x, nblocks);
    if (lid >= total) return;
    const int sl = lid % nslice;
    const int h = (lid / nslice) % s.H;
    const int seg = (lid / (nslice * s.H)) % nrun;
    const int b = lid / (nslice * s.H * nrun);
    const int g = (h * s.G) / s.H;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, kg = lane >> 5;
    const int nt0 = SPLIT > 1 ? wave / SPLIT : wave * NTW, part = SPLIT > 1 ? wave % SPLIT : 0;      // first tile of the wave
    const int c_begin = seg * steps_per_seg, c_end = min(s.nc, c_begin + steps_per_seg);
    const int p0 = 32 * sl, P = s.P;
    const float Ah = A[h] * LOG2E;
    const float dsk = (OUT && D) ? D[h] : 0.f;

    // ---- running state: rows n = 32 nt + 8a + 4kg + b, column p0 + l32, in register 4a + b ----
    f32x16_t st[NTW];
    const int p = p0 + l32;
    // a segment's contribution in hseg: (batch, segment, head, slice), then [nt][a][lane], the registers as they are
    auto hseg_frag = [&](int q) __attribute__((always_inline)) {
        return reinterpret_cast<float4 *>(hseg) + ((((int64_t)b * (nseg - 1) + q) * s.H + h) * nslice + sl) * (NT * 256) + lane;
    };
    auto state_at = [&](const float *base, int nt, int a, int q) -> float {      // base: one (P, N) state
        const int n = 32 * nt + 8 * a + 4 * kg + q;
        return (p < P && n < s.N) ? base[(int64_t)p * s.N + n] : 0.f;
    };
    if (!OUT && h_final && seg == 0 && p < P && part == 0) {
        const int64_t o = ((int64_t)b * s.H + h) * P * s.N;
#pragma unroll
        for (int k = 0; k < NTW; ++k)
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int n = 32 * (nt0 + k) + 8 * (v >> 2) + 4 * kg + (v & 3);
                if (n < s.N) h_final[o + (int64_t)p * s.N + n] = h0[o + (int64_t)p * s.N + n];
            }
    }
    // the state in front of this segment
    auto initial = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < NTW; ++k) {
            const int nt = nt0 + k;
#pragma unroll
            for (int v = 0; v < 16; ++v) st[k][v] = 0.f;
            if (OUT && h0 && part == 0) {
                const float *hp = h0 + ((int64_t)b * s.H + h) * P * s.N;
#pragma unroll
                for (int v = 0; v < 16; ++v) st[k][v] = state_at(hp, nt, v >> 2, v & 3);
            }
        }
        if (OUT && part == 0) {
            // the contributions of the segments in front, four requested together
            for (int q0 = 0; q0 < seg; q0 += 4) {
                float dec[4];
                float4 v[4][NTW][4];
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    const int q = min(q0 + u, seg - 1);
                    const float4 *hp = hseg_frag(q);
                    dec[u] = aseg[((int64_t)b * (nseg - 1) + q) * s.H + h];
#pragma unroll
                    for (int k = 0; k < NTW; ++k)
#pragma unroll
                        for (int a = 0; a < 4; ++a) v[u][k][a] = hp[(min(nt0 + k, NT - 1) * 4 + a) * 64];
                }
#pragma unroll
                for (int u = 0; u < 4; ++u) {
                    if (q0 + u >= seg) continue;
                    const float d = fast_exp2(dec[u]);
#pragma unroll
                    for (int k = 0; k < NTW; ++k)
#pragma unroll
                        for (int a = 0; a < 4; ++a) {
                            st[k][4 * a + 0] = d * st[k][4 * a + 0] + v[u][k][a].x;
                            st[k][4 * a + 1] = d * st[k][4 * a + 1] + v[u][k][a].y;
                            st[k][4 * a + 2] = d * st[k][4 * a + 2] + v[u][k][a].z;
                            st[k][4 * a + 3] = d * st[k][4 * a + 3] + v[u][k][a].w;
                        }
                }
            }
        }
    };

    // ---- loads of a step; every one is clamped and unconditional ----
    const int xj = tid >> 2, xp = (tid & 3) * 8;         // this thread's token and 8 channels of the x tile
    const bool vecx = (P % 8 == 0);
    float xn[8];
    float dtn = 0.f;
    auto load_x = [&](int c) __attribute__((always_inline)) {
        const int valid = min(CF_STEP, s.L - c * CF_STEP);
        const int64_t t0 = (int64_t)b * s.L + (int64_t)c * CF_STEP;
        const T *xr = x + ((t0 + min(xj, valid - 1)) * s.H + h) * P + p0;
        if (vecx) {
            const int pc = (p0 + xp < P) ? xp : 0;
            const float4 v0 = load4(xr + pc), v1 = load4(xr + pc + 4);
            xn[0] = v0.x; xn[1] = v0.y; xn[2] = v0.z; xn[3] = v0.w; xn[4] = v1.x; xn[5] = v1.y; xn[6] = v1.z; xn[7] = v1.w;
        } else {
#pragma unroll
            for (int q = 0; q < 8; ++q) xn[q] = to_float(xr[min(xp + q, P - 1 - p0)]);
        }
        dtn = to_float(dt[(t0 + min(lane, valid - 1)) * s.H + h]);
    };
    // In the state part alone the B operand of the next step has no readout to arrive behind: it gets registers of
    // its own (brn) and is requested a whole step ahead.
    float4 cr[NTW][ROWT][4], br[NTW][QW], brn[NTW][QW], gr[ROWT == 2 ? 3 : 1];
    const int64_t bg0 = ((int64_t)b * s.nc) * s.G + g;
    // of one tile row only the blocks with a token are there: the last of them comes for those behind it, to meet zeros
    const ChainOps ops = ROWT == 2 ? ChainOps{2, 8, CF_GBLK} : chain_ops(s.L);
    const int ql = ROWT == 2 ? 7 : ops.QN - 1;
    auto load_c = [&](int c) __attribute__((always_inline)) {
        const float4 *src = reinterpret_cast<const float4 *>(cop) + (bg0 + (int64_t)c * s.G) * (ops.IT * NT * 4 * 64) + lane;
#pragma unroll
        for (int k = 0; k < NTW; ++k)
#pragma unroll
            for (int I = 0; I < ROWT; ++I)
#pragma unroll
                for (int a = 0; a < 4; ++a)
                    cr[k][I][a] = src[((I * NT + min(nt0 + k, NT - 1)) * 4 + a) * 64];
    };
    auto load_b = [&](int c, float4 (&br)[NTW][QW]) __attribute__((always_inline)) {
        const float4 *src = reinterpret_cast<const float4 *>(bop) + (bg0 + (int64_t)c * s.G) * (NT * ops.QN * 64) + lane;
#pragma unroll
        for (int k = 0; k < NTW; ++k)
#pragma unroll
            for (int q = 0; q < QW; ++q) br[k][q] = src[(min(nt0 + k, NT - 1) * ops.QN + min(part * QW + q, ql)) * 64];
    };
    auto load_g = [&](int c) __attribute__((always_inline)) {
        const float4 *src = reinterpret_cast<const float4 *>(gop) + (bg0 + (int64_t)c * s.G) * (ops.GB * 64) + lane;
        gr[0] = src[(ROWT == 2 ? wave : min(wave, ql)) * 64];
#pragma unroll
        for (int t = 1; t < (ROWT == 2 ? 3 : 1); ++t) gr[t] = src[(3 + 2 * wave + t) * 64];
    };
    // x^T tile and tables of step c (in the registers) into buffer buf
    auto stage = [&](int c, int buf) __attribute__((always_inline)) {
        const int valid = min(CF_STEP, s.L - c * CF_STEP);
#pragma unroll
        for (int q = 0; q < 8; ++q)
            s_x[buf][(xp + q) * CF_XS + xj] = (xj < valid && p0 + xp + q < P) ? xn[q] : 0.f;
        if (wave == 3) {
            const float dv = (lane < valid) ? dtn : 0.f;
            const float cs = wave_scan(dv * Ah);
            const float last = __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(cs), 63));
            s_cs[buf][lane] = cs;
            s_dt[buf][lane] = dv;
            s_c[buf][lane] = dv * fast_exp2(last - cs);
        }
    };

    float atot = 0.f;
    float odd = 0.f;                                     // NaN once zero times anything not finite has been added
    auto step = [&](int c, float4 (&br)[NTW][QW], float4 (&brn)[NTW][QW], auto one_by_one) __attribute__((always_inline)) {
        const int buf = (c - c_begin) & 1;
        const int cn = min(c + 1, c_end - 1);
        float xc[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) xc[q] = xn[q];
        if constexpr (OUT && !decltype(one_by_one)::value) {
#pragma unroll
            for (int q = 0; q < 8; ++q) odd += 0.f * xn[q];
            odd += 0.f * dtn;
        }
        lds_barrier();                                   // step c is staged
        load_x(cn);
        if (!OUT) load_b(cn, brn);
        const float *sx = s_x[buf] + l32 * CF_XS + 4 * kg;
        const float cs_last = s_cs[buf][CF_STEP - 1];
        f32x16_t yt[ROWT];                               // Y^T: rows are channels, so a lane holds four of one token
        if (OUT) {
#pragma unroll
            for (int v = 0; v < 16; ++v) yt[0][v] = yt[ROWT - 1][v] = 0.f;
            const float ci[2] = {s_cs[buf][l32], s_cs[buf][32 * (ROWT - 1) + l32]};
            const float ei[2] = {fast_exp2(ci[0]), fast_exp2(ci[1])};
#pragma unroll
            for (int k = 0; k < NTW; ++k)
                if (nt0 + k < NT) {                      // wave-uniform
#pragma unroll
                    for (int a = 0; a < 4; ++a) {
                        if (SPLIT == 4 && 8 * a >= s.N) break;           // columns that do not exist
                        const float4 u0 = cr[k][0][a], u1 = cr[k][ROWT - 1][a];
                        yt[0] = mfma_f32(st[k][4 * a + 0], u0.x * ei[0], yt[0]);
                        if (ROWT == 2) yt[ROWT - 1] = mfma_f32(st[k][4 * a + 0], u1.x * ei[1], yt[ROWT - 1]);
                        yt[0] = mfma_f32(st[k][4 * a + 1], u0.y * ei[0], yt[0]);
                        if (ROWT == 2) yt[ROWT - 1] = mfma_f32(st[k][4 * a + 1], u1.y * ei[1], yt[ROWT - 1]);
                        yt[0] = mfma_f32(st[k][4 * a + 2], u0.z * ei[0], yt[0]);
                        if (ROWT == 2) yt[ROWT - 1] = mfma_f32(st[k][4 * a + 2], u1.z * ei[1], yt[ROWT - 1]);
                        yt[0] = mfma_f32(st[k][4 * a + 3], u0.w * ei[0], yt[0]);
                        if (ROWT == 2) yt[ROWT - 1] = mfma_f32(st[k][4 * a + 3], u1.w * ei[1], yt[ROWT - 1]);
                    }
                }
            load_c(cn);
            // the wave's 8-token blocks of M: one of tile row 0 and two of tile row 1, the same code in every wave
#pragma unroll
            for (int t = 0; t < (ROWT == 2 ? 3 : 1); ++t) {
                const int I = t > 0, q = t > 0 ? 2 * wave + t - 1 : wave;
                if constexpr (decltype(one_by_one)::value) {
#pragma unroll 1
                    for (int jj = 0; jj < 8; ++jj) {
                        const int j = 8 * q + jj, b4 = jj & 3;
                        const float g4 = b4 == 0 ? gr[t].x : b4 == 1 ? gr[t].y : b4 == 2 ? gr[t].z : gr[t].w;
                        const float m = __shfl(g4, l32 + 32 * (jj >> 2)) * s_dt[buf][j] *
                                        fast_exp2(fminf(ci[I] - s_cs[buf][j], 127.f));
#pragma unroll
                        for (int v = 0; v < 16; ++v) {
                            const float xv = s_x[buf][(8 * (v >> 2) + 4 * kg + (v & 3)) * CF_XS + j];
                            if (j <= 32 * I + l32) yt[I][v] += m * xv;
                        }
                    }
                    continue;
                }
                const float4 cj = *reinterpret_cast<const float4 *>(&s_cs[buf][8 * q + 4 * kg]);
                const float4 dj = *reinterpret_cast<const float4 *>(&s_dt[buf][8 * q + 4 * kg]);
                const float4 xv = *reinterpret_cast<const float4 *>(sx + 8 * q);
                // entries with j > i are zero in G; the clamp keeps their factor finite and, at 127, leaves the others
                // alone where a state grows (A > 0)
                const float m0 = (gr[t].x * dj.x) * fast_exp2(fminf(ci[I] - cj.x, 127.f));
                const float m1 = (gr[t].y * dj.y) * fast_exp2(fminf(ci[I] - cj.y, 127.f));
                const float m2 = (gr[t].z * dj.z) * fast_exp2(fminf(ci[I] - cj.z, 127.f));
                const float m3 = (gr[t].w * dj.w) * fast_exp2(fminf(ci[I] - cj.w, 127.f));
                yt[I] = mfma_f32(xv.x, m0, yt[I]);
                yt[I] = mfma_f32(xv.y, m1, yt[I]);
                yt[I] = mfma_f32(xv.z, m2, yt[I]);
                yt[I] = mfma_f32(xv.w, m3, yt[I]);
            }
            load_g(cn);
        } else {
            atot += cs_last;
        }
        // ---- state ----
        {
            const float dec = fast_exp2(cs_last);
#pragma unroll
            for (int k = 0; k < NTW; ++k)
#pragma unroll
                for (int v = 0; v < 16; ++v) st[k][v] *= dec;
#pragma unroll
            for (int k = 0; k < NTW; ++k) {
                if (nt0 + k >= NT) continue;             // wave-uniform; outside the token loop, whose LDS reads overlap
#pragma unroll
                for (int q = 0; q < QW; ++q) {
                    const int qb = part * QW + q;
                    const float4 cj = *reinterpret_cast<const float4 *>(&s_c[buf][8 * qb + 4 * kg]);
                    const float4 xv = *reinterpret_cast<const float4 *>(sx + 8 * qb);
                    st[k] = mfma_f32(br[k][q].x, xv.x * cj.x, st[k]);
                    st[k] = mfma_f32(br[k][q].y, xv.y * cj.y, st[k]);
                    st[k] = mfma_f32(br[k][q].z, xv.z * cj.z, st[k]);
                    st[k] = mfma_f32(br[k][q].w, xv.w * cj.w, st[k]);
                }
            }
            if (OUT) load_b(cn, br);
        }
        if (OUT) {
            // the partial tiles of the four waves meet in LDS (those of the previous step were added up in front
            // of the barrier at the top)
#pragma unroll
            for (int I = 0; I < ROWT; ++I)
#pragma unroll
                for (int a = 0; a < 4; ++a)
                    *reinterpret_cast<float4 *>(&s_y[wave][(32 * I + l32) * CF_YS + 8 * a + 4 * kg]) =
                        make_float4(yt[I][4 * a], yt[I][4 * a + 1], yt[I][4 * a + 2], yt[I][4 * a + 3]);
        }
        stage(cn, buf ^ 1);
        if (OUT) {
            if constexpr (!decltype(one_by_one)::value)
                if (__ballot(!(odd == 0.f))) s_odd = 1;
            lds_barrier();
            const int valid = min(CF_STEP, s.L - c * CF_STEP);
            if (xj < valid && p0 + xp < P) {
                float r[8];
#pragma unroll
                for (int q = 0; q < 2; ++q) {
                    const float4 a0 = *reinterpret_cast<const float4 *>(&s_y[0][xj * CF_YS + xp + 4 * q]);
                    const float4 a1 = *reinterpret_cast<const float4 *>(&s_y[1][xj * CF_YS + xp + 4 * q]);
                    const float4 a2 = *reinterpret_cast<const float4 *>(&s_y[2][xj * CF_YS + xp + 4 * q]);
                    const float4 a3 = *reinterpret_cast<const float4 *>(&s_y[3][xj * CF_YS + xp + 4 * q]);
                    r[4 * q + 0] = (a0.x + a1.x) + (a2.x + a3.x) + dsk * xc[4 * q + 0];
                    r[4 * q + 1] = (a0.y + a1.y) + (a2.y + a3.y) + dsk * xc[4 * q + 1];
                    r[4 * q + 2] = (a0.z + a1.z) + (a2.z + a3.z) + dsk * xc[4 * q + 2];
                    r[4 * q + 3] = (a0.w + a1.w) + (a2.w + a3.w) + dsk * xc[4 * q + 3];
                }
                T *yr = y + (((int64_t)b * s.L + (int64_t)c * CF_STEP + xj) * s.H + h) * P + p0 + xp;
                if (vecx) {
                    if constexpr (sizeof(T) == 4) {
                        *reinterpret_cast<float4 *>(yr) = make_float4(r[0], r[1], r[2], r[3]);
                        *reinterpret_cast<float4 *>(yr + 4) = make_float4(r[4], r[5], r[6], r[7]);
                    } else {
                        *reinterpret_cast<uint4 *>(yr) = pack8(r);
                    }
                } else {
#pragma unroll
                    for (int q = 0; q < 8; ++q)
                        if (p0 + xp + q < P) yr[q] = from_float<T>(r[q]);
                }
            }
        }
    };
    auto walk = [&](auto one_by_one) __attribute__((always_inline)) {
        initial();
        load_x(c_begin);
        if (OUT) { load_c(c_begin); load_g(c_begin); }
        load_b(c_begin, br);
        stage(c_begin, 0);
        if (OUT) {
            for (int c = c_begin; c < c_end; ++c) step(c, br, br, one_by_one);
        } else {
            for (int c = c_begin; c < c_end; c += 2) {
                step(c, br, brn, one_by_one);
                if (c + 1 < c_end) step(c + 1, brn, br, one_by_one);
            }
        }
    };
    if (OUT && tid == 0) s_odd = 0;
    walk(std::false_type{});
    // A masked entry of M (j > i) times an x or dt that is not finite is NaN, in tokens that such a value must not
    // reach.  The segment is then walked again with the products of M taken one by one, only those with j <= i.  (Testing
    // inside a step instead, with a branch there or with finite stand-ins for such values, keeps the products of M from
    // overlapping with the readout: 104.4 us on the 130M-shaped layer where this takes 101.4.)
    if constexpr (OUT)
        if (__builtin_amdgcn_readfirstlane(s_odd)) {
            __syncthreads();                             // every wave has read it
            walk(std::true_type{});
        }
    if constexpr (SPLIT > 1) {
        // the waves' states of a tile added up, in the first one of them
        static_assert(sizeof(s_x) >= 4 * 1024 * sizeof(float), "room for four tiles");
        float4 *tiles = reinterpret_cast<float4 *>(&s_x[0][0]) + lane;
        __syncthreads();                                 // every wave is done with x
#pragma unroll
        for (int a = 0; a < 4; ++a) tiles[(wave * 4 + a) * 64] = make_float4(st[0][4 * a], st[0][4 * a + 1], st[0][4 * a + 2], st[0][4 * a + 3]);
        __syncthreads();
        if (part) return;
#pragma unroll
        for (int w = 1; w < SPLIT; ++w)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const float4 v = tiles[((wave + w) * 4 + a) * 64];
                st[0][4 * a] += v.x; st[0][4 * a + 1] += v.y; st[0][4 * a + 2] += v.z; st[0][4 * a + 3] += v.w;
            }
    }
    if (!OUT) {
        float4 *dst = hseg_frag(seg);
#pragma unroll
        for (int k = 0; k < NTW; ++k) {
            if (nt0 + k >= NT) continue;                 // wave-uniform
#pragma unroll
            for (int a = 0; a < 4; ++a)
                dst[((nt0 + k) * 4 + a) * 64] =
                    make_float4(st[k][4 * a], st[k][4 * a + 1], st[k][4 * a + 2], st[k][4 * a + 3]);
        }
    }
    float *dst = OUT && seg == nseg - 1 && h_final ? h_final + ((int64_t)b * s.H + h) * P * s.N : nullptr;
    if (dst && p < P) {
#pragma unroll
        for (int k = 0; k < NTW; ++k)
#pragma unroll
            for (int a = 0; a < 4; ++a) {
                const int n = 32 * (nt0 + k) + 8 * a + 4 * kg;
                float *q = dst + (int64_t)p * s.N + n;
                if (s.N % 4 == 0) {
                    if (n < s.N)
                        *reinterpret_cast<float4 *>(q) = make_float4(st[k][4 * a], st[k][4 * a + 1], st[k][4 * a + 2], st[k][4 * a + 3]);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (n + e < s.N) q[e] = st[k][4 * a + e];
                }
            }
    }
    if (!OUT && sl == 0 && tid == 0) aseg[((int64_t)b * (nseg - 1) + seg) * s.H + h] = atot;
}

// Segments a sequence is walked in.  A chain keeps a quarter of a compute unit's two resident workgroups busy
// for its whole segment, so short of about 1.5 workgroups per compute unit the chip idles; the extra
// launch (state part of all segments but the last, 2/5 of the work) pays from four steps per segment on.  Short of 192
// chains most of the chip idles either way and the serial steps are all there is: two steps per segment, from six
// steps on (four heads, P = N = 16, 700 tokens: one segment 53.4 us, four 30.5; 1024 tokens, eight heads, P = 64,
// N = 128: four 47.1, eight 37.5; three to five steps: 28.3 -> 31.5, 32.4 -> 32.9, 36.1 -> 38.6 with 96 chains).
// Up to 64 segments: 16384 tokens of one head, P = N = 16, 206 us in 8, 115 in 16, 72 in 32, 56 in 64; of eight heads,
// P = 64, N = 128, 239 in 8, 138 in 16 (256 chains).  From 192 chains on eight at most: where a unit holds one chain
// (N > 128) 448 take two rounds (14 x 4347 tokens, two heads, N = 256: 180 us in 8, 209 in 16).
int chain_f32_segments(int64_t B, int64_t L, int64_t H, int64_t P)
{
    const int64_t steps = (L + CF_STEP - 1) / CF_STEP, chains = B * H * ((P + 31) / 32);
    if (chains == 0) return 1;
    int nseg = 1;
    while (nseg < CHAIN_F32_MAX_SEGMENTS && ((chains * nseg < 192 && steps > 5 && steps > 2 * (int64_t)nseg) ||
                                             (nseg < 8 && chains * nseg < 384 && steps >= 8 * (int64_t)nseg)))
        nseg *= 2;
    // Some compute units then hold one chain more than others and set the time: twice as many chains of half the
    // length where that takes a fifth off the fullest unit (96 chains of 32 steps: 4 segments 113 us, 8 102;
    // 128 chains, where it takes nothing off: 113 and 125).
    const int64_t cus = 256, full = (chains * nseg + cus - 1) / cus, full2 = (2 * chains * nseg + cus - 1) / cus;
    if (nseg > 1 && nseg < 8 && steps >= 8 * (int64_t)nseg && 10 * full2 <= 16 * full) nseg *= 2;
    return nseg;
}

void chain_f32_sizes(const swimba_dims *d, size_t *cop, size_t *bop, size_t *g, size_t *seg, size_t *dec, size_t *init)
{
    const size_t nc = ((size_t)d->seqlen + CF_STEP - 1) / CF_STEP, NT = ((size_t)d->dstate + 31) / 32;
    const size_t items = (size_t)d->batch * nc * d->ngroups;
    const size_t nseg = chain_f32_segments(d->batch, d->seqlen, d->nheads, d->headdim);
    const ChainOps o = chain_ops(d->seqlen);
    *cop = items * o.IT * NT * 4 * 64 * 16;
    *bop = items * o.QN * NT * 64 * 16;
    *g = items * o.GB * 64 * 16;
    *dec = (size_t)d->batch * (nseg - 1) * d->nheads * sizeof(float);
    *seg = (size_t)d->batch * (nseg - 1) * d->nheads * ((d->headdim + 31) / 32) * NT * 1024 * sizeof(float);
    *init = nseg > 1 ? (size_t)d->batch * d->nheads * d->headdim * d->dstate * sizeof(float) : 0;
}

template <typename T, int NTW, int SPLIT>
static void launch_chain_t(const Shape &s, const void *x, const void *dt, const float *A, const float *D, const float *cop,
                           const float *bop, const float *gop, const float *h0, float *h_final, float *hseg,
                           float *aseg, float *hinit, void *y, int NT, int nseg, hipStream_t st)
{
    const int nslice = (s.P + 31) / 32, sps = (s.nc + nseg - 1) / nseg;
    const int used = (s.nc + sps - 1) / sps;             // segments that have steps
    if (used > 1) {
        // With the final state written over the initial one the segments of the output launch read a copy: the last
        // segment of a sequence can end before another one has started.
        float *copy = h0 && h0 == h_final ? hinit : nullptr;
        const int total = s.B * (used - 1) * s.H * nslice, nblocks = xcd_padded(total);
        hipLaunchKernelGGL((chain_f32_kernel<T, NTW, false, 2, SPLIT>), dim3(nblocks), dim3(256), 0, st, (const T *)x, (const T *)dt,
                           A, D, cop, bop, gop, h0, copy, hseg, aseg, (T *)y, s, NT, nslice, used - 1, used, sps, total, nblocks);
        if (copy) h0 = copy;
    }
    const int total = s.B * used * s.H * nslice, nblocks = xcd_padded(total);
    // at most 32 tokens: one tile row, 36 MFMAs for 76 and three workgroups per compute unit
    auto out = s.L > 32 ? chain_f32_kernel<T, NTW, true, 2, SPLIT> : chain_f32_kernel<T, NTW, true, 1, SPLIT>;
    hipLaunchKernelGGL(out, dim3(nblocks), dim3(256), 0, st, (const T *)x, (const T *)dt, A, D, cop, bop, gop, h0, h_final,
                       hseg, aseg, (T *)y, s, NT, nslice, used, used, sps, total, nblocks);
}

template <typename T>
static swimba_status launch_f32_t(const Shape &s, const void *x, const void *dt, const float *A, const float *D,
                                  const void *Be, const void *Ce, const void *logits, const float *w_sel,
                                  const float *h0, void *y, float *h_final, int32_t *idx, float *w, float *cop,
                                  float *bop, float *gop, float *hseg, float *aseg, float *hinit, int nseg, hipStream_t st)
{
    const int NT = (s.N + 31) / 32;
    const size_t rows = (size_t)2 * CF_STEP * (32 * NT + 4), row_logits = w_sel ? 0 : (size_t)CF_STEP * (s.E | 1);
    const size_t shm = (size_t)CF_STEP * s.K * 8 + (rows > row_logits ? rows : row_logits) * sizeof(float);
    // more than 64 KB of dynamic LDS has to be allowed once per device
    static std::atomic<uint64_t> attr_set{0};            // one bit per device ordinal
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) { set_last_hip_error((int)e); return SWIMBA_ERR_HIP; }
    const uint64_t bit = 1ull << (dev & 63);
    if (!(attr_set.load(std::memory_order_acquire) & bit)) {
        constexpr size_t most = (size_t)CF_STEP * SWIMBA_MAX_TOPK * 8 + (size_t)2 * CF_STEP * (SWIMBA_MAX_DSTATE + 4) * sizeof(float);
        e = hipFuncSetAttribute((const void *)mix_ops_kernel<T, 1, 4>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)mix_ops_kernel<T, 1, 8>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
        if (e == hipSuccess)
            e = hipFuncSetAttribute((const void *)mix_ops_kernel<T, 4, 8>, hipFuncAttributeMaxDynamicSharedMemorySize, (int)most);
        if (e != hipSuccess) { set_last_hip_error((int)e); return SWIMBA_ERR_HIP; }
        attr_set.fetch_or(bit, std::memory_order_release);
    }
    const int64_t items = (int64_t)s.B * s.nc * s.G;
    // Up to a quarter as many steps as compute units (64 here) four workgroups share one, each on a unit of its own:
    // 4 steps 32.3 us for 35.4, 64 steps of the 130M-shaped layer 101.9 for 105.8.  Beyond, a part would wait for
    // another's unit: 96 steps 157.9 for 153.2, 256 steps 282 for 255.
    const int ncu = std::max(device_cus(), 1);   // without a device the launch below reports it
    if (items <= ncu / 4)
        hipLaunchKernelGGL((mix_ops_kernel<T, 4, 8>), dim3((unsigned)items * 4), dim3(CF_MIX_THREADS), shm, st, (const T *)Be,
                           (const T *)Ce, (const T *)logits, idx, w, w_sel, cop, bop, gop, s, NT, 1);
    else {
        // Groups share a workgroup and its routing (about one group's time, three beyond 16 experts) where that takes
        // time off the rounds of two workgroups per compute unit: 700 x 9 tokens, 4 groups, 64 experts, 136 us with a group
        // each, 95 with two, 81 with four; 89 x 146 tokens, 8 groups, N = 256, where four would leave 22 workgroups for
        // a second round, 273 with four, 246 with two.
        int gpb = 1;
        int64_t least = 0;
        for (int n = 1; n <= s.G; ++n) {
            const int64_t time = (items / n + 2 * ncu - 1) / (2 * ncu) * ((s.E > 16 && !w_sel ? 3 : 1) + n);
            if (s.G % n == 0 && (n == 1 || time < least)) {
                gpb = n;
                least = time;
            }
        }
        // more than half a unit's LDS (states beyond 128): no second workgroup beside it
        auto mix = 2 * shm > 160 * 1024 ? mix_ops_kernel<T, 1, 8> : mix_ops_kernel<T, 1, 4>;
        hipLaunchKernelGGL(mix, dim3((unsigned)(items / gpb)), dim3(CF_MIX_THREADS), shm, st, (const T *)Be,
                           (const T *)Ce, (const T *)logits, idx, w, w_sel, cop, bop, gop, s, NT, gpb);
    }
    SWIMBA_CHECK_LAUNCH();
    const auto chain = NT > 4 ? launch_chain_t<T, 2, 1> : NT > 2 ? launch_chain_t<T, 1, 1> : NT == 2 ? launch_chain_t<T, 1, 2> : launch_chain_t<T, 1, 4>;
    chain(s, x, dt, A, D, cop, bop, gop, h0, h_final, hseg, aseg, hinit, y, NT, nseg, st);
    SWIMBA_CHECK_LAUNCH();
    return SWIMBA_OK;
}

// logits / idx / w: routing inside (w_sel == nullptr); w_sel: rows of the selected experts with given weights
swimba_status launch_chain_f32(const Shape &s0, int io_dtype, const void *x, const void *dt, const float *A,
                               const float *D, const void *Be, const void *Ce, const void *logits, const float *w_sel,
                               const float *h0, void *y, float *h_final, int32_t *idx, float *w, float *cop, float *bop,
                               float *gop, float *hseg, float *aseg, float *hinit, hipStream_t st)
{
    Shape s = s0;
    s.Q = CF_STEP;
    s.nc = (s.L + CF_STEP - 1) / CF_STEP;
    if ((int64_t)s.B * s.nc == 0) return SWIMBA_OK;
    const int nseg = chain_f32_segments(s.B, s.L, s.H, s.P);
    if ((int64_t)s.B * s.nc * s.G > 0x7fffffffll || (int64_t)s.B * nseg * s.H * ((s.P + 31) / 32) > 0x7ffffff0ll)
        return SWIMBA_ERR_UNSUPPORTED;
    if (io_dtype == SWIMBA_BF16)
        return launch_f32_t<bf16>(s, x, dt, A, D, Be, Ce, logits, w_sel, h0, y, h_final, idx, w, cop, bop, gop, hseg, aseg,
                                  hinit, nseg, st);
    return launch_f32_t<float>(s, x, dt, A, D, Be, Ce, logits, w_sel, h0, y, h_final, idx, w, cop, bop, gop, hseg, aseg,
                               hinit, nseg, st);
}

}  // namespace swimba
