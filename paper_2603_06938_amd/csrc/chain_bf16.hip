// SSD forward for bf16 io on v_mfma_f32_32x32x16_bf16 as one walk over 64-token steps per (batch, head)
// (paper, background section on SSD: matrix work inside chunks, a linear recurrence between chunks; Theorem 1: the
// mixed streams feed one plain SSM).  The chunk length changes no bit of a finite result; ChainPieces has the other case.
//   mix_steps_kernel   (batch, step, groups): routes 64 tokens, mixes their B and C rows and writes them, and the masked
//                      products G = C B^T, as the operand registers the chain reads; and, in workgroups of its own, the
//                      decay tables of every (batch, head, step).  Shared by the heads of a group.
//   chain_bf16_kernel  (batch, head, 64 or 32 channels): the state never leaves the accumulators.  With a reference R of the
//                      step (ChainTables) x~_j = f_j x_j, H' = the state at R:
//                        Y[i][p]  = e_i (sum_n C[i][n] H'[n][p] + sum_j G[i][j] x~_j[p]) + D x_i[p]
//                        H'      <- 2^(R_next - ..) (H' + sum_j B[j][n] x~_j[p])
//                      so the three contractions take x~ alone, G as it was written, and no operand is scaled per head.
// Two state waves, half of the columns each, keep H' in the accumulators and write it, rounded to bf16, into LDS as the operand
// registers of the readout; two readout waves, 32 of the 64 tokens each, take it from there a step later with C, G and x~ and
// leave Y in LDS (N = 128 and 64 channels: 16 and 20 or 24 MFMAs each per step).  So every operand is read by one wave of the
// workgroup, and two steps ahead.  I/O waves load x three steps ahead, write x~ into LDS two steps ahead, and finish and store Y
// one step behind; one LDS-only barrier a step.  ds_read_b64_tr_b16 transposes x~ (and, in the mix kernel, B) on the way out of
// LDS.
// Too few chains to fill the chip: a sequence is walked as segments, whose initial states come from a launch in front of the
// chain (ChainPieces, chain_bf16_segments).
//
// Against four like waves of 32 channels x half of the columns, which read every operand twice, one step ahead, and met partial
// sums of Y in LDS: 130M-shaped layer 55.4 -> 50.7 us, 370M-shaped layer 115 -> 103, five sequences of 1237 tokens x 32 heads
// 34.9 -> 31.1, two of 16384 x 64 335 -> 316; 1 to 3 steps cost 0.2 to 0.4 us more (150 tokens x 24 heads 13.3 -> 13.5).
// Bound: a step takes 1.0 us wherever its x, y and operands lie in the caches (19 % of it MFMAs, 28 % vector instructions, 35 % of
// the waves' time waits for LDS and the barrier, all waves alike), 1.35 in the 370M-shaped layer, where x and y stream at
// 3.2 TB/s.  Worse: Y finished and stored by the readout waves, 32-byte pieces of rows (370M 131 us for the walk's 91); x read
// again for the finish (97); state and readout in the same four waves (96); one channel tile a workgroup, two to a unit (138).
#include "common.hpp"
#include "mfma_util.hpp"

#include <algorithm>
#include <atomic>
#include <initializer_list>
#include <type_traits>
#include <utility>

namespace swimba {

constexpr int CB_STEP = 64;            // tokens per step
constexpr int CB_MIX_THREADS = 512;
constexpr float CB_RANGE = 120.f;      // most that cs falls under one reference (ChainTables)
constexpr int CB_RING = 6;             // x tiles in an i/o wave's registers (a multiple of the 3 in LDS)

typedef __attribute__((ext_vector_type(4))) short cb_s16x4_t;
typedef __attribute__((address_space(3))) cb_s16x4_t cb_lds_s16x4_t;

typedef __attribute__((ext_vector_type(4))) float cb_f32x4_t;
typedef __attribute__((ext_vector_type(2))) float cb_f32x2_t;
typedef __attribute__((address_space(4))) cb_f32x2_t cb_scalar_f32x2_t;          // read through the scalar cache

// Largest of the 64 lanes' values, none of them negative, in lane 63
__device__ __forceinline__ float wave_max(float v)
{
#define WAVE_MAX_STEP(ctrl, rows) \
    v = fmaxf(v, __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), ctrl, rows, 0xf, false)))
    WAVE_MAX_STEP(0x111, 0xf);   // row_shr:1
    WAVE_MAX_STEP(0x112, 0xf);   // row_shr:2
    WAVE_MAX_STEP(0x114, 0xf);   // row_shr:4
    WAVE_MAX_STEP(0x118, 0xf);   // row_shr:8
    WAVE_MAX_STEP(0x142, 0xa);   // row_bcast:15 into rows 1 and 3
    WAVE_MAX_STEP(0x143, 0xc);   // row_bcast:31 into rows 2 and 3
#undef WAVE_MAX_STEP
    return v;
}

// 16 lanes read a 4 x 16 block of 16-bit elements, lane s four columns of row s / 4; lane s gets column s, rows 0..3
__device__ __forceinline__ uint2 lds_read_tr(const unsigned char *p)
{
    return __builtin_bit_cast(uint2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((cb_lds_s16x4_t *)(p)));
}

__device__ __forceinline__ float lane_value(float v, int l)
{
    return __uint_as_float((uint32_t)__builtin_amdgcn_readlane((int)__float_as_uint(v), l));
}

// Operand images, one item per (batch, step, group), NT tiles of 32 state columns:
//   C (2, 2 NT, 64, 8) [I][s][lane][e]   = C[32 I + lane%32][16 s + 8(e/4) + 4(lane/32) + e%4]
//   B (NT, 4, 64, 8)   [nt][ks][lane][e] = B[16 ks + 8(e/4) + 4(lane/32) + e%4][32 nt + lane%32]
//   G (6, 64, 8)       [f][lane][e]      = (j <= i) C[i] . B[j];  f < 2: i = lane%32, j = 16 f + ..; else i = 32 + lane%32,
//                                          j = 16 (f - 2) + 8(e/4) + 4(lane/32) + e%4
__host__ __device__ constexpr int cb_item_frags(int NT) { return 8 * NT + 6; }

// Per (batch, head, step), written by the mix launch (cs: inclusive sum of log2 e dt A from the step's first token, whole and
// part its nearest whole number and the rest):
//   fe  (B, H, nsteps, 32, 2, 2)  factor of x, dt_j 2^(R - cs_j), and of y, 2^(cs_i - R), tokens j and j + 32 side by side; of a
//                              direct step dt_j and cs_j
//   ref (B, H, nsteps, 2)      mode and references (pack_ref); 2^(part of cs_last)
//   sum (B, H, nsteps)         cs_last
//   mag (B, nsteps, G, 2)      bounds for x times its factor (mag_bounds)
// With a reference R in the middle of the step's range, 2^(cs_i - cs_j) dt_j is a factor of token j times a factor of token i,
// both far from the ends of the exponent range: no element of the masked products needs a factor of its own, and the state is
// updated and read at R, too.
//   mode 0  one reference for the step, whose cs falls by at most CB_RANGE
//   mode 1  one for each half of 32 tokens, each of which falls by at most that: the state and the second half's Y change over
//           in the middle of the step
//   mode 2  direct: the others, steps where cs rises, and values that are not finite.  Token j takes dt_j 2^(-part_j), the
//           masked products 2^(whole_i - whole_j) element by element, and the state another copy of x times
//           2^(whole_last - whole_j).
// The parts go where they go in every mode, and the rest are whole powers of two: the modes round alike, and the bits of a
// token do not depend on the tokens behind it, which choose the mode.
// A direct step takes 0.1 to 0.3 us longer: all steps direct, 130M-shaped layer 52 -> 55 us, 370M-shaped layer 100 -> 104,
// five sequences of 1237 tokens x 32 heads 32 -> 39.  A smaller CB_RANGE makes more steps direct: before the state and readout
// waves parted, when these were 56 -> 58, 115 -> 121 and 37 -> 41, a range of 32 took 66, 122 and 45 us.
// A step size or decay that is not finite makes the tokens from its own on and the state behind them NaN, those in front take
// the direct step without it.  A token's cs falls by 300 at most, which leaves nothing of any fp32 value.
// Factors of up to 2^60 either way could take a product that is in range by itself out of it.  So the waves that multiply x by
// its factor look at what comes out: a step with anything above an upper bound, or, where the reference is more than 8 from
// some token's cs, with eight channels of a token that are all below a lower one, is turned direct before it is used
// (mag_bounds; turn_direct).  The bounds leave 2^26 to the ends of the exponent range, for sums of up to N products and for
// elements of B, C and x far under the largest.  The check costs 45 ns of a step where memory does not set the time: five
// sequences of 1237 tokens 35.4 -> 36.6 us (some steps with two references), 150 tokens x 24 heads 12.9 -> 13.3.
struct ChainTables {
    float *fe, *ref, *sum, *mag;
};
constexpr float CB_NEAR = 16.f;        // most that cs falls in a step that takes no harm from small values
__device__ __forceinline__ float2 mag_bounds(float b, float c)      // largest |B| and |C|
{
    const int eb = __builtin_amdgcn_frexp_expf(b), ebc = eb + __builtin_amdgcn_frexp_expf(c);
    return make_float2(ldexpf(1.f, max(0, max(-eb, -ebc)) - 100), ldexpf(1.f, 100 - max(0, max(eb, ebc))));
}
// mode; R0, whole part of cs_last less the last reference, R1 - R0; of a direct step 0, 0, whole part of cs_last
__device__ __forceinline__ int pack_ref(int mode, int R0, int rem, int R1) { return mode | (R0 + 128) << 2 | (rem + 128) << 10 | (R1 - R0 + 128) << 18; }
__device__ __forceinline__ int pack_direct(int last) { return 2 | last << 2; }
__device__ __forceinline__ int ref_mode(int p) { return p & 3; }
__device__ __forceinline__ int ref_r0(int p) { return ref_mode(p) == 2 ? 0 : ((p >> 2) & 255) - 128; }
__device__ __forceinline__ int ref_rem(int p) { return ref_mode(p) == 2 ? 0 : ((p >> 10) & 255) - 128; }
__device__ __forceinline__ int ref_shift(int p) { return ref_mode(p) == 2 ? p >> 2 : ((p >> 18) & 255) - 128; }

__device__ __forceinline__ void chain_table(const ChainTables &t, int64_t bhs, float d, float Ah, int lane)
{
    const float raw = d * Ah;
    const uint64_t bad = __ballot(!(fabsf(d) <= 3e38f) || !(raw <= 3e38f));
    const float v = fminf(fmaxf(raw, -300.f), 300.f);
    const float cs = wave_scan(v);
    const float mid = lane_value(cs, 31), last = lane_value(cs, 63);
    const bool falls = bad == 0 && __ballot(v > 0.f) == 0;
    const int mode = falls && -last <= CB_RANGE ? 0 : falls && -mid <= CB_RANGE && mid - last <= CB_RANGE ? 1 : 2;
    const float last_whole = rintf(last);
    float2 fe = make_float2(d, cs);
    float frac = fast_exp2(last - last_whole), sum = last;
    int pack = pack_direct((int)last_whole);
    if (mode != 2) {
        const float R0 = rintf(0.5f * (mode == 0 ? last : mid)), R1 = mode == 0 ? R0 : rintf(0.5f * (mid + last));
        const float whole = rintf(cs), part = cs - whole, R = lane < 32 ? R0 : R1;
        fe.x = ldexpf(d * fast_exp2(-part), (int)(R - whole));
        fe.y = ldexpf(fast_exp2(part), (int)(whole - R));
        // mode 1: R0, R1 and cs_last can be far from the step's start, but not from each other's tile
        pack = pack_ref(mode, (int)R0, (int)(last_whole - R1), (int)R1);
    } else if (bad != 0) {
        if (lane >= __builtin_ctzll(bad)) fe = make_float2(0.f, NAN);
        frac = sum = NAN;
    }
    reinterpret_cast<float2 *>(t.fe)[bhs * CB_STEP + 2 * (lane & 31) + (lane >> 5)] = fe;
    if (lane == 0) {
        reinterpret_cast<float2 *>(t.ref)[bhs] = make_float2(__int_as_float(pack), frac);
        t.sum[bhs] = sum;
    }
}

template <int NT, bool SEL, bool ONCE>                   // SEL: rows of the selected experts and their weights; ONCE: row_piece
__global__ void __launch_bounds__(CB_MIX_THREADS, 4)
mix_steps_kernel(const bf16 *__restrict__ Be, const bf16 *__restrict__ Ce, const bf16 *__restrict__ logits,
                 int32_t *__restrict__ idx_out, float *__restrict__ w_out, const float *__restrict__ w_sel,
                 uint16_t *__restrict__ ops, const bf16 *__restrict__ dt, const float *__restrict__ A, ChainTables tb, Shape s,
                 int nsteps, int gpb, int items)
{
    constexpr int RS = 64 * NT + 16;                     // row stride of the mixed rows (bytes)
    constexpr int PPR = 4 * NT;                          // 16-byte pieces of a row
    extern __shared__ __align__(16) unsigned char smem_raw[];
    __shared__ float s_mag[CB_MIX_THREADS / 64];         // largest value a wave has mixed
    unsigned char *s_rows[2] = {smem_raw, smem_raw + CB_STEP * RS};              // B, C
    int32_t *s_idx = reinterpret_cast<int32_t *>(smem_raw + 2 * CB_STEP * RS);   // [64][K]
    float *s_w = reinterpret_cast<float *>(s_idx + CB_STEP * s.K);               // [64][K]
    float *s_l = s_w + CB_STEP * s.K;                                            // [64][E|1]
    const int K = s.K, tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    if ((int)blockIdx.x >= items) {
        // tables: a wave takes eight heads of a step
        const int octets = (s.H + 7) / 8;
        const int unit = ((int)blockIdx.x - items) * (CB_MIX_THREADS / 64) + wave;
        const int h0 = 8 * (unit % octets), c = (unit / octets) % nsteps, b = unit / (octets * nsteps);
        if (b >= s.B) return;
        const int t = c * CB_STEP + lane;
        const bf16 *src = dt + ((int64_t)b * s.L + min(t, s.L - 1)) * s.H;
        uint16_t d[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) d[k] = src[min(h0 + k, s.H - 1)].bits;
#pragma unroll
        for (int k = 0; k < 8; ++k)
            if (h0 + k < s.H)
                chain_table(tb, ((int64_t)b * s.H + h0 + k) * nsteps + c, t < s.L ? bf_lo(d[k]) : 0.f, A[h0 + k] * LOG2E, lane);
        return;
    }
    const int gblocks = s.G / gpb;
    const int item = blockIdx.x;
    const int g_begin = (item % gblocks) * gpb;
    const int c = (item / gblocks) % nsteps;
    const int b = item / (gblocks * nsteps);
    const int valid = min(CB_STEP, s.L - c * CB_STEP);
    const int64_t tok0 = (int64_t)b * s.L + (int64_t)c * CB_STEP;
    const bool is_c = wave >= CB_MIX_THREADS / 128;

    if (!SEL) {
        const int ES = s.E | 1;
        for (int i = tid; i < valid * s.E; i += CB_MIX_THREADS) s_l[i / s.E * ES + i % s.E] = to_float(logits[tok0 * s.E + i]);
        __syncthreads();
    }
    if (tid < CB_STEP) {
        int32_t *ix = s_idx + tid * K;
        float *wx = s_w + tid * K;
        if (tid >= valid) {
            for (int r = 0; r < K; ++r) { ix[r] = 0; wx[r] = 0.f; }
        } else if (SEL) {
            for (int r = 0; r < K; ++r) { ix[r] = r; wx[r] = w_sel[(tok0 + tid) * K + r]; }
        } else {
            const float *row = s_l + tid * (s.E | 1);
            route_token([&](int e) { return row[e]; }, s.E, K, ix, wx);
            if (g_begin == 0)
                for (int r = 0; r < K; ++r) { idx_out[(tok0 + tid) * K + r] = ix[r]; w_out[(tok0 + tid) * K + r] = wx[r]; }
        }
    }
    __syncthreads();

    const int rowsE = SEL ? K : s.E;
    const int64_t estride = (int64_t)s.G * s.N, tokstride = rowsE * estride;
    const int l32 = lane & 31, hi = lane >> 5, s16 = lane & 15, half = (lane >> 4) & 1;
    for (int g = g_begin; g < g_begin + gpb; ++g) {
        // ---- mixed rows: units of 8 columns, NT a thread; waves 0..3 B rows, the others C rows ----
        {
            float acc[NT][8];
#pragma unroll
            for (int m = 0; m < NT; ++m)
#pragma unroll
                for (int q = 0; q < 8; ++q) acc[m][q] = 0.f;
            auto source = [&](int m, int r, float &w) __attribute__((always_inline)) {
                const int u = m * (CB_MIX_THREADS / 2) + tid % (CB_MIX_THREADS / 2), row = u / PPR, pc = u % PPR;
                const uint16_t *base = reinterpret_cast<const uint16_t *>(is_c ? Ce : Be);
                const int j = min(row, valid - 1);
                w = s_w[row * K + r];
                return base + (tok0 + j) * tokstride + s_idx[row * K + r] * estride + (int64_t)g * s.N + min(8 * pc, s.N - 8);
            };
            auto row_piece = [&](const uint16_t *p) __attribute__((always_inline)) { return ONCE ? load_nt(p) : *reinterpret_cast<const uint4 *>(p); };
            int r = 0;
            for (; r + 1 < K; r += 2) {
                uint4 v0[NT], v1[NT];
                float w0[NT], w1[NT];
#pragma unroll
                for (int m = 0; m < NT; ++m) {
                    v0[m] = row_piece(source(m, r, w0[m]));
                    v1[m] = row_piece(source(m, r + 1, w1[m]));
                }
#pragma unroll
                for (int m = 0; m < NT; ++m) {
                    fma_bf16x8(acc[m], v0[m], w0[m]);
                    fma_bf16x8(acc[m], v1[m], w1[m]);
                }
            }
            if (r < K) {
                uint4 v0[NT];
                float w0[NT];
#pragma unroll
                for (int m = 0; m < NT; ++m) v0[m] = row_piece(source(m, r, w0[m]));
#pragma unroll
                for (int m = 0; m < NT; ++m) fma_bf16x8(acc[m], v0[m], w0[m]);
            }
            float most = 0.f;
#pragma unroll
            for (int m = 0; m < NT; ++m) {
                const int u = m * (CB_MIX_THREADS / 2) + tid % (CB_MIX_THREADS / 2), row = u / PPR, pc = u % PPR;
                uint4 v = pack8(acc[m]);
                if (row >= valid || 8 * pc >= s.N) v = make_uint4(0, 0, 0, 0);
                *reinterpret_cast<uint4 *>(s_rows[is_c] + row * RS + 16 * pc) = v;
#pragma unroll
                for (int q = 0; q < 8; ++q) most = fmaxf(most, fabsf(acc[m][q]));
            }
            most = wave_max(most);
            if (lane == 63) s_mag[wave] = most;
        }
        __syncthreads();
        uint4 *dst = reinterpret_cast<uint4 *>(ops) + (((int64_t)b * nsteps + c) * s.G + g) * (cb_item_frags(NT) * 64) + lane;
        if (tid == CB_MIX_THREADS - 1) {                 // of a wave that makes no tile
            float b_most = 0.f, c_most = 0.f;
#pragma unroll
            for (int q = 0; q < CB_MIX_THREADS / 64; ++q) (q < CB_MIX_THREADS / 128 ? b_most : c_most) = fmaxf(q < CB_MIX_THREADS / 128 ? b_most : c_most, s_mag[q]);
            reinterpret_cast<float2 *>(tb.mag)[((int64_t)b * nsteps + c) * s.G + g] = mag_bounds(b_most, c_most);
        }
        if (wave < 3) {                                  // G^T tiles (I, J) = (0, 0), (1, 0), (1, 1)
            const int I = wave > 0, J = wave == 2;
            const unsigned char *br = s_rows[0] + (32 * J + l32) * RS + 16 * hi, *cr = s_rows[1] + (32 * I + l32) * RS + 16 * hi;
            f32x16_t acc = {0};
#pragma unroll
            for (int k = 0; k < 2 * NT; ++k)
                acc = mfma32(*reinterpret_cast<const uint4 *>(br + 32 * k), *reinterpret_cast<const uint4 *>(cr + 32 * k), acc);
            float m[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) {
                const int j = 8 * (v >> 2) + 4 * hi + (v & 3);
                m[v] = (wave == 1 || j <= l32) ? acc[v] : 0.f;
            }
            dst[(8 * NT + 2 * wave) * 64] = pack8(m);
            dst[(8 * NT + 2 * wave + 1) * 64] = pack8(m + 8);
        }
        for (int f = CB_MIX_THREADS / 64 - 1 - wave; f < 8 * NT; f += CB_MIX_THREADS / 64) {
            if (f < 4 * NT) {                            // C
                const unsigned char *cr = s_rows[1] + (32 * (f / (2 * NT)) + l32) * RS + 32 * (f % (2 * NT)) + 8 * hi;
                const uint2 a = *reinterpret_cast<const uint2 *>(cr), e = *reinterpret_cast<const uint2 *>(cr + 16);
                dst[f * 64] = make_uint4(a.x, a.y, e.x, e.y);
            } else {                                     // B, tokens innermost
                const int fb = f - 4 * NT;
                const unsigned char *br = s_rows[0] + (16 * (fb & 3) + 4 * hi + (s16 >> 2)) * RS + 64 * (fb >> 2) + 32 * half + 8 * (s16 & 3);
                const uint2 a = lds_read_tr(br), e = lds_read_tr(br + 8 * RS);
                dst[f * 64] = make_uint4(a.x, a.y, e.x, e.y);
            }
        }
        if (g + 1 < g_begin + gpb) __syncthreads();      // the next group's rows
    }
}

// 2^e, also where it is no normal number, times v
__device__ __forceinline__ float scale_exp2(float v, float frac, int whole) { return ldexpf(v * frac, whole); }
__device__ __forceinline__ void split_exp2(float e, float &frac, int &whole)
{
    const float c = e != e ? e : fminf(fmaxf(e, -1000.f), 1000.f), w = rintf(c);
    frac = fast_exp2(c - w);
    whole = (int)w;
}

// A sequence walked as segments.  A first launch (OUT = false: the state part alone) walks pieces of the segments in front of
// the last from a zero state, pieces to a segment, and writes what each leaves behind; a segment of the output launch starts from
// their sum, each decayed to its first token (the recurrence is linear in the state).
//   piece(q) (B, H, P tiles, NT, 4, 64, 4) fp32 accumulator registers; the first n_a pieces lie in a, the others in b
//   sum (B, H, npiece, 2)  log2 of a piece's decay; 1 where the piece is written.  With skip set one whose factor up to the
//                          segment's end is under 2^-150, a factor of zero in fp32, is not walked.  It is set where the split
//                          pass over whole chunks left the same out, so there an x that is not finite can end with its
//                          segment, as it did; elsewhere it reaches all that follows.
struct ChainPieces {
    float *a, *b, *sum, *h0_copy;
    int npiece, n_a, per_seg, steps, skip;
};
__device__ __forceinline__ float4 *piece_frag(const ChainPieces &pc, int64_t bh, int64_t nbh, int q, int ptiles, int ptile, int NT)
{
    float *base = q < pc.n_a ? pc.a + (q * nbh + bh) * (int64_t)(ptiles * NT * 1024) : pc.b + ((q - pc.n_a) * nbh + bh) * (int64_t)(ptiles * NT * 1024);
    return reinterpret_cast<float4 *>(base + ptile * NT * 1024);
}

// Waves of a workgroup of PT channel tiles that writes Y (CW > 0): CW / 2 of the state, CW / 2 readout, 2 PT i/o; of one that
// does not (CW = 0), a state wave for each channel tile and half of the columns, 2 PT i/o.
constexpr int cb_state_waves(int PT, int CW) { return CW ? CW / 2 : 2 * PT; }
constexpr int cb_threads(int PT, int CW) { return 64 * (cb_state_waves(PT, CW) + CW / 2 + 2 * PT); }

// XONCE: x passes by the caches.  Registers for two workgroups to a unit where no Y is written: the pieces of two sequences of
// 16384 tokens x 64 heads, 512 workgroups, are one round then (314 -> 309 us).  With operands loaded two steps ahead the 128
// registers of that are 21 too few at N = 128 (11 with one channel tile; one step ahead it was 106 without spills).  The walk of
// one channel tile on four waves is 3 short.
template <int NT, int PT, int CW, bool XONCE = false>
__global__ void __launch_bounds__(cb_threads(PT, CW), CW == 0 ? 4 : PT == 1 && CW == 4 ? 3 : 2)
chain_bf16_kernel(const uint16_t *__restrict__ x, const float *__restrict__ D, const uint16_t *__restrict__ ops, ChainTables tb,
                  const float *h0, float *h_final, uint16_t *__restrict__ y, Shape s, int nsteps, int nslice, int nseg,
                  int steps_per_seg, int hblock, ChainPieces pieces, int total, int nblocks)
{
    constexpr bool OUT = CW > 0;
    constexpr int SW = cb_state_waves(PT, CW), NW = SW + CW / 2, NIO = 2 * PT;
    constexpr int DEPTH = CW == 2 ? 1 : 2;               // steps that operands are loaded ahead of their use
    constexpr int XROW = 64 * PT;                        // bytes of an x row
    constexpr int XB = CB_STEP * XROW, YB = 2 * XB;      // bytes of an x tile, of a Y tile
    constexpr int HB = PT * NT * 2048;                   // bytes of the state, rounded
    constexpr int PPR = 4 * PT;                          // 16-byte pieces of an x row
    constexpr int YM = 8 * PT - 1;                       // 16-byte pieces of a Y row, less one
    extern __shared__ __align__(16) unsigned char smem_raw[];
    unsigned char *s_x = smem_raw;                       // [3] x rows times f, bf16
    unsigned char *s_xs = s_x + (OUT ? 3 * XB : 0);      // [3] of direct steps: x as the state takes it
    unsigned char *s_y = s_xs + 3 * XB;                  // [2] Y, fp32
    unsigned char *s_h = s_y + (OUT ? 2 * YB : 0);       // [2] the state at a step's reference as operand registers
    // [3] mode and references, 2^(part of cs_last), and a byte an i/o wave: x times its factor left its bounds
    int4 *s_ref = reinterpret_cast<int4 *>(s_h + (OUT ? 2 * HB : 0));
    int *s_whole = reinterpret_cast<int *>(s_ref + 3);   // [3][64] of direct steps: whole parts of cs

    const int lid = xcd_logical_id(blockIdx.x, nblocks);
    if (lid >= total) return;
    // consecutive ids, which share an XCD: the slices, heads and segments of a sequence, innermost first; of pieces hblock heads,
    // then the pieces, then the other heads, so that every XCD gets near and far ones of those that are not walked
    const int sl = lid % nslice, hl = lid / nslice % hblock;
    const int seg = lid / (nslice * hblock) % nseg;
    const int h = lid / (nslice * hblock * nseg) % (s.H / hblock) * hblock + hl;
    const int b = lid / (nslice * s.H * nseg);
    const int g = (h * s.G) / s.H;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, hi = lane >> 5;
    const int c_begin = seg * steps_per_seg, c_end = min(nsteps, c_begin + steps_per_seg);
    const int t_end = min(s.L, c_end * CB_STEP);         // of the segment
    const int p0 = 32 * PT * sl, P = s.P;
    const int64_t tokb = (int64_t)b * s.L, trow = (int64_t)s.H * P;
    const int64_t bhs = ((int64_t)b * s.H + h) * nsteps;
    const int64_t bh = (int64_t)b * s.H + h, nbh = (int64_t)s.B * s.H;
    const int ptiles = (P + 31) / 32;

    if (!OUT) {
        if (seg == 0 && pieces.h0_copy)                  // of this workgroup's channels
            for (int i = tid; i < min(32 * PT, P - p0) * s.N / 4; i += cb_threads(PT, CW))
                reinterpret_cast<float4 *>(pieces.h0_copy + (bh * P + p0) * s.N)[i] = reinterpret_cast<const float4 *>(h0 + (bh * P + p0) * s.N)[i];
        // decay of this piece, and from its end to the end of its segment
        const float *last = tb.sum + bhs;
        const int s_end = (seg / pieces.per_seg + 1) * pieces.per_seg * pieces.steps;
        float own = 0.f, after = 0.f;
        for (int c = c_begin + lane; c < c_end; c += 64) own += last[c];
        if (pieces.skip)
            for (int c = c_end + lane; c < s_end; c += 64) after += last[c];
        own = lane_value(wave_scan(own), 63);
        after = lane_value(wave_scan(after), 63);
        const bool dead = pieces.skip && after < -150.f;
        if (sl == 0 && tid == 0) reinterpret_cast<float2 *>(pieces.sum)[bh * pieces.npiece + seg] = make_float2(own, dead ? 0.f : 1.f);
        if (dead) return;
    }

    auto flagged = [&](int w) __attribute__((always_inline)) {
        return (__builtin_amdgcn_readfirstlane(w) & (PT == 2 ? ~0 : 0xffff)) != 0;
    };
    // two pieces of 8 channels of one token a thread of either role: tokens xj0 and xj0 + 32
    const int io = (tid - NW * 64) & (NIO * 64 - 1), xpc = io % PPR, xp = p0 + 8 * xpc, xj0 = io / PPR;
    const bool xin = xp < P;
    const int64_t xbase = tokb * trow + (int64_t)h * P;                  // uniform
    auto x_at = [&](int row, int pc) __attribute__((always_inline)) {    // where a piece of 8 channels of a token lies in its tile
        return row * XROW + (((pc >> 1) ^ (PT == 2 ? (row & 3) : ((row >> 1) & 1))) << 5) + ((pc & 1) << 4);
    };
    const float2 *fe0 = reinterpret_cast<const float2 *>(tb.fe) + bhs * CB_STEP;
    // x of a direct step: f holds dt and the part of cs, w is the whole of cs
    auto stage_direct = [&](int at, int row, int pc, const float (&a)[8], float f, int w, int last) __attribute__((always_inline)) {
        const float fs = ldexpf(f, last - w);
        float q[8];
#pragma unroll
        for (int e = 0; e < 8; ++e) q[e] = a[e] * fs;
        *reinterpret_cast<uint4 *>(s_xs + at * XB + x_at(row, pc)) = pack8(q);
        if (!OUT) return;
#pragma unroll
        for (int e = 0; e < 8; ++e) q[e] = a[e] * f;
        *reinterpret_cast<uint4 *>(s_x + at * XB + x_at(row, pc)) = pack8(q);
        if (pc == 0) s_whole[at * CB_STEP + row] = w;
    };
    // what a factor of y moves to that of x in a step turned direct: any whole number near its exponent
    auto exponent = [](float v) __attribute__((always_inline)) { return (int)rintf(__builtin_amdgcn_logf(v)); };
    // Step c, whose x has been staged in slot at, turned direct by the compute waves: one copy of this code, where the i/o
    // waves' steps are unrolled.
    auto turn_direct = [&](int c, int at, int &pack) __attribute__((always_inline)) {
        const int R0 = ref_r0(pack), R1 = R0 + ref_shift(pack), last = R1 + ref_rem(pack);
#pragma unroll 1
        for (int q = tid; q < CB_STEP * PPR; q += 64 * NW) {
            const int row = q / PPR, pc = q % PPR, tok = c * CB_STEP + row;
            float a[8];
            unpack8(a, p0 + 8 * pc < P && tok < t_end ? *reinterpret_cast<const uint4 *>(x + xbase + tok * trow + p0 + 8 * pc) : make_uint4(0, 0, 0, 0));
            const float2 fe = fe0[c * CB_STEP + 2 * (row & 31) + (row >> 5)];
            const int e = exponent(fe.y);
            stage_direct(at, row, pc, a, ldexpf(fe.x, e), (row < 32 ? R0 : R1) + e, last);
        }
        pack = pack_direct(last);
        lds_barrier();
    };

    // operand of k-step ks from the x rows: channels 32 ph + lane%32, tokens 16 ks + 4 hi + 0..3 and + 8
    const int s16 = lane & 15, r4 = s16 >> 2;
    auto read_x = [&](const unsigned char *base, int ph, int ks) __attribute__((always_inline)) {
        const int x_fr = (4 * hi + r4) * XROW + (((ph * 2 + ((lane >> 4) & 1)) ^ (PT == 2 ? r4 : (r4 >> 1))) << 5) + 8 * (s16 & 3);
        const unsigned char *q = base + x_fr + ks * 16 * XROW;
        const uint2 a = lds_read_tr(q), e = lds_read_tr(q + 8 * XROW);
        return make_uint4(a.x, a.y, e.x, e.y);
    };
    // rows of x and y of step c, at the first of which x0 points: nothing is read or written past the segment's end
    auto rows = [&](const uint16_t *x0, int c) __attribute__((always_inline)) {
        const int left = __builtin_amdgcn_readfirstlane(max(0, min(CB_STEP, t_end - c * CB_STEP)));
        return __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t *>(x0 + xbase + c * (CB_STEP * trow)), 0, left * (int)trow * 2, 0x27000);
    };
    const uint4 *item0 = reinterpret_cast<const uint4 *>(ops) + ((int64_t)b * nsteps * s.G + g) * (cb_item_frags(NT) * 64) + lane;
    const int64_t item_step = (int64_t)s.G * (cb_item_frags(NT) * 64);
    auto item = [&](int c) __attribute__((always_inline)) { return item0 + min(c, c_end - 1) * item_step; };

    // ================= state waves: the state's tiles, a part of its columns each =================
    auto state_wave = [&](int sw) __attribute__((always_inline)) {
        constexpr int PHW = OUT ? PT : 1;                // channel tiles
        constexpr int SPLIT = CW == 2 ? 1 : 2;           // waves that share the columns
        constexpr int NTS = NT > SPLIT ? NT / SPLIT : 1;
        const int nh = OUT ? sw : sw / PT, ph0 = OUT ? 0 : sw % PT;
        const bool on = nh * NTS < NT;                   // one tile: the second wave has none
        const int nt0 = on ? nh * NTS : 0;
        uint4 bfr[DEPTH][NTS][4], xf[PHW][4];
        auto load_b = [&](uint4 (&v)[NTS][4], int c) __attribute__((always_inline)) {
            // in the order of the steps' loads: the waits on them stay exact counts
            const uint4 *src = item(c) + (4 * NT + nt0 * 4) * 64;
#pragma unroll
            for (int i = 0; i < 4 * NTS; ++i) {
                const int j = i % (2 * NTS), k = i < 2 * NTS ? j % NTS : j / 2, ks = i < 2 * NTS ? j / NTS : 2 + j % 2;
                v[k][ks] = src[(k * 4 + ks) * 64];
                __builtin_amdgcn_sched_barrier(0);
            }
        };
        f32x16_t st[PHW][NTS];
        auto hoff = [&](int ph) __attribute__((always_inline)) {
            return (((int64_t)b * s.H + h) * P + min(p0 + 32 * (ph0 + ph) + l32, P - 1)) * s.N;
        };
#pragma unroll
        for (int ph = 0; ph < PHW; ++ph)
#pragma unroll
            for (int k = 0; k < NTS; ++k)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int n = 32 * (nt0 + k) + 8 * q + 4 * hi;
                    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
                    if (OUT && h0 && p0 + 32 * (ph0 + ph) + l32 < P && n < s.N) v = *reinterpret_cast<const float4 *>(h0 + hoff(ph) + n);
                    st[ph][k][4 * q] = v.x; st[ph][k][4 * q + 1] = v.y; st[ph][k][4 * q + 2] = v.z; st[ph][k][4 * q + 3] = v.w;
                }
        auto scale = [&](float f) __attribute__((always_inline)) {
#pragma unroll
            for (int ph = 0; ph < PHW; ++ph)
#pragma unroll
                for (int k = 0; k < NTS; ++k)
#pragma unroll
                    for (int v = 0; v < 16; ++v) st[ph][k][v] *= f;
        };
        if (OUT && seg > 0) {
            // lane l: the piece l pieces in front of the segment's first step, and its factor
            const int np = seg * pieces.per_seg;
            float2 sum = make_float2(0.f, 0.f);
            if (lane < np) sum = reinterpret_cast<const float2 *>(pieces.sum)[bh * pieces.npiece + np - 1 - lane];
            const float upto = wave_scan(sum.x);
            float e = __shfl_up(upto, 1);
            if (lane == 0) e = 0.f;
            const uint64_t live = __ballot(sum.y != 0.f && !(pieces.skip && e < -150.f));
            float frac;
            int whole;
            split_exp2(lane_value(upto, 63), frac, whole);
#pragma unroll
            for (int ph = 0; ph < PHW; ++ph)
#pragma unroll
                for (int k = 0; k < NTS; ++k)
#pragma unroll
                    for (int v = 0; v < 16; ++v) st[ph][k][v] = scale_exp2(st[ph][k][v], frac, whole);
#pragma unroll
            for (int ph = 0; ph < PHW; ++ph) {
                auto add = [&](int i, const float4 (&v)[NTS][4]) __attribute__((always_inline)) {
                    split_exp2(lane_value(e, i), frac, whole);
#pragma unroll
                    for (int k = 0; k < NTS; ++k)
#pragma unroll
                        for (int q = 0; q < 4; ++q) {
                            st[ph][k][4 * q + 0] += scale_exp2(v[k][q].x, frac, whole);
                            st[ph][k][4 * q + 1] += scale_exp2(v[k][q].y, frac, whole);
                            st[ph][k][4 * q + 2] += scale_exp2(v[k][q].z, frac, whole);
                            st[ph][k][4 * q + 3] += scale_exp2(v[k][q].w, frac, whole);
                        }
                };
                auto fetch = [&](int i, float4 (&v)[NTS][4]) __attribute__((always_inline)) {
                    const float4 *src = piece_frag(pieces, bh, nbh, np - 1 - i, ptiles, min(sl * PT + ph0 + ph, ptiles - 1), NT) + nt0 * 256 + lane;
#pragma unroll
                    for (int k = 0; k < NTS; ++k)
#pragma unroll
                        for (int q = 0; q < 4; ++q) v[k][q] = src[(k * 4 + q) * 64];
                };
                for (uint64_t todo = live; todo;) {      // two pieces in flight
                    float4 v0[NTS][4], v1[NTS][4];
                    const int i0 = 63 - __builtin_clzll(todo);
                    todo &= ~(1ull << i0);
                    fetch(i0, v0);
                    if (todo) {
                        const int i1 = 63 - __builtin_clzll(todo);
                        todo &= ~(1ull << i1);
                        fetch(i1, v1);
                        add(i0, v0);
                        add(i1, v1);
                    } else {
                        add(i0, v0);
                    }
                }
            }
        }
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) load_b(bfr[u], c_begin + u);
        unsigned char *h_wr = s_h + nt0 * 2048 + lane * 16;
        // the state at a step's reference, rounded, for the readout
        auto write_h = [&](int par, int ph, int k) __attribute__((always_inline)) {
            float m[16];
#pragma unroll
            for (int v = 0; v < 16; ++v) m[v] = st[ph][k][v];
            uint4 *dst = reinterpret_cast<uint4 *>(h_wr + par * HB + (ph * NT + k) * 2048);
            const uint4 a = pack8(m), e = pack8(m + 8);
            if (on) {
                dst[0] = a;
                dst[64] = e;
            }
        };
        lds_barrier();                                   // x of the first step, references of the first two
        int4 rc = s_ref[0];
        int pc = __builtin_amdgcn_readfirstlane(rc.x);
        if (__builtin_expect(flagged(rc.w), 0)) turn_direct(c_begin, 0, pc);
        scale(ldexpf(1.f, ref_r0(pc)));
        if (OUT) {
#pragma unroll
            for (int ph = 0; ph < PHW; ++ph)
#pragma unroll
                for (int k = 0; k < NTS; ++k) write_h(0, ph, k);
        }
        auto x_base = [&](int pack, int at) __attribute__((always_inline)) { return (ref_mode(pack) == 2 ? s_xs : s_x) + at * XB; };
        {
            const unsigned char *base = x_base(pc, 0);
#pragma unroll
            for (int ph = 0; ph < PHW; ++ph)
#pragma unroll
                for (int ks = 0; ks < 4; ++ks) xf[ph][ks] = read_x(base, ph0 + ph, ks);
        }
        int slot = 0;                                    // of x, references and whole parts
        auto step = [&](int c, uint4 (&bf)[NTS][4]) __attribute__((always_inline)) {
            lds_barrier();
            const int next_slot = slot == 2 ? 0 : slot + 1;
            const int4 rn = s_ref[next_slot];
            if (__builtin_expect(ref_mode(pc) == 2, 0)) scale(ldexpf(1.f, ref_shift(pc)));   // to the step's end
            const uint4 *next = item(c + DEPTH) + (4 * NT + nt0 * 4) * 64;
            // Memory instructions go out one behind each use of what they replace: a wave that issues them in a row waits
            // for the CU's address unit and LDS each time, with its matrix core idle.
#pragma unroll
            for (int ks = 0; ks < 2; ++ks)
#pragma unroll
                for (int k = 0; k < NTS; ++k) {
#pragma unroll
                    for (int ph = 0; ph < PHW; ++ph) st[ph][k] = mfma32(bf[k][ks], xf[ph][ks], st[ph][k]);
                    bf[k][ks] = next[(k * 4 + ks) * 64];
                    __builtin_amdgcn_sched_barrier(0);
                }
            if (__builtin_expect(ref_mode(pc) == 1, 0)) scale(ldexpf(1.f, ref_shift(pc)));   // to the reference of the other 32 tokens
            int pn = __builtin_amdgcn_readfirstlane(rn.x);
            if (__builtin_expect(flagged(rn.w), 0)) turn_direct(c + 1, next_slot, pn);
            const float sc = ldexpf(__int_as_float(rc.y), ref_rem(pc) + (c + 1 < c_end ? ref_r0(pn) : 0));
            const unsigned char *base = x_base(pn, next_slot);
#pragma unroll
            for (int ph = 0; ph < PHW; ++ph)
#pragma unroll
                for (int ks = 0; ks < 2; ++ks) xf[ph][ks] = read_x(base, ph0 + ph, ks);
            // the state at the reference of the next step, a tile's behind the matrix work of the next
            auto finish = [&](int i) __attribute__((always_inline)) {
                const int k = i / PHW, ph = i % PHW;
#pragma unroll
                for (int v = 0; v < 16; ++v) st[ph][k][v] *= sc;
                if (OUT) write_h((c + 1 - c_begin) & 1, ph, k);
            };
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NTS * PHW; ++i) {
                const int k = i / PHW, ph = i % PHW;
#pragma unroll
                for (int ks = 2; ks < 4; ++ks) {
                    st[ph][k] = mfma32(bf[k][ks], xf[ph][ks], st[ph][k]);
                    if (ph == PHW - 1) bf[k][ks] = next[(k * 4 + ks) * 64];
                }
                if (i == NTS * PHW - 1) {
#pragma unroll
                    for (int q = 0; q < PHW; ++q)
#pragma unroll
                        for (int ks = 2; ks < 4; ++ks) xf[q][ks] = read_x(base, ph0 + q, ks);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (i > 0) finish(i - 1);
                __builtin_amdgcn_sched_barrier(0);
            }
            finish(NTS * PHW - 1);
            rc = rn;
            pc = pn;
            slot = next_slot;
        };
        int c = c_begin;
        for (; c + DEPTH <= c_end; c += DEPTH) {         // no way from one of two operand sets to itself: the waits stay exact counts
            step(c, bfr[0]);
            if (DEPTH == 2) step(c + 1, bfr[DEPTH - 1]);
        }
        if (DEPTH == 2 && c < c_end) step(c, bfr[0]);
        lds_barrier();
        if (!on) return;
#pragma unroll
        for (int ph = 0; ph < PHW; ++ph) {
            if (!OUT && sl * PT + ph0 + ph < ptiles) {
                float4 *dst = piece_frag(pieces, bh, nbh, seg, ptiles, sl * PT + ph0 + ph, NT) + nt0 * 256 + lane;
#pragma unroll
                for (int k = 0; k < NTS; ++k)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        dst[(k * 4 + q) * 64] = make_float4(st[ph][k][4 * q], st[ph][k][4 * q + 1], st[ph][k][4 * q + 2], st[ph][k][4 * q + 3]);
            }
            if (OUT && h_final && seg == nseg - 1 && p0 + 32 * ph + l32 < P) {
#pragma unroll
                for (int k = 0; k < NTS; ++k)
#pragma unroll
                    for (int q = 0; q < 4; ++q) {
                        const int n = 32 * (nt0 + k) + 8 * q + 4 * hi;
                        if (n < s.N)
                            *reinterpret_cast<float4 *>(h_final + hoff(ph) + n) =
                                make_float4(st[ph][k][4 * q], st[ph][k][4 * q + 1], st[ph][k][4 * q + 2], st[ph][k][4 * q + 3]);
                    }
            }
        }
    };

    // ================= readout waves: Y of 32 tokens (one channel tile: of all 64), one step behind the state =================
    auto readout_wave = [&](auto first_) __attribute__((always_inline)) {
        constexpr int I0 = decltype(first_)::value, IW = CW == 2 ? 2 : 1;      // token tiles
        constexpr int GF = IW == 2 ? 6 : 2 + 2 * I0, G0 = 2 * I0;              // operands of the masked products, from G0 on
        constexpr int XK = I0 + IW == 2 ? 4 : 2;                               // k-steps of x
        uint4 cf[DEPTH][IW][2 * NT], gf[DEPTH][GF], xf[PT][4];
        auto load = [&](uint4 (&cv)[IW][2 * NT], uint4 (&gv)[GF], int c) __attribute__((always_inline)) {
            const uint4 *src = item(c);
#pragma unroll
            for (int k = 0; k < 2 * NT; ++k)
#pragma unroll
                for (int i = 0; i < IW; ++i) {
                    cv[i][k] = src[((I0 + i) * 2 * NT + k) * 64];
                    __builtin_amdgcn_sched_barrier(0);
                }
#pragma unroll
            for (int k = 0; k < GF; ++k) {
                gv[k] = src[(8 * NT + G0 + k) * 64];
                __builtin_amdgcn_sched_barrier(0);
            }
        };
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) load(cf[u], gf[u], c_begin + u);
        lds_barrier();
        int pc = __builtin_amdgcn_readfirstlane(s_ref[0].x);
        if (__builtin_expect(flagged(s_ref[0].w), 0)) turn_direct(c_begin, 0, pc);
        int slot = 0;
        auto read_all_x = [&](int at) __attribute__((always_inline)) {
#pragma unroll
            for (int ph = 0; ph < PT; ++ph)
#pragma unroll
                for (int ks = 0; ks < XK; ++ks) xf[ph][ks] = read_x(s_x + at * XB, ph, ks);
        };
        read_all_x(0);
        unsigned char *y_wr = s_y + (32 * I0 + l32) * (128 * PT);
        auto step = [&](int c, uint4 (&cv)[IW][2 * NT], uint4 (&gv)[GF]) __attribute__((always_inline)) {
            lds_barrier();
            const int next_slot = slot == 2 ? 0 : slot + 1, par = (c - c_begin) & 1;
            const int4 rn = s_ref[next_slot];
            const int mode = ref_mode(pc);
            const uint4 *hr = reinterpret_cast<const uint4 *>(s_h + par * HB) + lane;
            constexpr int HF = PT == 1 && NT == 4 ? 2 : NT;      // operands of the state in flight
            uint4 hf[HF];
#pragma unroll
            for (int k = 0; k < HF; ++k) hf[k] = hr[k * 64];
            int wi[IW] = {};
            if (__builtin_expect(mode == 2, 0)) {
                const int *whole = s_whole + slot * CB_STEP;
#pragma unroll
                for (int i = 0; i < IW; ++i) wi[i] = whole[32 * (I0 + i) + l32];
#pragma unroll
                for (int k = 0; k < GF; ++k) {
                    const int f = G0 + k, it = f >= 2, ks = it ? f - 2 : f;
                    const int4 w0 = *reinterpret_cast<const int4 *>(whole + 16 * ks + 4 * hi), w1 = *reinterpret_cast<const int4 *>(whole + 16 * ks + 8 + 4 * hi);
                    const int wj[8] = {w0.x, w0.y, w0.z, w0.w, w1.x, w1.y, w1.z, w1.w};
                    float m[8];
                    unpack8(m, gv[k]);
#pragma unroll
                    for (int e = 0; e < 8; ++e) m[e] = ldexpf(m[e], wi[it - I0] - wj[e]);
                    gv[k] = pack8(m);
                }
            }
            const uint4 *next = item(c + DEPTH);
            f32x16_t yt[PT][IW];
            auto write_y = [&](int ph, int i, int q) __attribute__((always_inline)) {
                *reinterpret_cast<float4 *>(y_wr + par * YB + i * 32 * 128 * PT + (((4 * ph + q + 4 * PT * hi) ^ (l32 & YM)) << 4)) =
                    make_float4(yt[ph][i][4 * q], yt[ph][i][4 * q + 1], yt[ph][i][4 * q + 2], yt[ph][i][4 * q + 3]);
            };
            // one channel tile after the other: the first goes to LDS behind the matrix work of the second
#pragma unroll
            for (int ph = 0; ph < PT; ++ph) {
#pragma unroll
                for (int i = 0; i < IW; ++i)
#pragma unroll
                    for (int v = 0; v < 16; ++v) yt[ph][i][v] = 0.f;
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int k = 0; k < 2 * NT; ++k) {
#pragma unroll
                    for (int i = 0; i < IW; ++i) {
                        yt[ph][i] = mfma32(hf[k % HF], cv[i][k], yt[ph][i]);
                        if (ph == PT - 1) cv[i][k] = next[((I0 + i) * 2 * NT + k) * 64];
                    }
                    if (ph < PT - 1 || k < 2 * NT - HF) hf[k % HF] = hr[(ph * 2 * NT + k + HF) * 64];
                    if (ph > 0 && k >= NT) write_y(ph - 1, 0, k - NT);           // NT = 4: the whole tile
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (__builtin_expect(mode == 2, 0)) {
#pragma unroll
                    for (int i = 0; i < IW; ++i)
#pragma unroll
                        for (int v = 0; v < 16; ++v) yt[ph][i][v] = ldexpf(yt[ph][i][v], wi[i]);
                }
                auto masked_products = [&](int half) __attribute__((always_inline)) {
#pragma unroll
                    for (int k = 0; k < GF; ++k) {
                        const int f = G0 + k, it = f >= 2, ks = it ? f - 2 : f;
                        if (ks / 2 == half) {
                            yt[ph][it - I0] = mfma32(xf[ph][ks], gv[k], yt[ph][it - I0]);
                            if (ph == PT - 1) gv[k] = next[(8 * NT + G0 + k) * 64];
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    }
                };
                masked_products(0);
                if constexpr (I0 + IW == 2) {
                    if (__builtin_expect(mode == 1, 0)) {
                        // from the reference of the first 32 tokens to that of the others
                        const float over = ldexpf(1.f, ref_shift(pc));
#pragma unroll
                        for (int v = 0; v < 16; ++v) yt[ph][IW - 1][v] *= over;
                    }
                    masked_products(1);
                }
            }
            int pn = __builtin_amdgcn_readfirstlane(rn.x);
            if (__builtin_expect(flagged(rn.w), 0)) turn_direct(c + 1, next_slot, pn);
            read_all_x(next_slot);
#pragma unroll
            for (int ph = 0; ph < PT; ++ph)
#pragma unroll
                for (int i = 0; i < IW; ++i)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        if (ph == PT - 1 || q >= NT) write_y(ph, i, q);
            pc = pn;
            slot = next_slot;
        };
        int c = c_begin;
        for (; c + DEPTH <= c_end; c += DEPTH) {         // no way from one of two operand sets to itself: the waits stay exact counts
            step(c, cf[0], gf[0]);
            if (DEPTH == 2) step(c + 1, cf[DEPTH - 1], gf[DEPTH - 1]);
        }
        if (DEPTH == 2 && c < c_end) step(c, cf[0], gf[0]);
        lds_barrier();
    };

    if (wave < SW) {
        state_wave(wave);
    } else if (wave < NW) {
        if (CW == 2 || wave == SW) readout_wave(std::integral_constant<int, 0>{});
        else readout_wave(std::integral_constant<int, CW == 2 ? 0 : 1>{});
    } else {
        // ================= i/o waves: two pieces of 8 channels of one token a thread =================
        const int iow = wave - NW;
        int xoff[2], yoff[2];
#pragma unroll
        for (int m = 0; m < 2; ++m) {
            const int row = (xj0 + 32 * m) * (int)trow;
            xoff[m] = (row + (xin ? xp : 0)) * 2;
            yoff[m] = xin ? (row + xp) * 2 : (int)0x80000000;
        }
        const float dsk = D ? D[h] : 0.f;
        const bool skip = D != nullptr;
        // x of step c, zeros past the segment's end, and its factors
        auto load_x = [&](u32x4_t (&v)[2], float4 &fe, int c) __attribute__((always_inline)) {
            const auto xrows = rows(x, c);
#pragma unroll
            for (int m = 0; m < 2; ++m) v[m] = __builtin_amdgcn_raw_buffer_load_b128(xrows, xoff[m], 0, XONCE ? 2 : 0);   // 2: non-temporal
            fe = reinterpret_cast<const float4 *>(fe0 + min(c, c_end - 1) * CB_STEP)[xj0];
        };
        auto unpack = [&](float (&a)[8], const u32x4_t &v) __attribute__((always_inline)) { unpack8(a, make_uint4(v[0], v[1], v[2], v[3])); };
        // x of step c (v) times its factor into LDS; of a direct step two copies, and fe turns into the factors.  Channels past
        // P hold something else's x, for rows of Y and columns of the state that go nowhere.
        auto stage_x = [&](int c, int at, const u32x4_t (&v)[2], float4 &fe, const cb_f32x4_t &ref) __attribute__((always_inline)) {
            const int p = __float_as_int(ref[0]), left = t_end - c * CB_STEP;
            uint64_t in = ~0ull;
            if (__builtin_expect(ref_mode(p) == 2, 0)) {
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    float &f = m ? fe.z : fe.x, &e = m ? fe.w : fe.y;
                    const float cs = e, whole = rintf(cs), part = cs - whole;
                    f = cs == cs ? f * fast_exp2(-part) : 0.f;
                    e = fast_exp2(part);
                    float a[8];
                    unpack(a, v[m]);
                    stage_direct(at, xj0 + 32 * m, xpc, a, f, (int)whole, ref_shift(p));   // 0 of NaN
                }
            } else {
                float most[2] = {0.f, 0.f};
#pragma unroll
                for (int m = 0; m < 2; ++m) {
                    float a[8];
                    unpack(a, v[m]);
#pragma unroll
                    for (int q = 0; q < 8; ++q) a[q] *= m ? fe.z : fe.x;
#pragma unroll
                    for (int q = 0; q < 8; ++q) most[m] = fmaxf(most[m], fabsf(a[q]));
                    *reinterpret_cast<uint4 *>(s_x + at * XB + x_at(xj0, xpc) + m * 32 * XROW) = pack8(a);
                }
                if (__builtin_expect(left < CB_STEP, 0)) {
#pragma unroll
                    for (int m = 0; m < 2; ++m)
                        if (xj0 + 32 * m >= left) most[m] = ref[2];
                }
                const bool wide = ref_mode(p) == 1 || ref_r0(p) < -(int)CB_NEAR / 2;
                in = __ballot(fminf(most[0], most[1]) >= (wide ? ref[2] : -1.f) && fmaxf(most[0], most[1]) <= ref[3]);
            }
            reinterpret_cast<unsigned char *>(&s_ref[at].w)[iow] = left > 0 && in != ~0ull;
        };
        const int ya0 = xj0 * (128 * PT) + ((xpc ^ (xj0 & YM)) << 4), ya1 = xj0 * (128 * PT) + (((xpc + 4 * PT) ^ (xj0 & YM)) << 4);
        // stages step c + 2 (xn) and finishes step c - 1 (xo)
        auto pass = [&](int c, int at, const u32x4_t (&xn)[2], float4 &fn, const cb_f32x4_t &rn, const u32x4_t (&xo)[2], const float4 &fo, int ybuf) __attribute__((always_inline)) {
            if (!OUT) {
                stage_x(c + 2, at, xn, fn, rn);
                return;
            }
            const unsigned char *q = s_y + ybuf * YB;
            float4 v[2][2];
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                v[m][0] = *reinterpret_cast<const float4 *>(q + ya0 + m * 32 * 128 * PT);
                v[m][1] = *reinterpret_cast<const float4 *>(q + ya1 + m * 32 * 128 * PT);
            }
            stage_x(c + 2, at, xn, fn, rn);
            const auto yrows = rows(y, c > c_begin ? c - 1 : nsteps);    // no step in front of the first
#pragma unroll
            for (int m = 0; m < 2; ++m) {
                const float e = m ? fo.w : fo.y;
                float r[8] = {v[m][0].x * e, v[m][0].y * e, v[m][0].z * e, v[m][0].w * e, v[m][1].x * e, v[m][1].y * e, v[m][1].z * e, v[m][1].w * e};
                if (skip) {
                    float a[8];
                    unpack(a, xo[m]);
#pragma unroll
                    for (int k = 0; k < 8; ++k) r[k] += dsk * a[k];
                }
                const uint4 o = pack8(r);
                __builtin_amdgcn_raw_buffer_store_b128(u32x4_t{o.x, o.y, o.z, o.w}, yrows, yoff[m], 0, 2);
            }
        };
        // x of step k in xr[(k - c_begin) % CB_RING]: loaded CB_RING - 3 steps before it is staged, kept until its y goes out
        u32x4_t xr[CB_RING][2];
        float4 fr[CB_RING];
        // what all lanes take of a step comes through the scalar cache
        const cb_scalar_f32x2_t *refs = (const cb_scalar_f32x2_t *)tb.ref + bhs, *mags = (const cb_scalar_f32x2_t *)tb.mag + (int64_t)b * nsteps * s.G + g;
        auto load_ref = [&](int c) __attribute__((always_inline)) -> cb_f32x4_t {
            c = min(c, c_end - 1);
            const cb_f32x2_t r = refs[c], m = mags[(int64_t)c * s.G];
            return cb_f32x4_t{r.x, r.y, m.x, m.y};
        };
        auto put_ref = [&](int at, const cb_f32x4_t &r) __attribute__((always_inline)) {
            if (iow == 0) *reinterpret_cast<float2 *>(s_ref + at) = make_float2(r[0], r[1]);
        };
        const cb_f32x4_t first = load_ref(c_begin), second = load_ref(c_begin + 1);
        cb_f32x4_t after = load_ref(c_begin + 2);
#pragma unroll
        for (int u = 0; u < CB_RING - 1; ++u) load_x(xr[u], fr[u], c_begin + u);
        put_ref(0, first);
        put_ref(1, second);
        stage_x(c_begin, 0, xr[0], fr[0], first);
        lds_barrier();                                   // x of the first step
        // a step that the compute waves turn direct: its factor of y, and the barrier in turn_direct
        auto turned = [&](float4 &fe) __attribute__((always_inline)) {
            fe.y = ldexpf(fe.y, -exponent(fe.y));
            fe.w = ldexpf(fe.w, -exponent(fe.w));
            lds_barrier();
        };
        if (__builtin_expect(flagged(s_ref[0].w), 0)) turned(fr[0]);
        stage_x(c_begin + 1, 1, xr[1], fr[1], second);   // beside the first readout
        for (int c0 = c_begin;; c0 += CB_RING) {
#pragma unroll
            for (int u = 0; u < CB_RING; ++u) {
                const int c = c0 + u, n1 = (u + 1) % CB_RING, n2 = (u + 2) % CB_RING, o = (u + CB_RING - 1) % CB_RING;
                lds_barrier();
                const int next = s_ref[(u + 1) % 3].w;
                const cb_f32x4_t later = load_ref(c + 3);
                pass(c, (u + 2) % 3, xr[n2], fr[n2], after, xr[o], fr[o], (u + 1) & 1);
                if (c >= c_end) return;
                put_ref((u + 2) % 3, after);
                load_x(xr[o], fr[o], c + CB_RING - 1);
                after = later;
                if (__builtin_expect(flagged(next), 0)) turned(fr[n1]);
            }
        }
    }
}

size_t chain_bf16_table_bytes(const Shape &s)
{
    return (size_t)s.B * ((s.L + CB_STEP - 1) / CB_STEP) * (s.H * (size_t)(2 * CB_STEP + 4) + 2 * s.G) * sizeof(float);
}

// Segments of a sequence, before the scratch is asked how many pieces it holds.  A compute unit takes 1.35 us for a step of a
// head when all are busy, and a chain alone 0.7 a step, so short of a quarter as many chains as units the chip idles: as many
// segments as fill it, of at least 12 steps each, or 8 where it stays half empty (us; 24 chains of 256 steps: 1 segment 183, 5
// 76, 10 68; 64 of 64: 56, 4 segments 47.6; 8 of 256: 179, 16 45).  With less work than nine steps a unit and less than 160
// steps the kernels that parallelise over chunks are taken, segments / those: 48 chains of 40 36.2 / 34.8, 32 of 64 38.6 / 36.8,
// 16 of 128 40.0 / 41.9, 8 of 128 33.7 / 34.3; past the line 48 of 48 40.0 / 44.5, 32 of 72 42.4 / 46.2, 8 of 217 41.2 / 48.7.
// From a quarter as many chains on the extra launch pays from 128 steps on (1 segment / 2: 128 of 128 144 / 126, of 256 275 / 232,
// 128 of 64 62 / 69, 96 of 64 58 / 64), and two rounds of more segments where these are fuller by a sixth than one: of 96 chains,
// 2 segments / 5, 256 steps 230 / 228, 160 156 / 159, 128 119 / 129, so that it gains only at the longest.  Chains that fill three
// fifths of a round stay whole (156 of 200: 238, 2 segments 314); 144 of 200, just short of that, are cut and lose (236, 3
// segments 271).
int chain_bf16_segments(int64_t chains, int64_t steps, int64_t ncu)
{
    if (steps <= 32 || chains == 0 || 10 * chains >= 6 * ncu || (chains * steps < 9 * ncu && steps < 160)) return 1;
    const int64_t one = ncu / chains, two = 2 * ncu / chains;
    if (4 * chains <= ncu) return (int)std::min<int64_t>({one, 16, chains * (steps / 8) <= ncu / 2 ? steps / 8 : steps / 12});
    if (steps < (one > 1 ? 128 : 96)) return 1;
    return (int)(6 * two >= 14 * one && steps >= 24 * two ? two : one);
}

static int chain_tiles(const Shape &s) { return s.N > 64 ? 4 : s.N > 32 ? 2 : 1; }
// bytes of what one piece of a sequence leaves behind, of all (batch, head)
static size_t chain_piece_bytes(const Shape &s) { return (size_t)s.B * s.H * ((s.P + 31) / 32) * chain_tiles(s) * 4096; }

struct ChainPlan {
    int nsteps, nseg, steps_per_seg;
    ChainPieces pieces;
};
static ChainPlan chain_plan(const Shape &s, const ChainScratch &scr, bool skip, int ncu)
{
    const int nsteps = (s.L + CB_STEP - 1) / CB_STEP;
    // pieces that the scratch holds, one place kept for a copy of h0
    const size_t unit = chain_piece_bytes(s);
    ChainPieces pieces = {scr.a, scr.b, scr.sum, nullptr, 0, (int)std::min(scr.a_bytes / unit, (size_t)64), 1, nsteps, skip};
    const int cap = (int)std::min(pieces.n_a + scr.b_bytes / unit, (size_t)65) - 1;
    // A piece is about 32 steps at most: enough pieces to fill the chip where a segment is long.
    int nseg = chain_bf16_segments((int64_t)s.B * s.H, nsteps, ncu), steps_per_seg = nsteps;
    for (; nseg > 1; --nseg) {
        pieces.per_seg = std::max(1, (nsteps / nseg + 16) / 32);
        pieces.steps = (nsteps + nseg * pieces.per_seg - 1) / (nseg * pieces.per_seg);
        steps_per_seg = pieces.steps * pieces.per_seg;
        if ((nsteps + steps_per_seg - 1) / steps_per_seg <= nseg) nseg = (nsteps + steps_per_seg - 1) / steps_per_seg;
        if ((nseg - 1) * pieces.per_seg <= cap) break;
    }
    if (nseg == 1) steps_per_seg = nsteps;
    pieces.npiece = (nseg - 1) * pieces.per_seg;
    return {nsteps, nseg, steps_per_seg, pieces};
}
int chain_bf16_planned_segments(const Shape &s, const ChainScratch &scr, int ncu) { return chain_plan(s, scr, false, ncu).nseg; }

static ChainTables chain_tables(const Shape &s, const ChainScratch &scr)
{
    const int64_t bhs = (int64_t)s.B * s.H * ((s.L + CB_STEP - 1) / CB_STEP);
    float *t = (float *)scr.tables;
    return {t, t + bhs * 2 * CB_STEP, t + bhs * (2 * CB_STEP + 2), t + (bhs * (2 * CB_STEP + 3) + 1) / 2 * 2};
}

// more than 64 KB of dynamic LDS has to be allowed once per device and kernel; done holds one bit per device ordinal
static swimba_status allow_lds(std::atomic<uint64_t> &done, std::initializer_list<std::pair<const void *, size_t>> kernels)
{
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    const uint64_t bit = 1ull << (dev & 63);
    if (e == hipSuccess && (done.load(std::memory_order_acquire) & bit)) return SWIMBA_OK;
    for (const auto &k : kernels)
        if (e == hipSuccess) e = hipFuncSetAttribute(k.first, hipFuncAttributeMaxDynamicSharedMemorySize, (int)k.second);
    if (e != hipSuccess) { set_last_hip_error((int)e); return SWIMBA_ERR_HIP; }
    done.fetch_or(bit, std::memory_order_release);
    return SWIMBA_OK;
}

template <int NT>
static swimba_status launch_mix_t(const Shape &s, const void *dt, const float *A, const void *Be, const void *Ce, const void *logits,
                                  const float *w_sel, int32_t *idx, float *w, const ChainScratch &scr, hipStream_t st)
{
    const int nsteps = (s.L + CB_STEP - 1) / CB_STEP, ncu = device_cus();
    auto mix_shm = [](int K, int E) { return (size_t)2 * CB_STEP * (64 * NT + 16) + (size_t)CB_STEP * K * 8 + (E ? (size_t)CB_STEP * (E | 1) * 4 : 0); };
    static std::atomic<uint64_t> done{0};
    const swimba_status ok = allow_lds(done, {{(const void *)mix_steps_kernel<NT, false, true>, mix_shm(SWIMBA_MAX_TOPK, SWIMBA_MAX_EXPERTS)},
                                              {(const void *)mix_steps_kernel<NT, false, NT == 4>, mix_shm(SWIMBA_MAX_TOPK, SWIMBA_MAX_EXPERTS)},
                                              {(const void *)mix_steps_kernel<NT, true, false>, mix_shm(SWIMBA_MAX_TOPK, 0)}});
    if (ok != SWIMBA_OK) return ok;
    // A workgroup routes its tokens once for as many groups as leave two workgroups to a compute unit.
    int gpb = 1;
    for (int n = 2; n <= s.G; ++n)
        if (s.G % n == 0 && (int64_t)s.B * nsteps * s.G / n >= 2 * (int64_t)ncu) gpb = n;
    const int items = (int)((int64_t)s.B * nsteps * s.G / gpb);
    const int tblocks = (int)(((int64_t)s.B * nsteps * ((s.H + 7) / 8) + 7) / 8);
    // The experts' rows are read once and pass by the last-level cache (256 MB), which keeps x and the operands: of this call, or
    // of calls on a few sets of inputs in turn, where these fit it then.  Plain loads / past the cache, us, 8 sequences x 24 heads
    // x 2048 tokens, one group: one and two sets of inputs level (43.9 / 44.0), three 51.6 / 44.0, four and more 53.3 / 52.8; eight
    // groups 85 / 77 and 97.6 / 90.3; two sequences of 16384 x 64 heads 312 / 306 with any.
    // Rows of less than a line share it with other groups, for which it is fetched again: one, three and eight sets, N = 16 in
    // eight groups 42.4 / 50.0, 52.8 / 58.8, 52.9 / 59.0, N = 48 56.1 / 61.1, 67.8 / 72.9, 68.0 / 73.6 (N = 64 54.5 / 56.1,
    // 68.6 / 68.2, 69.1 / 68.5).  In four groups that counts for less, and three sets gain more: N = 16 38.5 / 41.4, 47.0 / 41.0,
    // 48.6 / 50.9, N = 48 45.2 / 47.5, 57.5 / 50.8, 58.0 / 59.3.
    // Selected rows have just been written by the projection.
    const bool once = !(s.N < 64 && s.G >= 8);
    const auto kernel = w_sel ? mix_steps_kernel<NT, true, false> : once ? mix_steps_kernel<NT, false, true> : mix_steps_kernel<NT, false, NT == 4>;
    hipLaunchKernelGGL(kernel, dim3(items + tblocks), dim3(CB_MIX_THREADS), mix_shm(s.K, w_sel ? 0 : s.E), st,
                       (const bf16 *)Be, (const bf16 *)Ce, (const bf16 *)logits, idx, w, w_sel, (uint16_t *)scr.ops,
                       (const bf16 *)dt, A, chain_tables(s, scr), s, nsteps, gpb, items);
    SWIMBA_CHECK_LAUNCH();
    return SWIMBA_OK;
}

template <int NT>
static swimba_status launch_walk_t(const Shape &s, const void *x, const float *D, const float *h0, void *y, float *h_final,
                                   const ChainScratch &scr, bool skip, hipStream_t st)
{
    const int ncu = std::max(device_cus(), 1);
    auto chain_shm = [](int PT, bool out) { return (size_t)(out ? 10 + NT : 3) * CB_STEP * 64 * PT + 48 + (out ? 12 * CB_STEP : 0); };
    static std::atomic<uint64_t> done{0};
    const swimba_status ok = allow_lds(done, {{(const void *)chain_bf16_kernel<NT, 1, 2>, chain_shm(1, true)},
                                              {(const void *)chain_bf16_kernel<NT, 1, 4>, chain_shm(1, true)},
                                              {(const void *)chain_bf16_kernel<NT, 2, 4>, chain_shm(2, true)},
                                              {(const void *)chain_bf16_kernel<NT, 2, 4, true>, chain_shm(2, true)}});
    if (ok != SWIMBA_OK) return ok;
    ChainPlan plan = chain_plan(s, scr, skip, ncu);
    ChainPieces &pieces = plan.pieces;
    const size_t unit = chain_piece_bytes(s);
    int hblock = std::min(s.H, 8);
    while (s.H % hblock) --hblock;
    // Workgroups of one channel tile where all of them find a compute unit at once; else of both tiles of a head, one to a unit,
    // where the heads fill one round or three fifths of several; else (300 heads of 1024 tokens 45 / 48 us with both tiles in
    // one), and for more heads of one tile than units (320 of 512 tokens, P = 64, N = 64: 29 / 38), of fewer waves, two to a unit.
    // x and y that fill the last-level cache (256 MB) by themselves: x passes by it, unless pieces of it are walked twice (two
    // sequences of 16384 tokens 309 -> 320 us).  On four and more sets of inputs in turn it is not found there, and passing by is
    // ahead (x and y of 134 MB 57.7 -> 55.1 us, 201 MB 80.0 -> 77.7, 268 MB, the 370M-shaped layer, 100.4 -> 98.2, 402 MB 146.3 ->
    // 143.9, 537 MB 190.8 -> 187.9).  An x that the cache still holds, because nothing else ran since it was written or read, is
    // lost with it (one set of inputs again and again: 134 MB 48.8 -> 58.5, 201 MB 69 -> 80, 268 MB 87 -> 99, 402 MB 135 -> 144, 537 MB
    // 189 -> 187).  The line lies where what a program ran before has left the less of x the larger it is.
    const bool x_once = plan.nseg == 1 && (int64_t)s.B * s.L * s.H * s.P * 4 >= 256 << 20;
    auto launch = [&](bool out, int count, int steps) {
        const int64_t chains = (int64_t)s.B * s.H * count, rounds = (chains + ncu - 1) / ncu;
        const int PT = s.P > 32 && 2 * chains > ncu && (rounds == 1 || 10 * chains >= 6 * rounds * ncu) ? 2 : 1;
        const int CW = !out ? 0 : PT == 1 && chains * ((s.P + 31) / 32) > ncu ? 2 : 4;
        const int nslice = (s.P + 32 * PT - 1) / (32 * PT);
        const int total = (int)chains * nslice, nblocks = xcd_padded(total);
        const auto kernel = PT == 2 ? (!out ? chain_bf16_kernel<NT, 2, 0> : x_once ? chain_bf16_kernel<NT, 2, 4, true> : chain_bf16_kernel<NT, 2, 4>)
                                    : CW == 4 ? chain_bf16_kernel<NT, 1, 4> : CW == 2 ? chain_bf16_kernel<NT, 1, 2> : chain_bf16_kernel<NT, 1, 0>;
        hipLaunchKernelGGL(kernel, dim3(nblocks), dim3(cb_threads(PT, CW)), chain_shm(PT, out), st, (const uint16_t *)x, D,
                           (const uint16_t *)scr.ops, chain_tables(s, scr), h0, h_final, (uint16_t *)y, s, plan.nsteps, nslice, count, steps,
                           out ? s.H : hblock, pieces, total, nblocks);
    };
    if (plan.nseg > 1) {
        // with the final state written over the initial one the first segment can start after the last one has ended
        if (h0 && h0 == h_final)
            pieces.h0_copy = pieces.npiece < pieces.n_a ? scr.a + pieces.npiece * (unit / 4) : scr.b + (pieces.npiece - pieces.n_a) * (unit / 4);
        launch(false, pieces.npiece, pieces.steps);
        SWIMBA_CHECK_LAUNCH();
        if (pieces.h0_copy) h0 = pieces.h0_copy;
    }
    launch(true, plan.nseg, plan.steps_per_seg);
    SWIMBA_CHECK_LAUNCH();
    return SWIMBA_OK;
}

swimba_status launch_chain_mix_bf16(const Shape &s, const void *dt, const float *A, const void *Be, const void *Ce, const void *logits,
                                    const float *w_sel, int32_t *idx, float *w, const ChainScratch &scr, hipStream_t st)
{
    const int NT = chain_tiles(s);
    return (NT == 4 ? launch_mix_t<4> : NT == 2 ? launch_mix_t<2> : launch_mix_t<1>)(s, dt, A, Be, Ce, logits, w_sel, idx, w, scr, st);
}
swimba_status launch_chain_walk_bf16(const Shape &s, const void *x, const float *D, const float *h0, void *y, float *h_final,
                                     const ChainScratch &scr, bool skip, hipStream_t st)
{
    const int NT = chain_tiles(s);
    return (NT == 4 ? launch_walk_t<4> : NT == 2 ? launch_walk_t<2> : launch_walk_t<1>)(s, x, D, h0, y, h_final, scr, skip, st);
}
swimba_status launch_chain_bf16(const Shape &s, const void *x, const void *dt, const float *A, const float *D, const void *Be,
                                const void *Ce, const void *logits, const float *w_sel, const float *h0, void *y,
                                float *h_final, int32_t *idx, float *w, const ChainScratch &scr, bool skip, hipStream_t st)
{
    const swimba_status ok = launch_chain_mix_bf16(s, dt, A, Be, Ce, logits, w_sel, idx, w, scr, st);
    return ok == SWIMBA_OK ? launch_chain_walk_bf16(s, x, D, h0, y, h_final, scr, skip, st) : ok;
}

}  // namespace swimba
