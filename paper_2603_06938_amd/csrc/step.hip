// Recurrent decode step of one or a few tokens per sequence (paper: selective SSM recurrence per channel,
// with the router-mixed injection and readout of Theorem 1).  One launch where the state size is a
// power of two and a row of lanes holds a token's logits (up to 16 experts): every block routes and mixes
// its tokens while its piece of the fp32 state is on its way in, applies them to it and writes it back.
// More experts: the same kernel behind a small one that routes and mixes (fp32 rows in the caller's
// workspace).  Other state sizes: that small kernel and one update launch per token.
#include "common.hpp"

#include <atomic>
#include <type_traits>

namespace swimba {

// Scratch of swimba_step_static, the decode step for callers that cannot provide (or allocate) a
// workspace: the mixed B and C rows of one step, B*G*2N fp32.  One copy per GPU the library runs
// on, held until the process ends.  In host code the array's name is only a handle for
// hipGetSymbolAddress; kernels and copies get the address that call returns for the current device.
static __device__ __align__(256) float scratch[SWIMBA_STATIC_SCRATCH_BYTES / sizeof(float)];

constexpr int STEP_THREADS = 256;
typedef float __attribute__((ext_vector_type(4))) f32x4_t;

// ---- routing + mixing: block = (b, g), mixed (B; C) rows of N fp32 each ------------------
template <typename T>
__global__ void __launch_bounds__(128)
step_mix_kernel(const T *__restrict__ Be, const T *__restrict__ Ce, const T *__restrict__ logits,
                float *__restrict__ bc, int32_t *__restrict__ idx_out, Shape s)
{
    __shared__ float s_w[SWIMBA_MAX_TOPK];
    __shared__ int32_t s_idx[SWIMBA_MAX_TOPK];
    const int b = blockIdx.x / s.G, g = blockIdx.x % s.G;
    const int tid = threadIdx.x;
    // the logits go through LDS first: one memory latency instead of one per pass of the router
    __shared__ float s_log[SWIMBA_MAX_EXPERTS];
    for (int e = tid; e < s.E; e += 128) s_log[e] = to_float(logits[(int64_t)b * s.E + e]);
    __syncthreads();
    if (tid == 0) route_token([&](int e) { return s_log[e]; }, s.E, s.K, s_idx, s_w);
    __syncthreads();
    if (idx_out && g == 0 && tid < s.K) idx_out[(int64_t)b * s.K + tid] = s_idx[tid];
    const T *Bb = Be + ((int64_t)b * s.E * s.G + g) * s.N;
    const T *Cb = Ce + ((int64_t)b * s.E * s.G + g) * s.N;
    float *out = bc + (int64_t)blockIdx.x * 2 * s.N;
    for (int n = tid; n < s.N; n += 128) {
        float bm = 0.f, cm = 0.f;
        for (int r = 0; r < s.K; ++r) {
            const int64_t o = (int64_t)s_idx[r] * s.G * s.N + n;
            bm += s_w[r] * to_float(Bb[o]);
            cm += s_w[r] * to_float(Cb[o]);
        }
        out[n] = bm;
        out[s.N + n] = cm;
    }
}

// ---- one launch: routing, mixing and update -----------------------------------------------
// Exchange of a butterfly step at distance D: returns the partner's value.  The partner of lane i is i ^ D,
// except for D = 4, where it is i ^ 7 (row_half_mirror); together with the steps at 2 and 1 that reaches
// the same eight lanes.  Register moves (DPP), no LDS pass.
template <int D>
__device__ __forceinline__ float lane_partner(float v)
{
    static_assert(D == 1 || D == 2 || D == 4 || D == 8, "distances inside a row of 16 lanes");
    constexpr int ctrl = D == 1 ? 0xB1 : D == 2 ? 0x4E : D == 4 ? 0x141 : 0x128;   // quad_perm, half mirror, row_ror:8
    return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), ctrl, 0xf, 0xf, true));
}
// v0 of the lanes with bit D clear and v1 of those with it set, each plus the partner's value of the same sum
template <int D>
__device__ __forceinline__ float halve(float v0, float v1, int lane)
{
    if constexpr (D >= 16) {
        const auto r = D == 16 ? __builtin_amdgcn_permlane16_swap(__float_as_uint(v0), __float_as_uint(v1), false, false)
                               : __builtin_amdgcn_permlane32_swap(__float_as_uint(v0), __float_as_uint(v1), false, false);
        return __uint_as_float(r[0]) + __uint_as_float(r[1]);
    } else {
        const bool hi = (lane & D) != 0;
        return (hi ? v1 : v0) + lane_partner<D>(hi ? v0 : v1);
    }
}
// Sums over groups of 2D lanes of NV values per lane: every step halves the values a lane carries while there
// are several.  Value i ends on the lanes whose bits from D downwards spell i, most significant first.
template <int D, int NV>
__device__ __forceinline__ float group_sums(const float (&v)[NV], int lane)
{
    if constexpr (D == 0) {
        static_assert(NV == 1, "");
        return v[0];
    } else if constexpr (NV == 1) {
        const float w[1] = {halve<D>(v[0], v[0], lane)};
        return group_sums<D / 2>(w, lane);
    } else {
        float w[NV / 2];
#pragma unroll
        for (int j = 0; j < NV / 2; ++j) w[j] = halve<D>(v[j], v[NV / 2 + j], lane);
        return group_sums<D / 2>(w, lane);
    }
}

// Router of one token inside a row of 16 lanes: lane e holds logit e (-inf past E; E <= 16).  Same order
// and arithmetic as route_token up to the order of the sum over experts; picks come back in every lane.
constexpr int STEP_FUSED_EXPERTS = 16, STEP_FUSED_TOKENS = 16;
__device__ __forceinline__ void route_row16(float v, int lane, int E, int K, int32_t *idx, float *w)
{
    const int e = lane & 15;
    auto max_row = [](float m) {
        m = fmaxf(m, lane_partner<8>(m));
        m = fmaxf(m, lane_partner<4>(m));
        m = fmaxf(m, lane_partner<2>(m));
        return fmaxf(m, lane_partner<1>(m));
    };
    const float m = max_row(v);
    const float one[1] = {e < E ? route_exp(v - m) : 0.f};
    const float invZ = 1.0f / group_sums<8>(one, lane);
    bool open = e < E;   // not picked yet
    for (int r = 0; r < K; ++r) {
        // largest open logit, then the lowest index that has it
        const float bv = max_row(open ? v : -INFINITY);
        // ballots of the row this lane is in; only logits outside the contract (NaN) leave no lane with bv,
        // and then the index is still a valid, open one
        const uint32_t row = (uint32_t)(__ballot(open && v == bv) >> (lane & 48)) & 0xffffu;
        const uint32_t left = (uint32_t)(__ballot(open) >> (lane & 48)) & 0xffffu;
        const int best = __ffs(row ? row : left) - 1;
        if (e == best) open = false;
        if (e == 0) {
            idx[r] = best;
            w[r] = route_exp(bv - m) * invZ;
        }
    }
}

// Block = (b, h, slice of R * 256 / (N/4) state rows); lane -> 4 columns of R rows, held in registers over
// the L tokens, so the state crosses memory once in each direction.  Every block routes and mixes its
// sequence's tokens itself (rows of a group's B and C come from L2 for all but the first head); the state
// loads are issued before that chain and the latency of both is the same one.  With bc (the output of
// step_mix_kernel, for more experts than a row of lanes has) the rows come mixed.
// HBM-bound at a full batch, launch- and latency-bound for a few sequences.
template <typename T, int N, int R>
__global__ void __launch_bounds__(STEP_THREADS, R > 4 ? 7 : 8)
step_fused_kernel(const float *state_in, float *state_out, const T *__restrict__ x, const T *__restrict__ dt,
                  const float *__restrict__ A, const float *__restrict__ D, const T *__restrict__ Be,
                  const T *__restrict__ Ce, const T *__restrict__ logits, T *__restrict__ y,
                  int32_t *__restrict__ idx_out, const float *__restrict__ bc, Shape s, int slices, int t0, int L)
{
    constexpr int LPR = N / 4;                       // lanes of a state row
    constexpr int STRIDE = STEP_THREADS / LPR;       // rows of one register
    constexpr int ROWS = R * STRIDE;
    static_assert(R <= LPR, "every row sum has a lane");
    extern __shared__ __align__(16) float smem[];
    const int K = s.K, E = s.E, P = s.P;
    float *s_b = smem, *s_c = s_b + L * N, *s_x = s_c + L * N, *s_dt = s_x + L * ROWS, *s_a = s_dt + L;
    float *s_w = s_a + L;
    int32_t *s_i = (int32_t *)(s_w + L * K);
    const int sl = blockIdx.x % slices;
    const int h = (blockIdx.x / slices) % s.H;
    const int b = blockIdx.x / (slices * s.H);
    const int g = (h * s.G) / s.H;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int n4 = (tid % LPR) * 4, r0 = tid / LPR;
    const int p0 = sl * ROWS;
    const int64_t base = (((int64_t)b * s.H + h) * P + p0) * N;
    const int64_t tok = (int64_t)b * s.L + t0;       // first token of this launch

    // logits first: memory operations retire in order, and the router waits for them
    const int e16 = lane & 15;
    const int rt = wave * 4 + (lane >> 4);           // the token this row of lanes routes
    const float lg = !bc && rt < L && e16 < E ? to_float(logits[(tok + rt) * E + e16]) : -INFINITY;
#pragma unroll 1
    for (int i = tid; i < L * ROWS; i += STEP_THREADS) {
        const int t = i / ROWS, p = p0 + i % ROWS;
        s_x[i] = p < P ? to_float(x[((tok + t) * s.H + h) * P + p]) : 0.f;
    }
    if (tid < L) {
        const float dtv = to_float(dt[(tok + tid) * s.H + h]);
        s_dt[tid] = dtv;
        s_a[tid] = expf(dtv * A[h]);
    }
    f32x4_t v[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const uint32_t o = (uint32_t)(min(r * STRIDE + r0, P - 1 - p0) * N + n4);
        v[r] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t *>(state_in + base + o));
    }
    if (!bc) {
        if (rt < L) route_row16(lg, lane, E, K, s_i + rt * K, s_w + rt * K);
        lds_barrier();
        if (idx_out && h == 0 && sl == 0 && tid < L * K) idx_out[tok * K + tid] = s_i[tid];
    }
    // mixed rows of the L tokens: 4 columns of B or C per thread and turn
#pragma unroll 1
    for (int i = tid; i < L * 2 * LPR; i += STEP_THREADS) {
        const int t = i / (2 * LPR), c = (i / LPR) & 1, n = (i % LPR) * 4;
        float *dst = (c ? s_c : s_b) + t * N + n;
        if (bc) {
            *reinterpret_cast<f32x4_t *>(dst) =
                *reinterpret_cast<const f32x4_t *>(bc + (((tok + t) * s.G + g) * 2 + c) * N + n);
            continue;
        }
        const T *src = (c ? Ce : Be) + ((tok + t) * E * s.G + g) * N + n;
        float m[4] = {0.f, 0.f, 0.f, 0.f};
        for (int r = 0; r < K; ++r) {
            const T *row = src + (int64_t)s_i[t * K + r] * s.G * N;
            const float w = s_w[t * K + r];
            struct alignas(sizeof(T) * 4) { T q[4]; } four;
            __builtin_memcpy(&four, __builtin_assume_aligned(row, sizeof(T) * 4), sizeof four);
#pragma unroll
            for (int q = 0; q < 4; ++q) m[q] += w * to_float(four.q[q]);
        }
        *reinterpret_cast<f32x4_t *>(dst) = f32x4_t{m[0], m[1], m[2], m[3]};
    }
    lds_barrier();
    const float dsk = D ? D[h] : 0.f;
    // the row whose sum this lane ends up with (see group_sums)
    constexpr int LOGR = R == 1 ? 0 : R == 2 ? 1 : R == 4 ? 2 : 3;
    constexpr int SHIFT = (LPR == 64 ? 6 : LPR == 32 ? 5 : LPR == 16 ? 4 : LPR == 8 ? 3 : 2) - LOGR;
    const int myrow = ((lane % LPR) >> SHIFT) * STRIDE + r0;
    const bool mine = (lane & ((1 << SHIFT) - 1)) == 0 && p0 + myrow < P;
    T *yr = y + (tok * s.H + h) * P + p0 + myrow;
#pragma unroll 1
    for (int t = 0; t < L; ++t) {
        const f32x4_t bm = *reinterpret_cast<const f32x4_t *>(s_b + t * N + n4);
        const f32x4_t cm = *reinterpret_cast<const f32x4_t *>(s_c + t * N + n4);
        const float dtv = s_dt[t], decay = s_a[t];
        float part[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float u = dtv * s_x[t * ROWS + r * STRIDE + r0];
#pragma unroll
            for (int q = 0; q < 4; ++q) v[r][q] = decay * v[r][q] + u * bm[q];
            part[r] = (v[r][0] * cm[0] + v[r][1] * cm[1]) + (v[r][2] * cm[2] + v[r][3] * cm[3]);
        }
        const float tot = group_sums<LPR / 2>(part, lane);
        if (mine) yr[(int64_t)t * s.H * P] = from_float<T>(tot + dsk * s_x[t * ROWS + myrow]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        const int p = r * STRIDE + r0;
        if (p0 + p < P) __builtin_nontemporal_store(v[r], reinterpret_cast<f32x4_t *>(state_out + base + (uint32_t)(p * N + n4)));
    }
}

// Sums over the 32 lanes of a half wave of NV values per lane at once (NV a power of two, at most
// 16): every butterfly step halves the number of values a lane carries, so NV values cost
// NV shuffles instead of 5 NV.  Returns sum number ((lane & 31) >> 1) % NV... see below: after
// log2(NV) halving steps a lane holds the value whose index is given by its lane bits, the
// remaining steps are plain xor reductions.  Value i ends up (complete) on the lanes whose bits
// 4 .. 5-log2(NV) spell i.
template <int NV>
__device__ __forceinline__ float half_wave_sums(float (&v)[NV], int lane)
{
    int off = 16;
#pragma unroll
    for (int n = NV / 2; n >= 1; n >>= 1, off >>= 1) {
        const bool hi = (lane & off) != 0;
#pragma unroll
        for (int j = 0; j < n; ++j) {
            const float keep = hi ? v[n + j] : v[j];
            const float send = hi ? v[j] : v[n + j];
            v[j] = keep + __shfl_xor(send, off);
        }
    }
    float r = v[0];
    for (; off >= 1; off >>= 1) r += __shfl_xor(r, off);
    return r;
}

// ---- state update, any N: block = (b, h), a wave walks one state row at a time ------------
template <typename T>
__global__ void __launch_bounds__(STEP_THREADS)
step_update_generic_kernel(const float *state_in, float *state_out, const T *__restrict__ x,
                           const T *__restrict__ dt, const float *__restrict__ A,
                           const float *__restrict__ D, const float *__restrict__ bc,
                           T *__restrict__ y, Shape s, int L, int t)
{
    // token t of L per sequence: x, dt, bc and y are indexed by bt = b * L + t
    const int b = blockIdx.x / s.H, h = blockIdx.x % s.H, g = (h * s.G) / s.H;
    const int64_t bt = (int64_t)b * L + t;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int N = s.N, P = s.P;
    const int64_t base = ((int64_t)b * s.H + h) * P * N;
    const float *bm = bc + (bt * s.G + g) * 2 * N;
    const float *cm = bm + N;
    const float dtv = to_float(dt[bt * s.H + h]);
    const float decay = expf(dtv * A[h]);
    const float dsk = D ? D[h] : 0.f;
    for (int p = wave; p < P; p += STEP_THREADS / 64) {
        const float xv = to_float(x[(bt * s.H + h) * P + p]);
        const float u = dtv * xv;
        float part = 0.f;
        for (int n = lane; n < N; n += 64) {
            const float v = decay * state_in[base + (int64_t)p * N + n] + u * bm[n];
            state_out[base + (int64_t)p * N + n] = v;
            part += v * cm[n];
        }
#pragma unroll
        for (int off = 32; off >= 1; off >>= 1) part += __shfl_xor(part, off);
        if (lane == 0) y[(bt * s.H + h) * P + p] = from_float<T>(part + dsk * xv);
    }
}

// Tokens go STEP_FUSED_TOKENS per launch (the mixed rows of a launch are in LDS).
template <typename T, int N, int R>
static void launch_fused(const Shape &s, const float *state_in, float *state_out, const void *x, const void *dt,
                         const float *A, const float *D, const void *Be, const void *Ce, const void *logits, void *y,
                         int32_t *idx, const float *bc, hipStream_t st)
{
    constexpr int ROWS = R * STEP_THREADS / (N / 4);
    const int slices = (s.P + ROWS - 1) / ROWS;
    for (int t0 = 0; t0 < s.L; t0 += STEP_FUSED_TOKENS) {
        const int L = s.L - t0 < STEP_FUSED_TOKENS ? s.L - t0 : STEP_FUSED_TOKENS;
        const size_t lds = (size_t)L * (2 * N + ROWS + 2 + 2 * s.K) * sizeof(float);
        hipLaunchKernelGGL((step_fused_kernel<T, N, R>), dim3((unsigned)(s.B * s.H * slices)), dim3(STEP_THREADS), lds,
                           st, t0 == 0 ? state_in : state_out, state_out, (const T *)x, (const T *)dt, A, D,
                           (const T *)Be, (const T *)Ce, (const T *)logits, (T *)y, idx, bc, s, slices, t0, L);
    }
}

// Four registers of rows per lane (16 KB of state per block at most) stream best: full batch of 64 sequences x
// 64 heads 46.4 us (5.8 TB/s) against 52.6 with two and 49.4 with eight (one with one: 83.9).  Eight where every
// block then finds a place at once (7 blocks per compute unit) and four would need a second round (24 sequences:
// 16.9 against 19.5 us), and from five tokens on, where the routing and mixing that every block repeats
// costs more than the rounds (8 tokens x 16 sequences: 16.2 against 17.3 us).
template <typename T, int N>
static void launch_fused_rows(const Shape &s, const float *state_in, float *state_out, const void *x, const void *dt,
                              const float *A, const float *D, const void *Be, const void *Ce, const void *logits,
                              void *y, int32_t *idx, const float *bc, hipStream_t st)
{
    constexpr int STRIDE = STEP_THREADS / (N / 4);
    auto blocks = [&](int r) { return (int64_t)s.B * s.H * ((s.P + r * STRIDE - 1) / (r * STRIDE)); };
    const int ncu = device_cus();
    int R = s.L > 4 || (blocks(4) > 8 * ncu && blocks(8) <= 7 * ncu) ? 8 : 4;
    while (R > 1 && (R / 2) * STRIDE >= s.P) R /= 2;
    auto go = [&](auto r) {
        launch_fused<T, N, decltype(r)::value>(s, state_in, state_out, x, dt, A, D, Be, Ce, logits, y, idx, bc, st);
    };
    if (R >= 8 && N >= 32) go(std::integral_constant<int, N >= 32 ? 8 : 4>{});
    else if (R >= 4) go(std::integral_constant<int, 4>{});
    else if (R >= 2) go(std::integral_constant<int, 2>{});
    else go(std::integral_constant<int, 1>{});
}

// L tokens per sequence (1 for the single step): x (B,L,H,P), dt (B,L,H), Be/Ce (B,L,E,G,N), logits (B,L,E),
// y (B,L,H,P), idx (B,L,k), bc (B,L,G,2N) fp32.
template <typename T>
static swimba_status launch_step_multi_t(const Shape &s, const float *state_in, float *state_out,
                                         const void *x, const void *dt, const float *A, const float *D,
                                         const void *Be, const void *Ce, const void *logits, void *y,
                                         int32_t *idx, float *bc, hipStream_t st)
{
    const int64_t blocks = (int64_t)s.B * s.H;
    if (blocks == 0 || s.L == 0) return SWIMBA_OK;
    const bool route_in_update = s.E <= STEP_FUSED_EXPERTS;
    const bool rows = (s.N & (s.N - 1)) == 0 && s.N >= 16 && s.N <= 256 && blocks * s.P < (1ll << 31);
    if (!rows || !route_in_update) {
        Shape tok = s;             // the mix kernel sees B*L independent tokens
        tok.B = s.B * s.L;
        tok.L = 1;
        hipLaunchKernelGGL(step_mix_kernel<T>, dim3((unsigned)(tok.B * s.G)), dim3(128), 0, st, (const T *)Be,
                           (const T *)Ce, (const T *)logits, bc, idx, tok);
        SWIMBA_CHECK_LAUNCH();
    }
    if (rows) {
        const float *mixed = route_in_update ? nullptr : bc;
        auto fused = [&](auto n) {
            launch_fused_rows<T, decltype(n)::value>(s, state_in, state_out, x, dt, A, D, Be, Ce, logits, y, idx, mixed, st);
        };
        switch (s.N) {
        case 16: fused(std::integral_constant<int, 16>{}); break;
        case 32: fused(std::integral_constant<int, 32>{}); break;
        case 64: fused(std::integral_constant<int, 64>{}); break;
        case 128: fused(std::integral_constant<int, 128>{}); break;
        default: fused(std::integral_constant<int, 256>{}); break;
        }
        SWIMBA_CHECK_LAUNCH();
        return SWIMBA_OK;
    }
    // other N: one launch per token
    for (int t = 0; t < s.L; ++t) {
        hipLaunchKernelGGL(step_update_generic_kernel<T>, dim3((unsigned)blocks), dim3(STEP_THREADS), 0, st,
                           t == 0 ? state_in : state_out, state_out, (const T *)x, (const T *)dt, A, D, bc,
                           (T *)y, s, s.L, t);
        SWIMBA_CHECK_LAUNCH();
    }
    return SWIMBA_OK;
}

swimba_status launch_step_multi(const Shape &s, int io_dtype, const float *state_in, float *state_out,
                                const void *x, const void *dt, const float *A, const float *D,
                                const void *Be, const void *Ce, const void *logits, void *y, int32_t *idx,
                                float *bc, hipStream_t st)
{
    if (io_dtype == SWIMBA_BF16)
        return launch_step_multi_t<bf16>(s, state_in, state_out, x, dt, A, D, Be, Ce, logits, y, idx, bc, st);
    return launch_step_multi_t<float>(s, state_in, state_out, x, dt, A, D, Be, Ce, logits, y, idx, bc, st);
}

// Device address of `scratch` on the current device, looked up once per device.
static swimba_status static_scratch(float **out)
{
    constexpr int MAXDEV = 64;
    static std::atomic<float *> ptr[MAXDEV];
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) { set_last_hip_error((int)e); return SWIMBA_ERR_HIP; }
    if (dev < 0 || dev >= MAXDEV) return SWIMBA_ERR_UNSUPPORTED;
    float *p = ptr[dev].load(std::memory_order_acquire);
    if (!p) {
        e = hipGetSymbolAddress((void **)&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) { set_last_hip_error((int)e); return SWIMBA_ERR_HIP; }
        ptr[dev].store(p, std::memory_order_release);   // every thread that gets here stores the same address
    }
    *out = p;
    return SWIMBA_OK;
}

swimba_status launch_step_static(const Shape &s, int io_dtype, const float *state_in, float *state_out,
                                 const void *x, const void *dt, const float *A, const float *D,
                                 const void *Be, const void *Ce, const void *logits, void *y, int32_t *idx,
                                 hipStream_t st)
{
    if ((int64_t)s.B * s.G * s.N * 2 * (int64_t)sizeof(float) > (int64_t)SWIMBA_STATIC_SCRATCH_BYTES)
        return SWIMBA_ERR_UNSUPPORTED;
    float *bc = nullptr;
    const swimba_status rs = static_scratch(&bc);
    if (rs != SWIMBA_OK) return rs;
    // the mix kernel overwrites every element the update kernel reads: nothing has to be cleared
    return launch_step(s, io_dtype, state_in, state_out, x, dt, A, D, Be, Ce, logits, y, idx, bc, st);
}

swimba_status launch_step(const Shape &s, int io_dtype, const float *state_in, float *state_out,
                          const void *x, const void *dt, const float *A, const float *D,
                          const void *Be, const void *Ce, const void *logits, void *y, int32_t *idx,
                          float *bc, hipStream_t st)
{
    if (io_dtype == SWIMBA_BF16)
        return launch_step_multi_t<bf16>(s, state_in, state_out, x, dt, A, D, Be, Ce, logits, y, idx, bc, st);
    return launch_step_multi_t<float>(s, state_in, state_out, x, dt, A, D, Be, Ce, logits, y, idx, bc, st);
}

}  // namespace swimba
