// Recurrent decode step of one or a few tokens per sequence (paper: selective SSM recurrence per channel,
// with the router-mixed injection and readout of Theorem 1).  State sizes that are a power of two: one launch where a
// row of lanes holds a token's logits (up to 16 experts) and a block routes all tokens at once (up to 16): every
// block routes and mixes its tokens while its piece of the fp32 state is on its way in, applies them to it and writes
// it back.  More experts or tokens: the update behind a small kernel that routes and mixes (fp32 rows in the
// caller's workspace); the state still crosses memory once.  Other state sizes: that small kernel and one update
// launch per token.
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

// ---- routing + mixing of a token: bc[g] = its mixed rows (B; C) of N fp32 each -------------
// Pieces of V columns of one row, four where N allows it, else one.  Block = (token, 128 U pieces), U per lane: one
// fills the chip at few tokens and groups; four requested together where blocks are plenty, for the routing in front
// of them is a chain that every block of a token repeats (64 x 32 tokens, 64 groups: 185 us for the call with one,
// 171 with four).
constexpr int STEP_MIX_THREADS = 128;
template <typename T, int V, int U>
__global__ void __launch_bounds__(STEP_MIX_THREADS)
step_mix_kernel(const T *__restrict__ Be, const T *__restrict__ Ce, const T *__restrict__ logits,
                float *__restrict__ bc, int32_t *__restrict__ idx_out, Shape s, int parts)
{
    __shared__ float s_w[SWIMBA_MAX_TOPK];
    __shared__ int32_t s_idx[SWIMBA_MAX_TOPK];
    __shared__ float s_log[SWIMBA_MAX_EXPERTS];
    const int part = blockIdx.x % parts;
    const int64_t tok = blockIdx.x / parts;
    const int tid = threadIdx.x;
    if (s.E <= STEP_FUSED_EXPERTS) {
        // as in the update that routes by itself (the four rows of lanes hold the same logits)
        if (tid < 64) {
            const int e = tid & 15;
            route_row16(e < s.E ? to_float(logits[tok * s.E + e]) : -INFINITY, tid, s.E, s.K, s_idx, s_w);
        }
    } else {
        // the logits go through LDS first: one memory latency instead of one per pass of the router
        for (int e = tid; e < s.E; e += STEP_MIX_THREADS) s_log[e] = to_float(logits[tok * s.E + e]);
        __syncthreads();
        if (tid == 0) route_token([&](int e) { return s_log[e]; }, s.E, s.K, s_idx, s_w);
    }
    __syncthreads();
    if (idx_out && part == 0 && tid < s.K) idx_out[tok * s.K + tid] = s_idx[tid];
    const int row = s.N / V, pieces = s.G * 2 * row;                          // (g, B or C, piece of the row)
    struct alignas(sizeof(T) * V) Piece { T q[V]; };
    const T *src[U];
    int to[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        const int i = min((part * U + u) * STEP_MIX_THREADS + tid, pieces - 1);
        const int n = i % row * V, c = i / row % 2, g = i / (2 * row);
        src[u] = (c ? Ce : Be) + (tok * s.E * s.G + g) * s.N + n;
        to[u] = (g * 2 + c) * s.N + n;
    }
    float m[U][V] = {};
    for (int r = 0; r < s.K; ++r) {
        const int64_t o = (int64_t)s_idx[r] * s.G * s.N;
        Piece v[U];
#pragma unroll
        for (int u = 0; u < U; ++u) __builtin_memcpy(&v[u], __builtin_assume_aligned(src[u] + o, sizeof v[u]), sizeof v[u]);
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
            for (int q = 0; q < V; ++q) m[u][q] += s_w[r] * to_float(v[u].q[q]);
    }
    float *out = bc + tok * s.G * 2 * s.N;
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if ((part * U + u) * STEP_MIX_THREADS + tid >= pieces) continue;
        if constexpr (V == 4) *reinterpret_cast<f32x4_t *>(out + to[u]) = f32x4_t{m[u][0], m[u][1], m[u][2], m[u][3]};
        else out[to[u]] = m[u][0];
    }
}

// Both kernels below: block = (b, h, slice of R * 256 / (N/4) state rows); lane -> 4 columns of R rows, held in
// registers over the L tokens, so the state crosses memory once in each direction.
// HBM-bound at a full batch, launch- and latency-bound for a few sequences.
template <int N, int R>
struct StepRows {
    static constexpr int LPR = N / 4;                       // lanes of a state row
    static constexpr int STRIDE = STEP_THREADS / LPR;       // rows of one register
    static constexpr int ROWS = R * STRIDE;
    static_assert(R <= LPR, "every row sum has a lane");
    // the row whose sum a lane ends up with (see group_sums)
    static constexpr int LOGR = R == 1 ? 0 : R == 2 ? 1 : R == 4 ? 2 : 3;
    static constexpr int SHIFT = (LPR == 64 ? 6 : LPR == 32 ? 5 : LPR == 16 ? 4 : LPR == 8 ? 3 : 2) - LOGR;

    int lane, r0, n4, p0, P, myrow;
    bool mine;
    f32x4_t v[R];

    __device__ __forceinline__ StepRows(int tid, int p0_, int P_)
        : lane(tid & 63), r0(tid / LPR), n4((tid % LPR) * 4), p0(p0_), P(P_)
    {
        myrow = ((lane % LPR) >> SHIFT) * STRIDE + r0;
        mine = (lane & ((1 << SHIFT) - 1)) == 0 && p0 + myrow < P;
    }
    __device__ __forceinline__ void load(const float *state)       // state: the slice's first row
    {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const uint32_t o = (uint32_t)(min(r * STRIDE + r0, P - 1 - p0) * N + n4);
            v[r] = __builtin_nontemporal_load(reinterpret_cast<const f32x4_t *>(state + o));
        }
    }
    __device__ __forceinline__ void store(float *state) const
    {
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const int p = r * STRIDE + r0;
            if (p0 + p < P) __builtin_nontemporal_store(v[r], reinterpret_cast<f32x4_t *>(state + (uint32_t)(p * N + n4)));
        }
    }
    // one token: mixed rows b and c (N), x(row): inputs of the slice's rows; y: the token's output of this lane's row
    template <typename T, typename X>
    __device__ __forceinline__ void token(const float *b, const float *c, X x, float dtv, float decay, float dsk, T *y)
    {
        const f32x4_t bm = *reinterpret_cast<const f32x4_t *>(b + n4);
        const f32x4_t cm = *reinterpret_cast<const f32x4_t *>(c + n4);
        float part[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const float u = dtv * x(r * STRIDE + r0);
#pragma unroll
            for (int q = 0; q < 4; ++q) v[r][q] = fmaf(u, bm[q], decay * v[r][q]);   // in place: no register moves
            part[r] = (v[r][0] * cm[0] + v[r][1] * cm[1]) + (v[r][2] * cm[2] + v[r][3] * cm[3]);
        }
        const float tot = group_sums<LPR / 2>(part, lane);
        if (mine) *y = from_float<T>(tot + dsk * x(myrow));
    }
};

// Up to STEP_FUSED_TOKENS tokens of up to STEP_FUSED_EXPERTS experts.  Every block routes and mixes its
// sequence's tokens itself (rows of a group's B and C come from L2 for all but the first head); the state
// loads are issued before that chain and the latency of both is the same one.
template <typename T, int N, int R>
__global__ void __launch_bounds__(STEP_THREADS, R > 4 ? 7 : 8)
step_fused_kernel(const float *state_in, float *state_out, const T *__restrict__ x, const T *__restrict__ dt,
                  const float *__restrict__ A, const float *__restrict__ D, const T *__restrict__ Be,
                  const T *__restrict__ Ce, const T *__restrict__ logits, T *__restrict__ y,
                  int32_t *__restrict__ idx_out, Shape s, int slices)
{
    constexpr int LPR = StepRows<N, R>::LPR, ROWS = StepRows<N, R>::ROWS;
    extern __shared__ __align__(16) float smem[];
    const int K = s.K, E = s.E, P = s.P, L = s.L;
    float *s_b = smem, *s_c = s_b + L * N, *s_x = s_c + L * N, *s_dt = s_x + L * ROWS, *s_a = s_dt + L;
    float *s_w = s_a + L;
    int32_t *s_i = (int32_t *)(s_w + L * K);
    const int sl = blockIdx.x % slices;
    const int h = (blockIdx.x / slices) % s.H;
    const int b = blockIdx.x / (slices * s.H);
    const int g = (h * s.G) / s.H;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int p0 = sl * ROWS;
    const int64_t base = (((int64_t)b * s.H + h) * P + p0) * N;
    const int64_t tok = (int64_t)b * L;

    // logits first: memory operations retire in order, and the router waits for them
    const int e16 = lane & 15;
    const int rt = wave * 4 + (lane >> 4);           // the token this row of lanes routes
    const float lg = rt < L && e16 < E ? to_float(logits[(tok + rt) * E + e16]) : -INFINITY;
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
    StepRows<N, R> rows(tid, p0, P);
    rows.load(state_in + base);
    if (rt < L) route_row16(lg, lane, E, K, s_i + rt * K, s_w + rt * K);
    lds_barrier();
    if (idx_out && h == 0 && sl == 0 && tid < L * K) idx_out[tok * K + tid] = s_i[tid];
    // mixed rows of the L tokens: 4 columns of B or C per thread and turn
#pragma unroll 1
    for (int i = tid; i < L * 2 * LPR; i += STEP_THREADS) {
        const int t = i / (2 * LPR), c = (i / LPR) & 1, n = (i % LPR) * 4;
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
        *reinterpret_cast<f32x4_t *>((c ? s_c : s_b) + t * N + n) = f32x4_t{m[0], m[1], m[2], m[3]};
    }
    lds_barrier();
    const float dsk = D ? D[h] : 0.f;
    T *yr = y + (tok * s.H + h) * P + p0 + rows.myrow;
#pragma unroll 1
    for (int t = 0; t < L; ++t)
        rows.token(s_b + t * N, s_c + t * N, [=](int p) { return s_x[t * ROWS + p]; }, s_dt[t], s_a[t], dsk, yr + (int64_t)t * s.H * P);
    rows.store(state_out + base);
}

// Any number of tokens and experts, behind step_mix_kernel: bc holds the mixed rows (B; C) of every token and group.
// The tokens pass through LDS TG at a time, the next ones on their way while these are applied.
template <typename T, int N, int R, int TG>
__global__ void __launch_bounds__(STEP_THREADS, TG > 4 ? 4 : R > 4 ? 7 : 8)
step_mixed_kernel(const float *state_in, float *state_out, const T *__restrict__ x, const T *__restrict__ dt,
                  const float *__restrict__ A, const float *__restrict__ D, const float *__restrict__ bc,
                  T *__restrict__ y, Shape s, int slices)
{
    constexpr int ROWS = StepRows<N, R>::ROWS;
    constexpr int NB = TG * 2 * N / 4 > STEP_THREADS ? TG * 2 * N / 4 / STEP_THREADS : 1;     // quads of bc per lane
    constexpr int NX = TG * ROWS > STEP_THREADS ? TG * ROWS / STEP_THREADS : 1;
    __shared__ __align__(16) float s_bc[TG * 2 * N], s_x[TG * ROWS];
    __shared__ float s_dt[TG], s_a[TG];
    const int P = s.P, L = s.L;
    const int sl = blockIdx.x % slices;
    const int h = (blockIdx.x / slices) % s.H;
    const int b = blockIdx.x / (slices * s.H);
    const int g = (h * s.G) / s.H;
    const int tid = threadIdx.x;
    const int p0 = sl * ROWS;
    const int64_t base = (((int64_t)b * s.H + h) * P + p0) * N;
    const int64_t tok = (int64_t)b * L;
    const float Ah = A[h], dsk = D ? D[h] : 0.f;

    f32x4_t nb[NB];
    float nx[NX], ndt = 0.f;
    // tokens past the last one are left out 256 lanes at a time and repeat the last one otherwise
    auto load = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int o = (tid + i * STEP_THREADS) * 4;
            if (t0 + i * STEP_THREADS * 4 / (2 * N) < L)
                nb[i] = *reinterpret_cast<const f32x4_t *>(bc + ((tok + min(t0 + o / (2 * N), L - 1)) * s.G + g) * 2 * N + o % (2 * N));
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int o = tid + i * STEP_THREADS;
            if (t0 + i * STEP_THREADS / ROWS < L)
                nx[i] = to_float(x[((tok + min(t0 + o / ROWS, L - 1)) * s.H + h) * P + min(p0 + o % ROWS, P - 1)]);
        }
        if (tid < TG) ndt = to_float(dt[(tok + min(t0 + tid, L - 1)) * s.H + h]);
    };
    auto stage = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int i = 0; i < NB; ++i) {
            const int o = (tid + i * STEP_THREADS) * 4;
            if (o < TG * 2 * N) *reinterpret_cast<f32x4_t *>(s_bc + o) = nb[i];
        }
#pragma unroll
        for (int i = 0; i < NX; ++i) {
            const int o = tid + i * STEP_THREADS;
            if (o < TG * ROWS) s_x[o] = nx[i];
        }
        if (tid < TG) {
            s_dt[tid] = ndt;
            s_a[tid] = expf(ndt * Ah);
        }
    };
    load(0);
    StepRows<N, R> rows(tid, p0, P);
    rows.load(state_in + base);
    T *yr = y + (tok * s.H + h) * P + p0 + rows.myrow;
    for (int t0 = 0; t0 < L; t0 += TG) {
        stage();
        lds_barrier();
        if (TG > 4 && t0 + TG < L) load(t0 + TG);             // (four tokens are the whole call)
        const int n = min(TG, L - t0);
#pragma unroll 1
        for (int t = 0; t < n; ++t)
            rows.token(s_bc + t * 2 * N, s_bc + t * 2 * N + N, [&](int p) { return s_x[t * ROWS + p]; }, s_dt[t], s_a[t], dsk,
                       yr + (int64_t)(t0 + t) * s.H * P);
        lds_barrier();
    }
    rows.store(state_out + base);
}

// One token whose rows come mixed: nothing to keep in LDS.
template <typename T, int N, int R>
__global__ void __launch_bounds__(STEP_THREADS, 8)
step_mixed_one_kernel(const float *state_in, float *state_out, const T *__restrict__ x, const T *__restrict__ dt,
                      const float *__restrict__ A, const float *__restrict__ D, const float *__restrict__ bc,
                      T *__restrict__ y, Shape s, int slices)
{
    const int P = s.P;
    const int sl = blockIdx.x % slices;
    const int h = (blockIdx.x / slices) % s.H;
    const int b = blockIdx.x / (slices * s.H);
    const int g = (h * s.G) / s.H;
    const int p0 = sl * StepRows<N, R>::ROWS;
    const int64_t bh = (int64_t)b * s.H + h, base = (bh * P + p0) * N;
    const float dtv = to_float(dt[bh]), decay = expf(dtv * A[h]), dsk = D ? D[h] : 0.f;
    const float *row = bc + ((int64_t)b * s.G + g) * 2 * N;
    const T *xr = x + bh * P + p0;
    const int last = P - 1 - p0;
    StepRows<N, R> rows(threadIdx.x, p0, P);
    rows.load(state_in + base);
    rows.token(row, row + N, [=](int p) { return to_float(xr[min(p, last)]); }, dtv, decay, dsk, y + bh * P + p0 + rows.myrow);
    rows.store(state_out + base);
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

template <typename T, int N, int R>
static void launch_rows(const Shape &s, const float *state_in, float *state_out, const void *x, const void *dt,
                        const float *A, const float *D, const void *Be, const void *Ce, const void *logits, void *y,
                        int32_t *idx, const float *bc, hipStream_t st)
{
    constexpr int ROWS = StepRows<N, R>::ROWS;
    const int slices = (s.P + ROWS - 1) / ROWS;
    const dim3 grid((unsigned)(s.B * s.H * slices));
    if (bc) {
        constexpr int R4 = R > 4 ? 4 : R;                    // at most, up to four tokens (launch_update)
        auto kernel = s.L > 4 ? step_mixed_kernel<T, N, R, 16> : s.L > 1 ? step_mixed_kernel<T, N, R4, 4> : step_mixed_one_kernel<T, N, R4>;
        hipLaunchKernelGGL(kernel, grid, dim3(STEP_THREADS), 0, st, state_in, state_out, (const T *)x, (const T *)dt, A, D,
                           bc, (T *)y, s, slices);
        return;
    }
    const size_t lds = (size_t)s.L * (2 * N + ROWS + 2 + 2 * s.K) * sizeof(float);
    hipLaunchKernelGGL((step_fused_kernel<T, N, R>), grid, dim3(STEP_THREADS), lds, st, state_in, state_out, (const T *)x,
                       (const T *)dt, A, D, (const T *)Be, (const T *)Ce, (const T *)logits, (T *)y, idx, s, slices);
}

// Registers of rows per lane.
// Routing inside: four (16 KB of state per block at most) stream best: full batch of 64 sequences x 64 heads 46.4 us
// (5.8 TB/s) against 52.6 with two and 49.4 with eight (one with one: 83.9).  Eight where every block then finds a
// place at once (7 blocks per compute unit) and four would need a second round (24 sequences: 16.9 against 19.5 us),
// and from five tokens on, where the routing and mixing that every block repeats costs more than the rounds
// (8 tokens x 16 sequences: 16.2 against 17.3 us).
// Rows that come mixed: up to four tokens four, as above (one token, 64 sequences x 64 heads: 57 us with two and
// with four, 63 with one, 86 with eight).  With more the tokens' chain counts: as many rows as leave 1.5 blocks per
// compute unit, and eight only from four blocks on.  64 tokens x 32 heads, one / two / four / eight registers:
// 1 sequence 21.2 / 24.0 / 30.1 / 41.5 us, 4: 27.8 / 25.8 / 30.9 / 42.4, 16: 70 / 55 / 47.9 / 49.3, 64: 244 / 169 / 145 / 136.
template <typename T, int N>
static void launch_update(const Shape &s, const float *state_in, float *state_out, const void *x, const void *dt,
                          const float *A, const float *D, const void *Be, const void *Ce, const void *logits,
                          void *y, int32_t *idx, const float *bc, hipStream_t st)
{
    constexpr int STRIDE = STEP_THREADS / (N / 4);
    auto blocks = [&](int r) { return (int64_t)s.B * s.H * ((s.P + r * STRIDE - 1) / (r * STRIDE)); };
    const int ncu = device_cus();
    int R;
    if (!bc) R = s.L > 4 || (blocks(4) > 8 * ncu && blocks(8) <= 7 * ncu) ? 8 : 4;
    else if (s.L <= 4) R = 4;
    else for (R = blocks(8) >= 4 * ncu ? 8 : 4; R > 1 && 2 * blocks(R) < 3 * ncu; R /= 2) {}
    while (R > 1 && (R / 2) * STRIDE >= s.P) R /= 2;
    auto go = [&](auto r) {
        launch_rows<T, N, decltype(r)::value>(s, state_in, state_out, x, dt, A, D, Be, Ce, logits, y, idx, bc, st);
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
    const bool route_in_update = s.E <= STEP_FUSED_EXPERTS && s.L <= STEP_FUSED_TOKENS;
    const bool rows = (s.N & (s.N - 1)) == 0 && s.N >= 16 && s.N <= 256 && blocks * s.P < (1ll << 31);
    if (!rows || !route_in_update) {
        const int V = s.N % 4 == 0 ? 4 : 1, pieces = s.G * 2 * (s.N / V);
        const int64_t tokens = (int64_t)s.B * s.L;
        auto parts = [&](int u) { return (pieces + u * STEP_MIX_THREADS - 1) / (u * STEP_MIX_THREADS); };
        const int U = parts(4) < parts(1) && tokens * parts(4) >= 16 * device_cus() ? 4 : 1;
        auto mix = V == 4 ? U == 4 ? step_mix_kernel<T, 4, 4> : step_mix_kernel<T, 4, 1>
                          : U == 4 ? step_mix_kernel<T, 1, 4> : step_mix_kernel<T, 1, 1>;
        hipLaunchKernelGGL(mix, dim3((unsigned)(tokens * parts(U))), dim3(STEP_MIX_THREADS), 0, st, (const T *)Be,
                           (const T *)Ce, (const T *)logits, bc, idx, s, parts(U));
        SWIMBA_CHECK_LAUNCH();
    }
    if (rows) {
        const float *mixed = route_in_update ? nullptr : bc;
        auto fused = [&](auto n) {
            launch_update<T, decltype(n)::value>(s, state_in, state_out, x, dt, A, D, Be, Ce, logits, y, idx, mixed, st);
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
