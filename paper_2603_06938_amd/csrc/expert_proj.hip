// Routed expert in-projection (paper, MoE-parameterized SSM: the expert streams are
// expert-specific linear projections of the same token features, and only the experts of the
// active set K_t enter the mix): for every token t and every e in K_t
//   B_t^(e)[c] = sum_d W_B[e][c][d] u_t[d],   C_t^(e)[c] = sum_d W_C[e][c][d] u_t[d],
// written either into the dense (B,L,E,G,N) layout (rows of inactive experts are not touched:
// the mixer never reads them) or, with `compact`, into (B,L,k,G,N): row r of a token is the
// stream of its r-th selected expert, so no buffer with an expert axis exists at all.
// The experts' input streams X^(e) (the mixed state update in its full form injects
// sum_e pi_e x^(e) (x) B^(e)) are a third block of output columns of the same product,
//   x_t^(e)[c] = sum_d W_X[e][c][d] u_t[d],  c over (head, channel),
// written the same way into (B,L,E,H,P) or (B,L,k,H,P).
//
// Three launches: clear the per-expert counters; route every token and append the entry
// t*k + r to the list of its r-th expert (LDS counters per block, one global atomic per block
// and expert); a grouped GEMM over (share of an expert's list, 256 output columns).
// The GEMM is a dense contraction, so it runs on v_mfma_f32_32x32x16_bf16.  Both operands
// are stored with the contraction index d contiguous (weights as (out, in), like a linear
// layer), which is the 8-consecutive-k operand layout.  The product is computed transposed,
// out^T[c][token], with the weight rows permuted so that a lane ends up with 16 consecutive
// output columns of one token (two 16-byte stores).
#include "common.hpp"

#include <atomic>
#include <type_traits>

namespace swimba {

typedef __attribute__((ext_vector_type(8))) __bf16 pj_bf16x8_t;
typedef __attribute__((ext_vector_type(2))) __bf16 pj_bf16x2_t;
typedef __attribute__((ext_vector_type(2))) float pj_f32x2_t;
typedef __attribute__((ext_vector_type(16))) float pj_f32x16_t;

constexpr int PJ_COLS = 256;   // output columns per workgroup: 4 column groups of 64

// The output columns of the product are the concatenation [B | C | X] of up to three blocks, each
// with its own weight tensor (E, n, Dm) and its own output tensor (rows of n columns).
struct ProjBlocks {
    const void *W[3];
    void *out[3];
    int n[3];       // columns of the block (0: absent); multiples of 64 on the MFMA path
    int tot;        // n[0] + n[1] + n[2]
};
// block of column c and the column inside it
__device__ __forceinline__ int proj_block_of(const ProjBlocks &pb, int c, int &local)
{
    const int s = (c >= pb.n[0]) + (c >= pb.n[0] + pb.n[1]);
    local = c - (s > 0 ? pb.n[0] : 0) - (s > 1 ? pb.n[1] : 0);
    return s;
}

__global__ void proj_clear_kernel(int32_t *counts, int E)
{
    for (int e = threadIdx.x; e < E; e += blockDim.x) counts[e] = 0;
}

// one token per lane: top-k routing, then one list entry per active expert
template <typename T>
__global__ void __launch_bounds__(256)
proj_route_kernel(const T *__restrict__ logits, int32_t *__restrict__ idx, float *__restrict__ w,
                  int32_t *__restrict__ counts, int32_t *__restrict__ lists, int64_t tokens, int E, int K)
{
    __shared__ int32_t s_cnt[SWIMBA_MAX_EXPERTS], s_base[SWIMBA_MAX_EXPERTS];
    extern __shared__ int32_t s_loc[];                       // [256][K] rank inside the block
    const int tid = threadIdx.x;
    const int64_t t = (int64_t)blockIdx.x * 256 + tid;
    for (int e = tid; e < E; e += 256) s_cnt[e] = 0;
    __syncthreads();
    if (t < tokens) {
        const T *g = logits + t * E;
        route_token([&](int e) { return to_float(g[e]); }, E, K, idx + t * K, w + t * K);
        for (int r = 0; r < K; ++r) s_loc[tid * K + r] = atomicAdd(&s_cnt[idx[t * K + r]], 1);
    }
    __syncthreads();
    for (int e = tid; e < E; e += 256) s_base[e] = s_cnt[e] ? atomicAdd(&counts[e], s_cnt[e]) : 0;
    __syncthreads();
    if (t < tokens) {
        for (int r = 0; r < K; ++r) {
            const int e = idx[t * K + r];
            lists[(int64_t)e * tokens + s_base[e] + s_loc[tid * K + r]] = (int32_t)(t * K + r);
        }
    }
}

__device__ __forceinline__ uint32_t pj_pack(float lo, float hi)
{
    pj_f32x2_t f = {lo, hi};
    pj_bf16x2_t h = __builtin_convertvector(f, pj_bf16x2_t);   // round to nearest even
    return __builtin_bit_cast(uint32_t, h);
}

// Workgroup = (share of one expert's list, block of 256 output columns), 8 waves: wave w owns
// columns 64 (w & 3) .. + 63 of the block and one of two row groups.  The `nslots` workgroups
// that fit on the chip at once (one per compute unit) are divided among the experts in
// proportion to their list lengths (known on the device only), and a workgroup walks its share
// in passes of up to 256 entries (2 to 4 row tiles of 32 per row group, one code path each): the
// whole launch is one round of co-resident workgroups, whatever the routing.  The contraction
// runs in stages of 64 features: both operands (256 weight rows, 64 per row tile of a group of
// token rows, 128 bytes each) are read with fully coalesced 16-byte loads (8 lanes per row),
// parked in registers while earlier stages are multiplied, and passed through one of two LDS
// buffers, from where the lanes read their operand registers: one barrier a stage.
// Against one code path of three row tiles per group, one LDS buffer and shares spread over the
// XCDs: 8192 tokens x 1792 columns (130M-shaped layer with input streams) 86 -> 75 us, the whole
// call 171 -> 164, of which the shares' place on the XCDs is 5; 16384 tokens x 256 columns 31 -> 30.
// What is left there (us, 75 / 30): without the MFMAs and operand reads 45 / 19, without the writes
// of a stage into LDS 50 / 20, without the stores of the results 60 / 25; the loads are hidden.
// LDS is busy a quarter of the time, so its waits and the stages' order count, not its rate: the
// barrier moved between the k-steps of a stage measured the same (75.6 / 31), results through LDS
// to store whole lines worse (79 / 34).
constexpr int PJ_THREADS = 512;
constexpr int PJ_KT = 64;             // features per stage
constexpr int PJ_STR = PJ_KT + 8;     // LDS row stride (elements): rows stay 16-byte aligned
constexpr int PJ_MAX_RT = 4;          // row tiles (of 32 list entries) per wave and pass
constexpr int PJ_BUF = (PJ_COLS + 64 * PJ_MAX_RT) * PJ_STR;   // elements of an LDS buffer
constexpr size_t PJ_SHM = 2 * PJ_BUF * sizeof(uint16_t);

// workgroups expert e gets out of nslots, given its list length
__device__ __forceinline__ int proj_share(int cnt, int nslots, int64_t total)
{
    return cnt > 0 ? max(1, (int)((int64_t)nslots * cnt / total)) : 0;
}

__global__ void __launch_bounds__(PJ_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
proj_mfma_kernel(const uint16_t *__restrict__ u, ProjBlocks pb, const int32_t *__restrict__ counts,
                 const int32_t *__restrict__ lists, int64_t tokens, int E, int K, int Dm, int nslots,
                 int colblocks, int compact)
{
    extern __shared__ __align__(16) uint16_t s_buf[];        // [2] weight rows, then token rows
    __shared__ int32_t s_share[SWIMBA_MAX_EXPERTS];
    __shared__ int32_t s_sel[3];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int64_t total = tokens * K;

    // ---- which expert, which part of its list: prefix sum of the shares (E <= 256 = 4 per lane) ----
    // Workgroups of one XCD (ids equal mod 8) take neighbouring shares with all their column blocks, so
    // that its L2 holds the weights of about one expert and the token rows are read into it once.
    if (tid < SWIMBA_MAX_EXPERTS) s_share[tid] = tid < E ? proj_share(counts[tid], nslots, total) : 0;
    if (tid == 0) s_sel[0] = -1;
    __syncthreads();
    if (wave == 0) {
        int v[4], sum = 0;
#pragma unroll
        for (int q = 0; q < 4; ++q) { v[q] = s_share[4 * lane + q]; sum += v[q]; }
        int incl = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(incl, d);
            if (lane >= d) incl += t;
        }
        const int used = __builtin_amdgcn_readlane(incl, 63) * colblocks, per = (used + 7) / 8;
        const int j = (int)blockIdx.x >> 3, lid = ((int)blockIdx.x & 7) * per + j;
        int r = lid / colblocks - (incl - sum);
        if (j < per && lid < used && r >= 0 && r < sum) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (r >= 0 && r < v[q]) { s_sel[0] = 4 * lane + q; s_sel[1] = r; s_sel[2] = lid % colblocks; }
                r -= v[q];          // negative from the match on: no later q matches
            }
        }
    }
    __syncthreads();
    const int e = __builtin_amdgcn_readfirstlane(s_sel[0]);
    if (e < 0) return;                                       // whole workgroup: no barrier is skipped
    const int part = __builtin_amdgcn_readfirstlane(s_sel[1]);
    const int cnt = counts[e];
    const int nparts = proj_share(cnt, nslots, total);
    const int n32 = (cnt + 31) / 32;
    const int t_begin = (int)((int64_t)part * n32 / nparts), t_end = (int)((int64_t)(part + 1) * n32 / nparts);
    const int nt = t_end - t_begin;
    if (nt <= 0) return;
    const int npass = (nt + 2 * PJ_MAX_RT - 1) / (2 * PJ_MAX_RT);

    const int cw = wave & 3, rg = wave >> 2;                 // column group, row group of the wave
    const int colblk = __builtin_amdgcn_readfirstlane(s_sel[2]) * PJ_COLS;   // first column of the workgroup in [B | C | X]
    const int col0 = colblk + cw * 64;
    const bool active = col0 < pb.tot;                       // wave-uniform; idle waves still stage
    const int l32 = lane & 31, kg = lane >> 5;

    // ---- staging map: lane -> 16-byte piece `piece` of rows row0 + 64 i ----
    const int piece = tid & 7, row0 = tid >> 3;              // row0 = 32 rg + (row inside a 32-block)
    // Every block has a multiple of 32 columns, so the 32 rows of a staging step of one wave lie in
    // one weight tensor: a uniform base (scalar registers) + one per-lane offset for all four.
    const uint16_t *wbase[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        int cl;
        const int sb = proj_block_of(pb, min(colblk + 64 * i + 32 * rg, pb.tot - 32), cl);   // past the end: the last rows again
        wbase[i] = (const uint16_t *)pb.W[sb] + ((int64_t)e * pb.n[sb] + cl) * Dm;
    }
    const int r32 = row0 & 31;
    const int wlane = r32 * Dm;
    const int k_last = ((Dm - 1) / PJ_KT) * PJ_KT;
    // Operand row r of a 32-column weight tile must hold column 16*((r>>2)&1) + 4*(r>>3) + (r&3)
    // for accumulator register v of lane (l32, kg) to be column 16 kg + v of the tile.  The
    // permutation is applied when the rows are staged (column x goes to LDS row wrow), so the
    // lanes of a wave read consecutive LDS rows: no bank conflicts.
    const int wrow = 8 * ((r32 >> 2) & 3) + 4 * ((r32 >> 4) & 1) + (r32 & 3) + 32 * rg;
    const int wr_at = wrow * PJ_STR + piece * 8, ur_at = (PJ_COLS + row0) * PJ_STR + piece * 8;
    const int a_at = (cw * 64 + l32) * PJ_STR + 8 * kg;
    int cc;                                                  // column inside the row of the wave's block
    const int ob = proj_block_of(pb, min(col0, pb.tot - 64), cc);
    uint16_t *out = (uint16_t *)pb.out[ob];
    const int ncol = pb.n[ob];                               // row length of that output

    // entries [32 p_begin, 32 p_end) of the list, at most 2 RT tiles.  SETS: stages parked in registers.
    auto run_pass = [&](auto rt_, auto sets_, int p_begin, int p_end) __attribute__((always_inline)) {
        constexpr int RT = decltype(rt_)::value, SETS = decltype(sets_)::value;
        const int ptiles = p_end - p_begin;
        const int half = (ptiles + 1) / 2;
        const int tbase = rg ? half : 0;                                 // first tile of this wave's row group
        const int nrt = rg ? ptiles - half : half;                       // its tiles, wave-uniform
        const int nvalid = min(32 * p_end, cnt) - 32 * p_begin;          // entries of this pass
        const int32_t *lst = lists + (int64_t)e * tokens + 32 * p_begin;
        const uint16_t *usrc[RT];
#pragma unroll
        for (int i = 0; i < RT; ++i) usrc[i] = u + (int64_t)(lst[min(row0 + 64 * i, nvalid - 1)] / K) * Dm;
        const int b_at = (PJ_COLS + 32 * tbase + l32) * PJ_STR + 8 * kg;
        // All loads are clamped and unconditional, so that the waits on them stay exact counts;
        // the issues past the last stage re-read it and are not used.
        uint4 wreg[SETS][4], ureg[SETS][RT];
        auto load = [&](uint4 (&wr)[4], uint4 (&ur)[RT], int k0) __attribute__((always_inline)) {
            const int kk = min(min(k0, k_last) + piece * 8, Dm - 8);   // a short last stage stays inside the row
#pragma unroll
            for (int i = 0; i < 4; ++i) wr[i] = *reinterpret_cast<const uint4 *>(wbase[i] + (wlane + kk));
#pragma unroll
            for (int i = 0; i < RT; ++i) ur[i] = *reinterpret_cast<const uint4 *>(usrc[i] + kk);
        };
        // registers -> LDS; pieces past the end of a short last stage as zeros: every stage is 4 k-steps
        auto put = [&](uint16_t *buf, const uint4 (&wr)[4], const uint4 (&ur)[RT], int k0) __attribute__((always_inline)) {
            const uint32_t m = k0 + piece * 8 < Dm ? ~0u : 0u;
#pragma unroll
            for (int i = 0; i < 4; ++i)
                *reinterpret_cast<uint4 *>(buf + wr_at + 64 * i * PJ_STR) = make_uint4(wr[i].x & m, wr[i].y & m, wr[i].z & m, wr[i].w & m);
#pragma unroll
            for (int i = 0; i < RT; ++i)
                *reinterpret_cast<uint4 *>(buf + ur_at + 64 * i * PJ_STR) = make_uint4(ur[i].x & m, ur[i].y & m, ur[i].z & m, ur[i].w & m);
        };
        pj_f32x16_t acc[2][RT];
#pragma unroll
        for (int ct = 0; ct < 2; ++ct)
#pragma unroll
            for (int rt = 0; rt < RT; ++rt) acc[ct][rt] = pj_f32x16_t{0};
        auto read_ops = [&](const uint16_t *buf, uint4 (&a)[2], uint4 (&b)[RT], int s4) __attribute__((always_inline)) {
#pragma unroll
            for (int q = 0; q < 2; ++q) a[q] = *reinterpret_cast<const uint4 *>(buf + a_at + 32 * q * PJ_STR + 16 * s4);
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
                b[rt] = *reinterpret_cast<const uint4 *>(buf + b_at + 32 * rt * PJ_STR + 16 * s4);
        };
        auto mfmas = [&](const uint4 (&a)[2], const uint4 (&b)[RT]) __attribute__((always_inline)) {
#pragma unroll
            for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                for (int ct = 0; ct < 2; ++ct)
                    acc[ct][rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        __builtin_bit_cast(pj_bf16x8_t, a[ct]), __builtin_bit_cast(pj_bf16x8_t, b[rt]),
                        acc[ct][rt], 0, 0, 0);
        };
        // One stage: multiply buf; the next one's rows go into other, behind the first MFMAs, and its registers are
        // refilled.  The operands of k-step s + 1 are read from LDS before the MFMAs of k-step s are issued (two sets
        // rotated by name).  All RT row tiles are multiplied whether the wave has that many or not (the rows are staged
        // clamped, the epilogue skips them): a branch per row tile would make every pair of MFMAs wait for its own read.
        auto stage = [&](const uint16_t *buf, uint16_t *other, uint4 (&wr)[4], uint4 (&ur)[RT], int k0) __attribute__((always_inline)) {
            lds_barrier();                       // buf is written; every wave is done with other
            uint4 a0[2], b0[RT], a1[2], b1[RT];
            read_ops(buf, a0, b0, 0);
            read_ops(buf, a1, b1, 1);
            __builtin_amdgcn_sched_barrier(0);
            mfmas(a0, b0);
            __builtin_amdgcn_sched_barrier(0);
            read_ops(buf, a0, b0, 2);
            __builtin_amdgcn_sched_barrier(0);
            put(other, wr, ur, k0 + PJ_KT);
            load(wr, ur, k0 + (1 + SETS) * PJ_KT);
            __builtin_amdgcn_sched_barrier(0);
            mfmas(a1, b1);
            __builtin_amdgcn_sched_barrier(0);
            read_ops(buf, a1, b1, 3);
            __builtin_amdgcn_sched_barrier(0);
            mfmas(a0, b0);
            mfmas(a1, b1);
        };
        // prologue in the order the loop consumes (scheduling barriers keep the issue order)
        load(wreg[0], ureg[0], 0);
        __builtin_amdgcn_sched_barrier(0);
        if (SETS == 2) load(wreg[SETS - 1], ureg[SETS - 1], PJ_KT);
        __builtin_amdgcn_sched_barrier(0);
        lds_barrier();                           // every wave is done with the pass in front
        put(s_buf, wreg[0], ureg[0], 0);
        load(wreg[0], ureg[0], SETS * PJ_KT);
        // pairs of stages (an odd count runs an all-zero one): no branch between the buffers and register sets
        for (int k0 = 0; k0 < Dm; k0 += 2 * PJ_KT) {
            stage(s_buf, s_buf + PJ_BUF, wreg[SETS - 1], ureg[SETS - 1], k0);
            stage(s_buf + PJ_BUF, s_buf, wreg[0], ureg[0], k0 + PJ_KT);
        }
        if (!active) return;
#pragma unroll
        for (int rt = 0; rt < RT; ++rt) {
            const int prow = 32 * (tbase + rt) + l32;                         // entry inside the pass
            if (rt < nrt && prow < nvalid) {
                const int64_t ent = lst[prow];                                // t*K + r
                const int64_t row = compact ? ent : (ent / K) * E + e;
#pragma unroll
                for (int ct = 0; ct < 2; ++ct) {
                    uint16_t *dst = out + row * ncol + cc + 32 * ct + 16 * kg;
                    const pj_f32x16_t v = acc[ct][rt];
                    *reinterpret_cast<uint4 *>(dst) =
                        make_uint4(pj_pack(v[0], v[1]), pj_pack(v[2], v[3]), pj_pack(v[4], v[5]), pj_pack(v[6], v[7]));
                    *reinterpret_cast<uint4 *>(dst + 8) = make_uint4(pj_pack(v[8], v[9]), pj_pack(v[10], v[11]),
                                                                     pj_pack(v[12], v[13]), pj_pack(v[14], v[15]));
                }
            }
        }
    };
    for (int pass = 0; pass < npass; ++pass) {
        const int p_begin = t_begin + (int)((int64_t)pass * nt / npass);
        const int p_end = t_begin + (int)((int64_t)(pass + 1) * nt / npass);
        if (p_end - p_begin <= 4)
            run_pass(std::integral_constant<int, 2>{}, std::integral_constant<int, 2>{}, p_begin, p_end);
        else if (p_end - p_begin <= 6)
            run_pass(std::integral_constant<int, 3>{}, std::integral_constant<int, 2>{}, p_begin, p_end);
        else
            run_pass(std::integral_constant<int, 4>{}, std::integral_constant<int, 1>{}, p_begin, p_end);
    }
}

// any shape, fp32 arithmetic: block = (token, slot), the token's features in LDS, one lane
// per output column of [B | C]
template <typename T>
__global__ void __launch_bounds__(256)
proj_generic_kernel(const T *__restrict__ u, ProjBlocks pb, const int32_t *__restrict__ idx, int E, int K,
                    int Dm, int compact)
{
    extern __shared__ float s_u[];
    const int64_t t = blockIdx.x / K;
    const int e = idx[blockIdx.x];
    const int64_t row = compact ? (int64_t)blockIdx.x : t * E + e;
    for (int d = threadIdx.x; d < Dm; d += 256) s_u[d] = to_float(u[t * Dm + d]);
    __syncthreads();
    for (int c = threadIdx.x; c < pb.tot; c += 256) {
        int cc;
        const int sb = proj_block_of(pb, c, cc);
        const T *wr = (const T *)pb.W[sb] + ((int64_t)e * pb.n[sb] + cc) * Dm;
        float acc = 0.f;
        for (int d = 0; d < Dm; ++d) acc += to_float(wr[d]) * s_u[d];
        ((T *)pb.out[sb])[row * pb.n[sb] + cc] = from_float<T>(acc);
    }
}

bool expert_proj_on_mfma(int io_dtype, int GN, int HP, int Dm)
{
    return io_dtype == SWIMBA_BF16 && Dm % 16 == 0 && GN % 64 == 0 && HP % 64 == 0;
}

// WX / Xo / HP: the third block of columns (input streams), nullptr / nullptr / 0 when not wanted
swimba_status launch_expert_proj(int64_t tokens, int E, int K, int GN, int Dm, int io_dtype, const void *u,
                                 const void *WB, const void *WC, const void *logits, void *Be, void *Ce,
                                 int32_t *idx, float *w, int32_t *counts, int32_t *lists, int compact,
                                 hipStream_t st, const void *WX, void *Xo, int HP)
{
    if (tokens == 0) return SWIMBA_OK;
    if (tokens * K > 0x7fffffffll) return SWIMBA_ERR_UNSUPPORTED;   // list entries are 32-bit
    ProjBlocks pb;
    pb.W[0] = WB; pb.W[1] = WC; pb.W[2] = WX;
    pb.out[0] = Be; pb.out[1] = Ce; pb.out[2] = Xo;
    pb.n[0] = GN; pb.n[1] = GN; pb.n[2] = WX ? HP : 0;
    pb.tot = 2 * GN + pb.n[2];
    const bool mfma = expert_proj_on_mfma(io_dtype, GN, pb.n[2], Dm);
    const unsigned rgrid = (unsigned)((tokens + 255) / 256);
    if (!mfma) {
        swimba_status rs = launch_router(tokens, E, K, io_dtype, logits, idx, w, st);
        if (rs != SWIMBA_OK) return rs;
        const size_t shm = (size_t)Dm * sizeof(float);
        if (io_dtype == SWIMBA_BF16)
            hipLaunchKernelGGL(proj_generic_kernel<bf16>, dim3((unsigned)(tokens * K)), dim3(256), shm, st,
                               (const bf16 *)u, pb, idx, E, K, Dm, compact);
        else
            hipLaunchKernelGGL(proj_generic_kernel<float>, dim3((unsigned)(tokens * K)), dim3(256), shm, st,
                               (const float *)u, pb, idx, E, K, Dm, compact);
        SWIMBA_CHECK_LAUNCH();
        return SWIMBA_OK;
    }
    hipLaunchKernelGGL(proj_clear_kernel, dim3(1), dim3(256), 0, st, counts, E);
    SWIMBA_CHECK_LAUNCH();
    hipLaunchKernelGGL(proj_route_kernel<bf16>, dim3(rgrid), dim3(256), (size_t)256 * K * sizeof(int32_t), st,
                       (const bf16 *)logits, idx, w, counts, lists, tokens, E, K);
    SWIMBA_CHECK_LAUNCH();
    // one place per compute unit (a workgroup is 8 waves with up to 256 registers each), shared
    // by the column blocks; the kernel divides them among the experts
    int devid = 0, ncu = 0;
    hipError_t he = hipGetDevice(&devid);
    if (he == hipSuccess) he = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, devid);
    if (he != hipSuccess) { set_last_hip_error((int)he); return SWIMBA_ERR_HIP; }
    const int colblocks = (pb.tot + PJ_COLS - 1) / PJ_COLS;
    const int nslots = max(1, ncu / colblocks);
    // more than 64 KB of dynamic LDS has to be allowed once per device
    static std::atomic<uint64_t> attr_set{0};                // one bit per device ordinal
    const uint64_t bit = 1ull << (devid & 63);
    if (!(attr_set.load(std::memory_order_acquire) & bit)) {
        he = hipFuncSetAttribute((const void *)proj_mfma_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)PJ_SHM);
        if (he != hipSuccess) { set_last_hip_error((int)he); return SWIMBA_ERR_HIP; }
        attr_set.fetch_or(bit, std::memory_order_release);
    }
    // the shares sum to at most nslots + E
    const unsigned grid = (unsigned)(((int64_t)(nslots + E) * colblocks + 7) / 8 * 8);
    hipLaunchKernelGGL(proj_mfma_kernel, dim3(grid), dim3(PJ_THREADS), PJ_SHM, st, (const uint16_t *)u, pb, counts, lists,
                       tokens, E, K, Dm, nslots, colblocks, compact);
    SWIMBA_CHECK_LAUNCH();
    return SWIMBA_OK;
}

// idx[t*K + r] = r: with streams stored per selected slot, slot r is "expert" r
__global__ void slot_ids_kernel(int32_t *idx, int64_t n, int K)
{
    const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) idx[i] = (int32_t)(i % K);
}

swimba_status launch_slot_ids(int32_t *idx, int64_t tokens, int K, hipStream_t st)
{
    const int64_t n = tokens * K;
    if (n == 0) return SWIMBA_OK;
    hipLaunchKernelGGL(slot_ids_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, st, idx, n, K);
    SWIMBA_CHECK_LAUNCH();
    return SWIMBA_OK;
}

}  // namespace swimba
