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
// Two launches: route every token and append the entry t*k + r to the list of its r-th expert; a
// grouped GEMM over (share of an expert's list, 256 output columns).  Above 32 experts a third one in
// front of them clears the lists' lengths.
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

// Lists of the experts' entries t*k + r, in segments: block b of the routing (tb tokens) has the tb places from b*tb on of every
// expert's list and says in counts[e][b] how many it filled, so nothing has to be cleared and no block waits for another.
// One token per lane.  The logits of 256 tokens go through LDS: the routing reads them K + 2 times, one after the other.
template <typename T>
__global__ void __launch_bounds__(256)
proj_route_segments_kernel(const T *__restrict__ logits, int32_t *__restrict__ idx, float *__restrict__ w,
                           int32_t *__restrict__ counts, int32_t *__restrict__ lists, int64_t tokens, int E, int K, int tb)
{
    __shared__ int32_t s_cnt[PJ_SEG_EXPERTS];
    extern __shared__ int32_t s_dyn[];
    int32_t *s_idx = s_dyn;                                  // [256][K]
    float *s_w = reinterpret_cast<float *>(s_idx + 256 * K); // [256][K]
    float *s_l = s_w + 256 * K;                              // [256][E | 1]
    const int tid = threadIdx.x;
    const int64_t begin = (int64_t)blockIdx.x * tb, end = min(begin + tb, tokens);
    if (tid < E) s_cnt[tid] = 0;
    for (int64_t t0 = begin; t0 < end; t0 += 256) {
        const int valid = (int)min((int64_t)256, end - t0);
        __syncthreads();
        for (int i = tid; i < valid * E; i += 256) s_l[i / E * (E | 1) + i % E] = to_float(logits[t0 * E + i]);
        __syncthreads();
        if (tid < valid) {
            const float *row = s_l + tid * (E | 1);
            int32_t *ix = s_idx + tid * K;
            route_token([&](int e) { return row[e]; }, E, K, ix, s_w + tid * K);
            for (int r = 0; r < K; ++r)
                lists[ix[r] * tokens + begin + atomicAdd(&s_cnt[ix[r]], 1)] = (int32_t)((t0 + tid) * K + r);
        }
        __syncthreads();
        for (int i = tid; i < valid * K; i += 256) {
            idx[t0 * K + i] = s_idx[i];
            w[t0 * K + i] = s_w[i];
        }
    }
    __syncthreads();
    if (tid < E) counts[tid * (int)gridDim.x + blockIdx.x] = s_cnt[tid];
}

// the same into whole lists, for many experts: counters cleared before, one global atomic per block and expert
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
// that fit on the chip at once (one per compute unit) are divided among the experts by tiles of 32
// entries (list lengths are known on the device only), and a workgroup walks its share in passes of
// up to 256 entries (2 to 4 row tiles per row group, one code path each).  The contraction runs in
// stages of 64 features: 256 weight rows and the pass's token rows, 128 bytes each, go from memory
// straight into one of the LDS buffers (1 KB an instruction, 8 rows), a stage or, where three buffers
// fit, two ahead, and from there into the lanes' operand registers: one barrier a stage.  A row's
// 16-byte pieces lie exclusive-or'ed with half its number, so that the 16 rows that 16 lanes read lie
// in different banks (with the number itself every read took twice as long).
// Against the same stages through registers and padded LDS rows, and shares by rounded-down counts: 8192 tokens x 1792 columns
// (130M-shaped layer with input streams) 78 -> 65 to 67 us, 16384 tokens x 256 columns 30 -> 27 to 29 (kernel trace).  Counters of
// the two: matrix pipes busy 32 and 16 % of the kernel's time, no bank conflicts, operand reads 28 and 16 % of what LDS carries at
// 128 bytes a clock, waves waiting for an instruction 44 and 35 % of theirs: no unit is near its rate, the waits between the
// phases of a stage are what is left.  Left out one at a time, in a build whose reads still met in LDS banks, calls (lists and
// product) of 79.6 and 42.3 us: the MFMAs 20 / 6.5, the stores of the results 11.6 / 6, the copies 9 / 4; 2.3 until a
// workgroup has its share.  Worse: all copies of a stage in front of its MFMAs (2 / 3 us), one behind each pair of
// MFMAs (4 / 5), the first wait of a pass that counts the stores in front of it (2 / 0).
constexpr int PJ_THREADS = 512;
constexpr int PJ_KT = 64;             // features per stage
constexpr int PJ_ROW = 2 * PJ_KT;     // bytes of a row in LDS
constexpr int PJ_MAX_RT = 4;          // row tiles (of 32 list entries) per wave and pass
constexpr int PJ_WBYTES = PJ_COLS * PJ_ROW;
constexpr int pj_buf(int RT) { return PJ_WBYTES + 64 * RT * PJ_ROW; }
constexpr int pj_nbuf(int RT) { return RT == 2 ? 3 : 2; }
constexpr size_t PJ_SHM = 3 * pj_buf(2);
static_assert(PJ_SHM >= 2 * pj_buf(3) && PJ_SHM >= 2 * pj_buf(4), "LDS of the widest pass");

// 16 bytes a lane from memory to LDS byte address lds (uniform) + 16 lane.  The compiler does not see these loads: it keeps its
// own waits exact or longer, and pj_wait waits for them.  m0, which holds the address, is no register that the compiler
// allocates, and it warns at the name; named, no instruction that sets m0 for its own use is moved across.
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
__device__ __forceinline__ void pj_copy(uint32_t lds, const void *base, uint32_t off)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" :: "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(off), "s"(base) : "memory", "m0");
}
__device__ __forceinline__ void pj_copy(uint32_t lds, const void *p)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(__builtin_amdgcn_readfirstlane(lds)), "v"(p) : "memory", "m0");
}
#pragma clang diagnostic pop
// until at most n vector memory operations of the wave are outstanding
template <int n> __device__ __forceinline__ void pj_wait() { __builtin_amdgcn_s_waitcnt(0x0f70 | (n & 15) | (n >> 4) << 14); }

// sum over the 64 lanes
__device__ __forceinline__ int pj_wave_sum(int v)
{
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) v += __shfl_xor(v, d);
    return v;
}

__global__ void __launch_bounds__(PJ_THREADS) __attribute__((amdgpu_waves_per_eu(2, 2)))
proj_mfma_kernel(const uint16_t *__restrict__ u, ProjBlocks pb, const int32_t *__restrict__ counts,
                 const int32_t *__restrict__ lists, int64_t tokens, int E, int K, int Dm, int nslots,
                 int colblocks, int compact, int nseg, int seg_len)
{
    extern __shared__ __align__(16) unsigned char s_buf[];   // weight rows, then token rows of each buffer
    __shared__ int32_t s_sel[4];
    __shared__ int32_t s_cnt[SWIMBA_MAX_EXPERTS];            // entries of every expert's list
    __shared__ int32_t s_seg[PJ_MAX_SEGS + 1];               // of the workgroup's expert: entries in front of each segment
    __shared__ int32_t s_ent[2][64 * PJ_MAX_RT];             // list entries of a pass
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);

    // ---- which expert, which part of its list (E <= 256 = 4 per lane) ----
    // Every workgroup gets the same number of tiles or less: the smallest even number, from the average on, with which the
    // shares fit nslots.  Where that is not found (few slots an expert) there are up to E more shares, in a second round.
    // Workgroups of one XCD (ids equal mod 8) take neighbouring shares with all their column blocks, so
    // that its L2 holds the weights of about one expert and the token rows are read into it once.
    if (tid == 0) s_sel[0] = -1;
    if (nseg == 1) {
        if (tid < E) s_cnt[tid] = counts[tid];
    } else {
        for (int e = wave; e < E; e += PJ_THREADS / 64) {
            int c[PJ_MAX_SEGS / 64], n = 0;
#pragma unroll
            for (int q = 0; q < PJ_MAX_SEGS / 64; ++q) c[q] = counts[e * nseg + min(64 * q + lane, nseg - 1)];
#pragma unroll
            for (int q = 0; q < PJ_MAX_SEGS / 64; ++q) n += 64 * q + lane < nseg ? c[q] : 0;
            n = pj_wave_sum(n);
            if (lane == 0) s_cnt[e] = n;
        }
    }
    __syncthreads();
    if (wave == 0) {
        int tiles[4], sum = 0, v[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) { tiles[q] = 4 * lane + q < E ? (s_cnt[4 * lane + q] + 31) / 32 : 0; sum += tiles[q]; }
        const int all = pj_wave_sum(sum);
        int per = max(2, 2 * ((all + 2 * nslots - 1) / (2 * nslots)));
        for (int tries = 0;; ++tries) {
            sum = 0;
#pragma unroll
            for (int q = 0; q < 4; ++q) { v[q] = (tiles[q] + per - 1) / per; sum += v[q]; }
            if (tries == 6 || pj_wave_sum(sum) <= nslots) break;
            per += max(2, per / 16 * 2);
        }
        int incl = sum;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int t = __shfl_up(incl, d);
            if (lane >= d) incl += t;
        }
        const int used = __builtin_amdgcn_readlane(incl, 63) * colblocks, each = (used + 7) / 8;
        const int j = (int)blockIdx.x >> 3, lid = ((int)blockIdx.x & 7) * each + j;
        int r = lid / colblocks - (incl - sum);
        if (j < each && lid < used && r >= 0 && r < sum) {
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                if (r >= 0 && r < v[q]) { s_sel[0] = 4 * lane + q; s_sel[1] = r; s_sel[2] = lid % colblocks; s_sel[3] = v[q]; }
                r -= v[q];          // negative from the match on: no later q matches
            }
        }
    }
    __syncthreads();
    const int e = __builtin_amdgcn_readfirstlane(s_sel[0]);
    if (e < 0) return;                                       // whole workgroup: no barrier is skipped
    const int part = __builtin_amdgcn_readfirstlane(s_sel[1]), nparts = __builtin_amdgcn_readfirstlane(s_sel[3]);
    const int cnt = s_cnt[e];
    const int n32 = (cnt + 31) / 32;
    const int t_begin = (int)((int64_t)part * n32 / nparts), t_end = (int)((int64_t)(part + 1) * n32 / nparts);
    const int nt = t_end - t_begin;
    if (nt <= 0) return;
    const int npass = (nt + 2 * PJ_MAX_RT - 1) / (2 * PJ_MAX_RT);
    if (nseg > 1) {
        if (wave == 0) {
            int c[PJ_MAX_SEGS / 64], n = 0;                  // four segments a lane
#pragma unroll
            for (int q = 0; q < 4; ++q) { c[q] = counts[e * nseg + min(4 * lane + q, nseg - 1)]; n += 4 * lane + q < nseg ? c[q] : 0; }
            int in_front = n;
#pragma unroll
            for (int d = 1; d < 64; d <<= 1) {
                const int t = __shfl_up(in_front, d);
                if (lane >= d) in_front += t;
            }
            in_front -= n;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                if (4 * lane + q < nseg) { s_seg[4 * lane + q] = in_front; in_front += c[q]; }
        }
        __syncthreads();
    }
    // entry r of the list
    auto entry_at = [&](int r) __attribute__((always_inline)) {
        if (nseg == 1) return r;
        int seg = 0;                                         // the last one with at most r entries in front
#pragma unroll
        for (int d = PJ_MAX_SEGS / 2; d > 0; d >>= 1)
            if (seg + d < nseg && s_seg[seg + d] <= r) seg += d;
        return seg * seg_len + r - s_seg[seg];
    };

    const int cw = wave & 3, rg = wave >> 2;                 // column group, row group of the wave
    const int colblk = __builtin_amdgcn_readfirstlane(s_sel[2]) * PJ_COLS;   // first column of the workgroup in [B | C | X]
    const int col0 = colblk + cw * 64;
    const bool active = col0 < pb.tot;                       // wave-uniform; idle waves still stage
    const int l32 = lane & 31, kg = lane >> 5;

    // ---- staging map: a wave copies 8 rows an instruction, lane -> piece pieces[row / 8 % 2] of row r8 of them ----
    const int r8 = lane >> 3, pieces[2] = {(lane & 7) ^ (r8 >> 1), (lane & 7) ^ (4 + (r8 >> 1))};
    // A wave stages the 32 rows of one column tile, which lie in one weight tensor: a uniform base and a per-lane offset.
    // Operand row r of a tile must hold column 16*((r>>2)&1) + 4*(r>>3) + (r&3) for accumulator register v of lane (l32, kg)
    // to be column 16 kg + v of the tile: row 8 i + r8 is 4 i more than the lane's first.
    const char *wbase;
    {
        int cl;
        const int sb = proj_block_of(pb, min(colblk + 32 * wave, pb.tot - 32), cl);   // past the end: the last rows again
        wbase = (const char *)((const uint16_t *)pb.W[sb] + ((int64_t)e * pb.n[sb] + cl) * Dm);
    }
    const uint32_t wlane = (uint32_t)(16 * (r8 >> 2) + (r8 & 3)) * Dm * 2;
    const uint32_t lds0 = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)s_buf);
    const int stages = (Dm + PJ_KT - 1) / PJ_KT;
    const int xo = kg ^ ((l32 >> 1) & 7);                           // of k-step s: pieces (2 s) ^ xo
    int cc;                                                  // column inside the row of the wave's block
    const int ob = proj_block_of(pb, min(col0, pb.tot - 64), cc);
    uint16_t *out = (uint16_t *)pb.out[ob];
    const int ncol = pb.n[ob];                               // row length of that output
    const int32_t *list = lists + (int64_t)e * tokens;

    auto run = [&](auto rt_) __attribute__((always_inline)) {
        constexpr int RT = decltype(rt_)::value, BUF = pj_buf(RT), NBUF = pj_nbuf(RT), LOADS = 4 + RT;
        auto first_tile = [&](int pass) __attribute__((always_inline)) { return t_begin + (int)((int64_t)pass * nt / npass); };
        // the list entries whose token rows the lane copies
        auto entries = [&](int32_t (&row)[RT], int pass) __attribute__((always_inline)) {
            const int begin = 32 * first_tile(pass), last = min(32 * first_tile(pass + 1), cnt) - 1;
#pragma unroll
            for (int i = 0; i < RT; ++i) row[i] = list[entry_at(min(begin + 8 * (RT * wave + i) + r8, last))];
        };
        // kept for the pass's results, and turned into tokens
        auto to_tokens = [&](int32_t (&row)[RT], int pass) __attribute__((always_inline)) {
#pragma unroll
            for (int i = 0; i < RT; ++i) {
                if ((lane & 7) == 0) s_ent[pass & 1][8 * (RT * wave + i) + r8] = row[i];
                row[i] /= K;
            }
        };
        int32_t row[RT], next_row[RT];
        int slot = 0;                                        // buffer of the next stage to be copied
        auto copy_weights = [&](int st) __attribute__((always_inline)) {
            uint32_t at_piece[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) at_piece[i] = wlane + 2 * min(st * PJ_KT + pieces[i] * 8, Dm - 8);   // a short last stage stays inside the row
            const uint32_t at = lds0 + slot * BUF + wave * (32 * PJ_ROW);
#pragma unroll
            for (int i = 0; i < 4; ++i) pj_copy(at + i * 8 * PJ_ROW, wbase + (int64_t)i * 8 * Dm, at_piece[i & 1]);
        };
        auto copy_tokens = [&](int st) __attribute__((always_inline)) {
            const int odd = (RT * wave) & 1;                 // of the wave's first 8 rows
            const uint16_t *from[2] = {u + min(st * PJ_KT + pieces[0] * 8, Dm - 8), u + min(st * PJ_KT + pieces[1] * 8, Dm - 8)};
            const uint32_t at = lds0 + slot * BUF + PJ_WBYTES + wave * (8 * RT * PJ_ROW);
#pragma unroll
            for (int i = 0; i < RT; ++i) pj_copy(at + i * 8 * PJ_ROW, ((i + odd) & 1 ? from[1] : from[0]) + (int64_t)row[i] * Dm);
            slot = slot == NBUF - 1 ? 0 : slot + 1;
        };
        entries(row, 0);
        to_tokens(row, 0);
#pragma unroll
        for (int st = 0; st < NBUF - 1; ++st)
            if (st < stages) {
                copy_weights(st);
                copy_tokens(st);
            }
        int buf = 0;                                         // of the stage that is multiplied
        for (int pass = 0; pass < npass; ++pass) {
            const int begin = first_tile(pass), end = first_tile(pass + 1);
            const int ptiles = end - begin, half = (ptiles + 1) / 2;
            const int tbase = rg ? half : 0;                                 // first tile of this wave's row group
            const int nrt = rg ? ptiles - half : half;                       // its tiles, wave-uniform
            const bool more = NBUF == 2 && pass + 1 < npass;                 // two tiles a group: one pass
            if (more) entries(next_row, pass + 1);
            const unsigned char *a_at = s_buf + (cw * 64 + l32) * PJ_ROW, *b_at = s_buf + PJ_WBYTES + (32 * tbase + l32) * PJ_ROW;
            pj_f32x16_t acc[2][RT];
#pragma unroll
            for (int ct = 0; ct < 2; ++ct)
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) acc[ct][rt] = pj_f32x16_t{0};
            auto stage = [&](int st, auto whole_) __attribute__((always_inline)) {
                // with three buffers the next stage may be under way
                if (NBUF == 3 && st + 1 < stages) pj_wait<LOADS>();
                else pj_wait<0>();
                lds_barrier();                               // the stage is in LDS; every wave is done with the one in front
                const int at = buf * BUF;
                uint4 a0[2], b0[RT], a1[2], b1[RT];
                auto read_ops = [&](uint4 (&a)[2], uint4 (&b)[RT], int s4) __attribute__((always_inline)) {
                    const int o = at + (((2 * s4) ^ xo) << 4);
#pragma unroll
                    for (int k = 0; k < 2; ++k) a[k] = *reinterpret_cast<const uint4 *>(a_at + o + 32 * k * PJ_ROW);
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt) b[rt] = *reinterpret_cast<const uint4 *>(b_at + o + 32 * rt * PJ_ROW);
                };
                // All RT row tiles are multiplied whether the wave has that many or not (the rows are staged clamped, the
                // epilogue skips them): a branch per row tile would make every pair of MFMAs wait for its own read.
                auto mfmas = [&](const uint4 (&a)[2], const uint4 (&b)[RT]) __attribute__((always_inline)) {
#pragma unroll
                    for (int rt = 0; rt < RT; ++rt)
#pragma unroll
                        for (int ct = 0; ct < 2; ++ct)
                            acc[ct][rt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(pj_bf16x8_t, a[ct]),
                                                                                  __builtin_bit_cast(pj_bf16x8_t, b[rt]), acc[ct][rt], 0, 0, 0);
                };
                const int ahead = st + NBUF - 1;
                const bool copies = ahead < stages || more;
                const int ast = ahead < stages ? ahead : ahead - stages;
                if (ahead == stages && more) {
#pragma unroll
                    for (int i = 0; i < RT; ++i) row[i] = next_row[i];
                    to_tokens(row, pass + 1);
                }
                if constexpr (decltype(whole_)::value) {
                    read_ops(a0, b0, 0);
                    read_ops(a1, b1, 1);
                    __builtin_amdgcn_sched_barrier(0);
                    if (copies) copy_weights(ast);
                    mfmas(a0, b0);
                    __builtin_amdgcn_sched_barrier(0);
                    if (copies) copy_tokens(ast);
                    read_ops(a0, b0, 2);
                    __builtin_amdgcn_sched_barrier(0);
                    mfmas(a1, b1);
                    __builtin_amdgcn_sched_barrier(0);
                    read_ops(a1, b1, 3);
                    __builtin_amdgcn_sched_barrier(0);
                    mfmas(a0, b0);
                    mfmas(a1, b1);
                } else {
                    if (copies) {
                        copy_weights(ast);
                        copy_tokens(ast);
                    }
#pragma unroll 1
                    for (int s4 = 0; s4 < (Dm - st * PJ_KT) / 16; ++s4) {
                        read_ops(a0, b0, s4);
                        mfmas(a0, b0);
                    }
                }
                buf = buf == NBUF - 1 ? 0 : buf + 1;
            };
            int st = 0;
            for (; st < Dm / PJ_KT; ++st) stage(st, std::true_type{});
            if (st < stages) stage(st, std::false_type{});
            if (active) {
                const int nvalid = min(32 * end, cnt) - 32 * begin;          // entries of this pass
#pragma unroll
                for (int rt = 0; rt < RT; ++rt) {
                    const int prow = 32 * (tbase + rt) + l32;                    // entry inside the pass
                    if (rt < nrt && prow < nvalid) {
                        const int64_t ent = s_ent[pass & 1][prow];               // t*K + r
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
            }
        }
    };
    // Several passes have more than four tiles each, so two tiles a group are always one pass: its three buffers need not look
    // past it.
    const int widest = (nt + npass - 1) / npass;
    if (nt <= 4) run(std::integral_constant<int, 2>{});
    else if (widest <= 6) run(std::integral_constant<int, 3>{});
    else run(std::integral_constant<int, 4>{});
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
    int devid = 0, ncu = 0;
    hipError_t he = hipGetDevice(&devid);
    if (he == hipSuccess) he = hipDeviceGetAttribute(&ncu, hipDeviceAttributeMultiprocessorCount, devid);
    if (he != hipSuccess) { set_last_hip_error((int)he); return SWIMBA_ERR_HIP; }
    // more than 64 KB of dynamic LDS has to be allowed once per device: the product's, and the lists' of 32 experts and 16 slots
    auto route_shm = [](int K, int E) { return (size_t)256 * (2 * K + (E | 1)) * 4; };
    static std::atomic<uint64_t> attr_set{0};                // one bit per device ordinal
    const uint64_t bit = 1ull << (devid & 63);
    if (!(attr_set.load(std::memory_order_acquire) & bit)) {
        he = hipFuncSetAttribute((const void *)proj_mfma_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)PJ_SHM);
        if (he == hipSuccess)
            he = hipFuncSetAttribute((const void *)proj_route_segments_kernel<bf16>, hipFuncAttributeMaxDynamicSharedMemorySize,
                                     (int)route_shm(SWIMBA_MAX_TOPK, PJ_SEG_EXPERTS));
        if (he != hipSuccess) { set_last_hip_error((int)he); return SWIMBA_ERR_HIP; }
        attr_set.fetch_or(bit, std::memory_order_release);
    }
    const int nseg = proj_segments(tokens, E), seg_len = (int)proj_seg_len(tokens);
    if (E <= PJ_SEG_EXPERTS) {
        hipLaunchKernelGGL(proj_route_segments_kernel<bf16>, dim3(nseg), dim3(256), route_shm(K, E), st,
                           (const bf16 *)logits, idx, w, counts, lists, tokens, E, K, seg_len);
    } else {
        hipLaunchKernelGGL(proj_clear_kernel, dim3(1), dim3(256), 0, st, counts, E);
        SWIMBA_CHECK_LAUNCH();
        hipLaunchKernelGGL(proj_route_kernel<bf16>, dim3(rgrid), dim3(256), (size_t)256 * K * sizeof(int32_t), st,
                           (const bf16 *)logits, idx, w, counts, lists, tokens, E, K);
    }
    SWIMBA_CHECK_LAUNCH();
    // one place per compute unit (a workgroup is 8 waves with up to 256 registers each), shared
    // by the column blocks; the kernel divides them among the experts
    const int colblocks = (pb.tot + PJ_COLS - 1) / PJ_COLS;
    const int nslots = max(1, ncu / colblocks);
    // the shares sum to at most nslots + E: each but one of an expert has the average of tiles a slot or more
    const unsigned grid = (unsigned)(((int64_t)(nslots + E) * colblocks + 7) / 8 * 8);
    hipLaunchKernelGGL(proj_mfma_kernel, dim3(grid), dim3(PJ_THREADS), PJ_SHM, st, (const uint16_t *)u, pb, counts, lists,
                       tokens, E, K, Dm, nslots, colblocks, compact, nseg, seg_len);
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
