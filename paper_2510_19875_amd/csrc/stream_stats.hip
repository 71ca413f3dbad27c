// stream_receiver_stats: block means of a head's dense attention pattern and their vertical
// kurtosis (Section 4.1, "Thought Anchors": receiver heads) on gfx950.
//
// The T x T probability matrix is never stored, and every score is computed once.  A wavefront owns up
// to 64 queries of a head, keeps their fragments in registers and streams the visible 64-key tiles
// (32x32 MFMA, S^T = K Q^T: a lane owns a query column).  Per query and key block it writes the sum
// of the exponentials, relative to a reference that is fixed for the row, to a scratch row of its own;
// when the row is through its normalisers are known, and the scratch is read back (by the wavefront
// that wrote it) to form the sums of the normalised probabilities over every span.  A second kernel turns
// the sums into means and adds up their powers per column, in fp64 and shifted by the column's first
// value; a third, tiny one reduces the column statistics to the two numbers per (head, sequence).
// Memory O(T): the scratch belongs to the wavefronts in flight, and the sums are kept for a chunk of
// query blocks at a time.  Where the workspace has no room for the scratch every score is computed twice
// instead: once for the normalisers, once more for the spans.
#include "stream_mfma.h"

#include <math.h>

namespace stream {

struct StatsParams {
    const char *Q, *Kp;         // Q as given; K packed fragments [kv_heads][global block][b * d]
    long long q_sh_b, q_st_b;   // byte strides of Q (head, token)
    float *scratch;             // per wavefront of the row kernel: scratch_wave floats (nullptr: none, see below)
    long long scratch_wave;
    float *sums;                // [heads, (qb1 - qb0) * subs, NBk]: span sums of this chunk, per query tile
    int *queue;                 // [kXcds]: row groups handed out so far (zero before the first chunk, zeroed by the second kernel)
    double *state;              // [6, heads, NBk]: count, shift, four power sums between chunks (nullptr: one chunk)
    float *block_mean;          // nullable [heads, NB, NBk]
    float *col_mean, *col_kurt; // [heads, NBk]
    float *head_stats;          // [heads, batch, 2]
    float c;                    // scale * log2(e)
    int H, g, NB, b;            // NB query blocks of b = b_q tokens
    int NBk, bk;                // NBk key blocks of b_k tokens (NB * b = NBk * bk padded tokens)
    int qb0, qb1;               // the chunk: query blocks qb0 .. qb1 - 1
    int mask, window;
    // STREAM_MASK_ARRAY (ARB kernels): the bit array C, the "some pair visible" summary per (query
    // block, key block), and the number of query blocks every column is defined on
    const unsigned *cbits, *cany;
    long long cpitch;
    int cw;
    int *col_n;                 // [heads, NBk]
    WgMap map;
    SeqTable seqs;
};
static_assert(sizeof(StatsParams) <= 4096, "kernel arguments are limited to 4 KB");

// Query blocks (of bq tokens) that can see key block j (of bk tokens) of a sequence of L tokens:
// imin .. imax, contiguous for all three mask rules (the counterpart of mask_rmin / mask_rmax);
// imin > imax for a key block of padding only.
__host__ __device__ __forceinline__ void mask_irange(int mask, int window, int j, int bq, int bk, int L,
                                                     int &imin, int &imax)
{
    const long long k_first = (long long)j * bk;
    if (k_first >= L) { imin = 0; imax = -1; return; }
    // causal rules: the first query block whose last query is at or after the block's first key
    imin = mask == STREAM_MASK_FULL ? 0 : (int)(k_first / bq);
    long long hi = ((long long)L - 1) / bq;                       // last query block with a real token
    if (mask == STREAM_MASK_SLIDING) {
        // the block's last key, j*bk + bk - 1, is seen by queries < j*bk + bk - 1 + window
        const long long w = (k_first + bk + window - 2) / bq;
        hi = w < hi ? w : hi;
    }
    imax = (int)hi;
}

// ---------------------------------------------------------------------------------------------
// Sums over the spans of one query tile (see above).  NS = 32-query groups per wavefront (1 for block
// 32).  BK32: key blocks of 32 keys, two scratch rows per 64-key tile instead of one.
// ARB: the mask is an explicit bit array: the tiles between the first and the last key block the
// query block sees are streamed and every element takes its bit (a lane owns a query: one mask word
// per 32 keys).  A query that sees no key has a zero row of probabilities.
// SCRATCH: the sums per query wait in scratch for the normalisers; else the scores are computed twice.
//
// Per element one fused multiply-add, one exp2 (8 cycles) and one add, besides 16 cycles of MFMA for 16
// of them: vector ALU and matrix core are about equally loaded, so two wavefronts share a SIMD.  With the
// running maximum in the loop and a second pass over all scores for the spans, 32 k tokens on 32/8 heads
// took 4.57 + 5.04 ms; see stats_wgs for the time of this form.
//
// The normaliser is added up in fp64 (one addition per tile) and a span's sum in four parts: error of the block
// means against 64 bits 0.5e-7, of the column kurtosis 1.7e-7 (16 k tokens, 12/2 heads; added up in fp32 in one
// row each 1.2e-7 and 3.9e-7; time the same).
//
// The reference exponent of a query is the maximum of the first tile in which it sees a key; any
// magnitude fp32 holds may follow.  Should a sum overflow, the row is run again: once for the true maxima,
// then with those as references.
//
// The grid is as large as the chip holds; a workgroup takes row groups (the heads of a KV group at one
// query tile, which read the same keys) from a queue per XCD, longest first.  (Dealt out beforehand, 8
// per workgroup and equally long in sum, they left SIMDs with one wavefront for the last third of the
// launch: of two wavefronts on a SIMD one is served first and ends first.)
template <bool BF16, int D, int NS, int OCC, bool ARB, bool BK32, bool SCRATCH>
__global__ void __launch_bounds__(256, OCC) stats_rows_kernel(const StatsParams p)
{
    constexpr int ES = BF16 ? 2 : 4;
    constexpr int FR = D * ES / 32;                 // fragments per 32-token group
    constexpr int GROUP_BYTES = 32 * D * ES;
    constexpr int QT = 32 * NS;                     // queries of this wavefront
    constexpr int RPT = BK32 ? 2 : 1;               // scratch rows per 64-key tile
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const unsigned lane_off = lane * 16;
    const int subs = p.b / QT;                      // query tiles per block
    const long long items_per_kv = (long long)(p.qb1 - p.qb0) * subs * p.g;
    float *scr = SCRATCH ? p.scratch + ((long long)blockIdx.x * 4 + wave) * p.scratch_wave : nullptr;
    // (a workgroup stays on the kv heads of its XCD)
    __shared__ int s_next;
    const int xcd = blockIdx.x % kXcds;
    for (;;) {
        if (threadIdx.x == 0) s_next = atomicAdd(p.queue + xcd, 1);
        __syncthreads();
        const int vwg = xcd + kXcds * __builtin_amdgcn_readfirstlane(s_next);
        __syncthreads();
        if (vwg >= p.map.grid) break;
        int kvh, slot;
        if (!wg_decode(p.map, vwg, kvh, slot)) continue;
        const long long rk = (long long)slot * 4 + wave;
        if (rk >= items_per_kv) continue;
        const long long tile_id = (long long)(p.qb1 - p.qb0) * subs - 1 - rk / p.g;    // long rows first
        const int h = kvh * p.g + (int)(rk % p.g);
        const int gb = p.qb0 + (int)(tile_id / subs), sub = (int)(tile_id % subs);
        const SeqDesc sd = p.seqs.d[seq_of_block(p.seqs, gb)];
        const int L = sd.len, qb = gb - sd.blk0;
        const int tq0 = qb * p.b + sub * QT;
        const int kblk0 = (int)((long long)sd.blk0 * p.b / p.bk);
        // key blocks of this query block: the spans whose sums the second kernel reads
        int j_lo = mask_rmin(p.mask, p.window, qb, p.b, p.bk), j_hi = mask_rmax(p.mask, qb, p.b, p.bk, L);
        if constexpr (ARB) {
            // from the first to the last key block some query of this block sees (the block summary of
            // the array): a causal or a document mask then costs its triangle, not the square
            const unsigned *anyrow = p.cany + (long long)gb * p.cw;
            const int nkb = (int)(((long long)sd.nblk * p.b) / p.bk);      // key blocks of the sequence
            j_lo = 0; j_hi = -1;
            for (int w0 = 0; w0 * 32 < nkb; w0 += 64) {
                const int widx = w0 + lane;
                const unsigned x = widx * 32 < nkb ? anyrow[widx] : 0u;
                const unsigned long long nz = __ballot(x != 0u);
                if (nz) {
                    const int wf = w0 + __builtin_ctzll(nz), wl = w0 + 63 - __builtin_clzll(nz);
                    if (j_hi < 0) j_lo = wf * 32 + __builtin_ctz(__builtin_amdgcn_readlane(x, wf - w0));
                    j_hi = wl * 32 + 31 - __builtin_clz(__builtin_amdgcn_readlane(x, wl - w0));
                }
            }
        }
        if (j_hi < j_lo) continue;                      // a block of padding only, or one that sees nothing
        float *sums = p.sums + ((long long)h * (p.qb1 - p.qb0) * subs + (long long)(gb - p.qb0) * subs + sub) * p.NBk + kblk0;
        if (tq0 >= L) {                                 // a tile of padding only in a block that is not
            for (int j = j_lo + lane; j <= j_hi; j += 64) sums[j] = 0.f;
            continue;
        }
        // visible 64-key tiles of these queries
        int kt_lo, kt_hi;
        if constexpr (ARB) {
            kt_lo = (int)((long long)j_lo * p.bk / 64);
            kt_hi = (int)((((long long)j_hi + 1) * p.bk - 1) / 64);
            if (kt_hi > (L - 1) / 64) kt_hi = (L - 1) / 64;
        } else {
            const int last_q = tq0 + QT - 1 < L - 1 ? tq0 + QT - 1 : L - 1;
            const int hi_tok = p.mask == STREAM_MASK_FULL ? L - 1 : last_q;
            const int lo_tok = p.mask == STREAM_MASK_SLIDING && tq0 - p.window + 1 > 0 ? tq0 - p.window + 1 : 0;
            kt_lo = lo_tok / 64; kt_hi = hi_tok / 64;
        }
        const __amdgpu_buffer_rsrc_t krs = make_tile_rsrc(
            p.Kp + ((long long)kvh * p.NB + sd.blk0) * p.b * D * ES, (unsigned)((long long)sd.nblk * p.b * D * ES));
        uint4 qf[NS][FR];
        {
            // (rows past the end of the sequence repeat the last one: every score of theirs is masked)
            const int qrows = L - tq0 < QT ? L - tq0 : QT;
#pragma unroll
            for (int qs = 0; qs < NS; ++qs) {
                const int row = qs * 32 + (lane & 31);
                const char *src = p.Q + (long long)h * p.q_sh_b + (sd.tok0 + tq0 + (row < qrows ? row : qrows - 1)) * p.q_st_b + (lane >> 5) * 16;
#pragma unroll
                for (int fr = 0; fr < FR; ++fr) qf[qs][fr] = *reinterpret_cast<const uint4 *>(src + fr * 32);
            }
        }
        float m[NS];                                    // reference per query (log2 domain)
        double l = 0.0;                                 // lane t: sum of query t's exponentials (NS == 1: lanes below 32)
        float inv = 0.f;                                // ... and 1 / l
#pragma unroll
        for (int qs = 0; qs < NS; ++qs) m[qs] = -INFINITY;
        // 0: first attempt, references set on the way; 1: true maxima only; 2: references given; 3 (no
        // scratch): references and normalisers given, the spans' sums are formed tile by tile
        for (int mode = 0;;) {
            float span = 0.f;                           // mode 3: sum of the span so far (blocks of 128 keys: two tiles)
            if (mode < 3) l = 0.0;
            bool track = mode == 0;                     // wave-uniform: some query has no reference yet
            uint4 kf[2][FR];
#pragma unroll
            for (int fr = 0; fr < FR; ++fr)
#pragma unroll
                for (int kb = 0; kb < 2; ++kb) {
                    kf[kb][fr] = load_frag(krs, lane_off, (unsigned)kt_lo * 2u * GROUP_BYTES, kb * FR + fr);
                    __builtin_amdgcn_sched_barrier(0);
                }
            for (int kt = kt_lo; kt <= kt_hi; ++kt) {
                const unsigned nxt = (unsigned)(kt < kt_hi ? kt + 1 : kt) * 2u * GROUP_BYTES;
                const int tk0 = kt * 64;
                unsigned cwd[NS][2];                    // ARB: this lane's queries against the tile's two key groups
                if constexpr (ARB) {
#pragma unroll
                    for (int qs = 0; qs < NS; ++qs) {
                        const int tq = tq0 + qs * 32 + (lane & 31);
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb)
                            cwd[qs][kb] = (tq < L && tk0 + kb * 32 < L) ? p.cbits[(long long)tq * p.cpitch + (tk0 >> 5) + kb] : 0u;
                    }
                }
                floatx16 acc[2][NS];
#pragma unroll
                for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                    for (int qs = 0; qs < NS; ++qs)
#pragma unroll
                        for (int i = 0; i < 16; ++i) acc[kb][qs][i] = 0.f;
#pragma unroll
                for (int fr = 0; fr < FR; ++fr) {
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
                        for (int qs = 0; qs < NS; ++qs)
                            acc[kb][qs] = mfma_frag<BF16>(kf[kb][fr], qf[qs][fr], acc[kb][qs]);
                        // consumed: refill from the next tile so that it has a whole tile of MFMA time
                        __builtin_amdgcn_sched_barrier(0);
                        kf[kb][fr] = load_frag(krs, lane_off, nxt, kb * FR + fr);
                        __builtin_amdgcn_sched_barrier(0);
                    }
                }
                const bool cut = ARB | (tq0 + QT > L) | (tk0 + 64 > L) |
                                 ((p.mask != STREAM_MASK_FULL) & (tk0 + 63 > tq0)) |
                                 ((p.mask == STREAM_MASK_SLIDING) & (tq0 + QT - 1 - tk0 >= p.window));
                // accumulator layout: lane holds query column (lane % 32); element i is key row
                // 8*(i/4) + 4*(lane/32) + (i%4)
                if (cut) {
#pragma unroll
                    for (int qs = 0; qs < NS; ++qs)
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                            for (int i = 0; i < 16; ++i) {
                                const int tq = tq0 + qs * 32 + (lane & 31);
                                const int kr = (i >> 2) * 8 + (lane >> 5) * 4 + (i & 3), tk = tk0 + kb * 32 + kr;
                                bool vis = (tq < L) & (tk < L);
                                if constexpr (ARB) vis = vis & ((cwd[qs][kb] >> kr) & 1u);
                                else vis = vis & mask_token(p.mask, p.window, tq, tk);
                                acc[kb][qs][i] = vis ? acc[kb][qs][i] : -INFINITY;
                            }
                }
                if (track | (mode == 1)) {
                    bool unset = false;
#pragma unroll
                    for (int qs = 0; qs < NS; ++qs) {
                        float mx = -INFINITY;
#pragma unroll
                        for (int kb = 0; kb < 2; ++kb)
#pragma unroll
                            for (int i = 0; i < 16; ++i) mx = fmaxf(mx, acc[kb][qs][i]);
                        mx = fmaxf(mx, __shfl_xor(mx, 32)) * p.c;
                        m[qs] = mode == 1 ? fmaxf(m[qs], mx) : (m[qs] == -INFINITY ? mx : m[qs]);
                        unset = unset | (m[qs] == -INFINITY);
                    }
                    track = mode == 0 && __any(unset);
                    if (mode == 1) continue;
                }
                float part[2][NS];                       // sums over this lane half's keys of a group
#pragma unroll
                for (int qs = 0; qs < NS; ++qs) {
                    const float m_use = m[qs] == -INFINITY ? 0.f : m[qs];
#pragma unroll
                    for (int kb = 0; kb < 2; ++kb) {
                        float sum = 0.f;
#pragma unroll
                        for (int i = 0; i < 16; ++i) sum += __builtin_amdgcn_exp2f(fmaf(acc[kb][qs][i], p.c, -m_use));
                        part[kb][qs] = sum;
                    }
                }
#pragma unroll
                for (int rr = 0; rr < RPT; ++rr) {
                    float v;
                    if constexpr (NS == 2) {
                        // both halves' sums of both query groups -> lane t holds query t's
                        const float a0 = BK32 ? part[rr][0] : part[0][0] + part[1][0], a1 = BK32 ? part[rr][1] : part[0][1] + part[1][1];
                        const auto sw = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, a0), __builtin_bit_cast(unsigned, a1), false, false);
                        const unsigned lo = sw[0], hi = sw[1];    // (by value: a bit cast of a vector's element reads element 0)
                        v = __builtin_bit_cast(float, lo) + __builtin_bit_cast(float, hi);
                    } else {
                        v = BK32 ? part[rr][0] : part[0][0] + part[1][0];
                        v += __shfl_xor(v, 32);
                    }
                    if (!SCRATCH && mode == 3) {
                        const int j = p.bk == 32 ? kt * 2 + rr : (p.bk == 64 ? kt : kt >> 1);
                        const float sum = wave_sum(NS == 2 || lane < 32 ? v * inv : 0.f);
                        span = (p.bk == 128 && (kt & 1)) ? span + sum : sum;
                        if (lane == 0 && j >= j_lo && j <= j_hi) sums[j] = span;
                        continue;
                    }
                    l += (double)v;
                    if (SCRATCH && (NS == 2 || lane < 32)) scr[((kt - kt_lo) * RPT + rr) * QT + (NS == 2 ? lane : lane & 31)] = v;
                }
            }
            if (!SCRATCH && mode == 3) break;
            if (mode == 1) { mode = 2; continue; }
            bool seen = m[0] != -INFINITY;
            if constexpr (NS == 2) seen = lane < 32 ? m[0] != -INFINITY : m[1] != -INFINITY;
            if (mode == 0 && __any(seen & (!(l > 1e-30) | !(l < 3e38)))) { mode = 1; continue; }
            inv = l == 0.0 ? 0.f : (float)(1.0 / l);    // (a NaN stays one)
            if (SCRATCH) break;
            mode = 3;
        }
        if constexpr (!SCRATCH) {
            const int jf = (int)((long long)kt_lo * 64 / p.bk), jl = (int)(((long long)kt_hi * 64 + 63) / p.bk);
            for (int j = j_lo + lane; j <= j_hi; j += 64)
                if (j < jf || j > jl) sums[j] = 0.f;    // blocks these queries do not reach
            continue;
        }

        // span sums of the normalised probabilities: lane j of a chunk of 64 key blocks reads the row of
        // its block from the scratch (all of a row's 64 queries, four at a time)
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");
        const int nrows = (kt_hi - kt_lo + 1) * RPT, ksub = p.bk > 64 ? 2 : 1;
        for (int j0 = j_lo; j0 <= j_hi; j0 += 64) {
            const int j = j0 + lane;
            float s = 0.f;
            for (int ks = 0; ks < ksub; ++ks) {
                const int row = j * ksub + ks - kt_lo * RPT;
                const bool in = (j <= j_hi) & (row >= 0) & (row < nrows);
                const float4 *src = reinterpret_cast<const float4 *>(scr + (long long)(in ? row : 0) * QT);
                float4 v[QT / 4];
#pragma unroll
                for (int t4 = 0; t4 < QT / 4; ++t4) v[t4] = src[t4];
                float a[4] = {0.f, 0.f, 0.f, 0.f};      // (four sums of a quarter each: less rounding than one)
#pragma unroll
                for (int t4 = 0; t4 < QT / 4; ++t4) {
                    a[0] = fmaf(v[t4].x, __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, inv), t4 * 4 + 0)), a[0]);
                    a[1] = fmaf(v[t4].y, __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, inv), t4 * 4 + 1)), a[1]);
                    a[2] = fmaf(v[t4].z, __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, inv), t4 * 4 + 2)), a[2]);
                    a[3] = fmaf(v[t4].w, __builtin_bit_cast(float, __builtin_amdgcn_readlane(__builtin_bit_cast(int, inv), t4 * 4 + 3)), a[3]);
                }
                s += in ? (a[0] + a[1]) + (a[2] + a[3]) : 0.f;
            }
            if (j <= j_hi) sums[j] = s;
        }
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "workgroup");   // the next row overwrites the scratch
    }
}

// ---------------------------------------------------------------------------------------------
// columns: block means of the chunk and the moments of every column.  A lane owns a key block, the four
// wavefronts of a workgroup share its query blocks.  Bound: reading the sums once.
// ---------------------------------------------------------------------------------------------
template <bool ARB>
__global__ void __launch_bounds__(256) stats_cols_kernel(const StatsParams p)
{
    __shared__ double s_part[4][5][64];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x < kXcds) p.queue[threadIdx.x] = 0;   // for the next chunk
    const int h = blockIdx.y;
    const int gbj = blockIdx.x * 64 + lane;
    const bool live = gbj < p.NBk;
    // the sequence that owns this key block (lanes of a workgroup may lie in several)
    SeqDesc sd = p.seqs.d[0];
    for (int s = 1; s < p.seqs.n; ++s)
        if (gbj >= (int)((long long)p.seqs.d[s].blk0 * p.b / p.bk)) sd = p.seqs.d[s];
    const int L = sd.len, subs = p.b == 128 ? 2 : 1;
    const int j = gbj - (int)((long long)sd.blk0 * p.b / p.bk);
    int imin, imax;
    if constexpr (ARB) { imin = 0; imax = sd.nblk - 1; }
    else mask_irange(p.mask, p.window, j, p.b, p.bk, L, imin, imax);
    if (!live) imax = imin - 1;
    auto defined = [&](int i) -> bool {             // does query block i see key block j at all?
        if constexpr (ARB) return (p.cany[(long long)(sd.blk0 + i) * p.cw + (gbj >> 5)] >> (gbj & 31)) & 1u;
        return true;
    };
    const int nk = L - j * p.bk < p.bk ? L - j * p.bk : p.bk;     // real keys of the block
    const long long tiles = (long long)(p.qb1 - p.qb0) * subs;
    auto mean_of = [&](int i) -> float {            // over the real token pairs of span (i, j)
        const float *src = p.sums + ((long long)h * tiles + (long long)(sd.blk0 + i - p.qb0) * subs) * p.NBk + gbj;
        float v = src[0];
        if (subs == 2) v += src[p.NBk];
        const int nq = L - i * p.b < p.b ? L - i * p.b : p.b;
        return v / (float)(nq * nk);
    };
    // this chunk's part of the column
    const int i_lo = imin > p.qb0 - sd.blk0 ? imin : p.qb0 - sd.blk0;
    const int i_hi = imax < p.qb1 - 1 - sd.blk0 ? imax : p.qb1 - 1 - sd.blk0;
    const long long o = (long long)h * p.NBk + gbj, HN = (long long)p.H * p.NBk;
    double cn = 0.0, x0 = 0.0, s1 = 0.0, s2 = 0.0, s3 = 0.0, s4 = 0.0;
    if (live && p.state && p.qb0 > 0) {
        cn = p.state[o]; x0 = p.state[HN + o];
        if (wave == 0) { s1 = p.state[2 * HN + o]; s2 = p.state[3 * HN + o]; s3 = p.state[4 * HN + o]; s4 = p.state[5 * HN + o]; }
    }
    // power sums shifted by the column's first value (the diagonal block), so that the central moments
    // formed from them at the end lose nothing that matters
    if (cn == 0.0) {
        int i = i_lo;
        while (i <= i_hi && !defined(i)) ++i;
        if (i <= i_hi) x0 = (double)mean_of(i);
    }
    double n_here = 0.0;
    float *bm = p.block_mean ? p.block_mean + ((long long)h * p.NB + sd.blk0) * p.NBk + gbj : nullptr;
#pragma unroll 4
    for (int i = i_lo + wave; i <= i_hi; i += 4) {
        if (!defined(i)) continue;
        const float mval = mean_of(i);
        if (bm) bm[(long long)i * p.NBk] = mval;
        const double y = (double)mval - x0, y2 = y * y;
        s1 += y;
        s2 += y2;
        s3 = fma(y2, y, s3);
        s4 = fma(y2, y2, s4);
        n_here += 1.0;
    }
    s_part[wave][0][lane] = s1; s_part[wave][1][lane] = s2; s_part[wave][2][lane] = s3; s_part[wave][3][lane] = s4;
    s_part[wave][4][lane] = n_here;
    __syncthreads();
    if (wave != 0 || !live) return;
    for (int w = 1; w < 4; ++w) {
        s1 += s_part[w][0][lane]; s2 += s_part[w][1][lane]; s3 += s_part[w][2][lane]; s4 += s_part[w][3][lane];
        n_here += s_part[w][4][lane];
    }
    cn += n_here;
    if (p.qb1 < p.NB) {                              // more chunks to come
        p.state[o] = cn; p.state[HN + o] = x0;
        p.state[2 * HN + o] = s1; p.state[3 * HN + o] = s2; p.state[4 * HN + o] = s3; p.state[5 * HN + o] = s4;
        return;
    }
    if constexpr (ARB) p.col_n[o] = (int)cn;
    if (cn == 0.0) {                                 // a key block of padding only (or hidden from everyone): no column
        p.col_mean[o] = 0.f; p.col_kurt[o] = 0.f;
        return;
    }
    const double mu = s1 / cn;                       // mean of the shifted values
    const double m2 = s2 / cn - mu * mu;
    const double m4 = s4 / cn - 4.0 * mu * (s3 / cn) + 6.0 * mu * mu * (s2 / cn) - 3.0 * mu * mu * mu * mu;
    p.col_mean[o] = (float)(x0 + mu);
    p.col_kurt[o] = (cn >= 4.0 && m2 > 0.0) ? (float)(m4 / (m2 * m2) - 3.0) : 0.f;
}

// ---------------------------------------------------------------------------------------------
// heads: one wavefront per (head, sequence) reduces the column statistics.
// ---------------------------------------------------------------------------------------------
__device__ __forceinline__ double wave_sum_f64(double v)
{
#pragma unroll
    for (int s = 32; s >= 1; s >>= 1) v += __shfl_xor(v, s);
    return v;
}

__global__ void __launch_bounds__(64) stats_heads_kernel(const StatsParams p)
{
    const int lane = threadIdx.x;
    const int h = blockIdx.x / p.seqs.n, s = blockIdx.x % p.seqs.n;
    const SeqDesc sd = p.seqs.d[s];
    const int L = sd.len;
    const int N = (L + p.bk - 1) / p.bk;            // columns: the key blocks that hold a real key
    const long long kblk0 = (long long)sd.blk0 * p.b / p.bk;
    const float *cm = p.col_mean + (long long)h * p.NBk + kblk0;
    const float *ck = p.col_kurt + (long long)h * p.NBk + kblk0;
    const bool arb = p.mask == STREAM_MASK_ARRAY;
    const int *cnn = p.col_n + (long long)h * p.NBk + kblk0;     // (read with an array only)
    double s1 = 0.0;
    float mx = -INFINITY;
    int n_cols = 0;                                 // columns some query block sees
    for (int j = lane; j < N; j += 64) {
        int imin, imax;
        mask_irange(p.mask, p.window, j, p.b, p.bk, L, imin, imax);
        const int n = arb ? cnn[j] : imax - imin + 1;
        if (n > 0) { s1 += (double)cm[j]; ++n_cols; }
        if (n >= 4) mx = fmaxf(mx, ck[j]);
    }
    for (int sft = 32; sft >= 1; sft >>= 1) n_cols += __shfl_xor(n_cols, sft);
    if (!arb) n_cols = N;
    const int Ncol = n_cols;
    const double mean = wave_sum_f64(s1) / (double)(Ncol > 0 ? Ncol : 1);
    double c2 = 0.0, c4 = 0.0;
    for (int j = lane; j < N; j += 64) {
        if (arb && cnn[j] <= 0) continue;
        const double c = (double)cm[j] - mean;
        c2 += c * c;
        c4 += c * c * c * c;
    }
    const double m2 = wave_sum_f64(c2) / (double)(Ncol > 0 ? Ncol : 1), m4 = wave_sum_f64(c4) / (double)(Ncol > 0 ? Ncol : 1);
    mx = wave_max(mx);
    if (lane == 0) {
        float *o = p.head_stats + ((long long)h * p.seqs.n + s) * 2;
        o[0] = mx == -INFINITY ? 0.f : mx;
        o[1] = (Ncol >= 4 && m2 > 0.0) ? (float)(m4 / (m2 * m2) - 3.0) : 0.f;
    }
}

__global__ void __launch_bounds__(256) stats_zero_kernel(float *p, long long n)
{
    const long long stride = (long long)gridDim.x * blockDim.x;
    for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride) p[i] = 0.f;
}

struct StatsWorkspace {
    bool scratch_rows;           // one pass over the scores
    size_t kp, queue, scratch, sums, state, cany, call, coln, total;
    long long scratch_wave;      // floats per wavefront of the row kernel
    int wgs;                     // workgroups of the row kernel
    int chunk;                   // query blocks per chunk
};

// Workgroups of the row kernel that the chip holds: 2 wavefronts per SIMD; 3 with 32 queries each (not with an
// array and rows of more than 128 bytes, which take the registers of the third); 1 with fp32 at d = 128.
// 32 k tokens, 32/8 heads: rows 4.40 ms (1.0 PFLOP/s
// of scores), columns 74 us; two thirds of that time are what the MFMAs alone take at the clock the power
// limit leaves (0.64 us per tile and SIMD, 0.92-0.97 with the exponentials and nothing else, 1.07 here).
static int stats_wgs(const Problem &pb)
{
    if (pb.dtype == STREAM_F32 && pb.d == 128) return 256;
    const bool third = pb.b == 32 && (pb.mask != STREAM_MASK_ARRAY || pb.d * pb.esize <= 128);
    return third ? 768 : 512;
}

// Span sums kept at a time.  (A chunk is one launch of either kernel; 128 MiB are 512 query blocks at 131 k
// tokens and 32 heads, several rounds of the row kernel's grid.)
constexpr size_t kStatsSumsBytes = (size_t)128 << 20;

// Scratch rows are taken up to this size, or up to the size of Q: a wavefront's is as long as a row, whatever the
// number of heads (one head of 131 k tokens 1 GiB, of 1 M tokens 8 GiB).  Beyond, or in a workspace that has
// no room for them, the scores are computed twice (32 k tokens, 32/8 heads: 8.3 ms instead of 4.4).
constexpr size_t kStatsScratchBytes = (size_t)1 << 30;

static StatsWorkspace stats_layout_as(const Problem &pb, bool scratch_rows)
{
    StatsWorkspace w;
    size_t off = 0;
    const size_t NBk = (size_t)pb.NB * pb.b / pb.bk, subs = pb.b == 128 ? 2 : 1;
    const size_t q_bytes = (size_t)pb.H * pb.NB * pb.b * pb.d * pb.esize;
    w.scratch_rows = scratch_rows;
    w.kp = off;   off += align_up((size_t)pb.Hkv * pb.NB * pb.b * pb.d * pb.esize, 256);
    w.queue = off; off += 256;
    // (without the scratch the whole stays below packed copies of Q and K)
    const size_t per_block = (size_t)pb.H * subs * NBk * 4;
    size_t chunk = (scratch_rows || q_bytes > kStatsSumsBytes ? kStatsSumsBytes : q_bytes) / per_block;
    chunk = chunk < 1 ? 1 : (chunk > (size_t)pb.NB ? (size_t)pb.NB : chunk);
    w.chunk = (int)chunk;
    w.sums = off; off += align_up(per_block * chunk, 256);
    w.state = off; off += w.chunk < pb.NB ? align_up((size_t)6 * pb.H * NBk * 8, 256) : 0;
    // a scratch row of 32 or 64 floats per 64 (b_k = 32: per 32) keys that a row may see
    const int qt = pb.b == 32 ? 32 : 64;
    long long keys = 0;
    for (int i = 0; i < pb.seqs.n; ++i) keys = pb.seqs.d[i].len > keys ? pb.seqs.d[i].len : keys;
    long long tiles = (keys + 63) / 64;
    if (pb.mask == STREAM_MASK_SLIDING && ((long long)pb.window + qt + 61) / 64 + 1 < tiles)
        tiles = ((long long)pb.window + qt + 61) / 64 + 1;        // window + qt - 1 keys, from anywhere in a tile on
    w.scratch_wave = tiles * (pb.bk == 32 ? 2 : 1) * qt;
    // a workgroup per four rows of the longest chunk, as many as the chip holds at the most
    const long long row_items = (long long)chunk * (pb.b / qt) * pb.g;
    const int full = (make_wg_map(pb.Hkv, (int)((row_items + 3) / 4)).grid + kXcds - 1) / kXcds * kXcds;
    w.wgs = full < stats_wgs(pb) ? full : stats_wgs(pb);
    const size_t scratch_bytes = align_up((size_t)w.wgs * 4 * w.scratch_wave * 4, 256);
    if (scratch_rows && scratch_bytes > kStatsScratchBytes && scratch_bytes > q_bytes) return stats_layout_as(pb, false);
    w.scratch = off; off += scratch_rows ? scratch_bytes : 0;
    // with a mask array: its block-level summaries and the number of spans of every column
    const bool arb = pb.mask == STREAM_MASK_ARRAY;
    const size_t bm = arb ? align_up((size_t)pb.NB * block_bitmap_words(pb) * 4, 256) : 0;
    w.cany = off; off += bm;
    w.call = off; off += bm;
    w.coln = off; off += arb ? align_up((size_t)pb.H * NBk * 4, 256) : 0;
    w.total = off;
    return w;
}

// The layout to ask for.
static StatsWorkspace stats_layout(const Problem &pb) { return stats_layout_as(pb, true); }

// The layout for a workspace of `bytes` (its total is larger: refused).  Packed copies of Q and K and 4 bytes per
// padded token and head are enough for the one without scratch rows.
static StatsWorkspace stats_layout_in(const Problem &pb, size_t bytes)
{
    const StatsWorkspace w = stats_layout(pb);
    const StatsWorkspace small = stats_layout_as(pb, false);
    const size_t tokens = (size_t)pb.NB * pb.b;
    const size_t copies = align_up(pb.H * tokens * pb.d * pb.esize, 256) + align_up(pb.Hkv * tokens * pb.d * pb.esize, 256) +
                          align_up(pb.H * tokens * 4, 256) + (small.total - small.cany);
    return bytes < w.total && bytes >= copies ? small : w;
}

typedef void (*stats_fn)(const StatsParams);

template <bool BF16, int D, int NS, bool SCRATCH>
static stats_fn pick_stats_rows(bool arb, bool bk32)
{
    constexpr int OCC = (BF16 || D == 64) ? 2 : 1;   // fp32 with d = 128 holds 16 fragments per group
    if (arb) return bk32 ? stats_rows_kernel<BF16, D, NS, OCC, true, true, SCRATCH> : stats_rows_kernel<BF16, D, NS, OCC, true, false, SCRATCH>;
    return bk32 ? stats_rows_kernel<BF16, D, NS, OCC, false, true, SCRATCH> : stats_rows_kernel<BF16, D, NS, OCC, false, false, SCRATCH>;
}

template <bool SCRATCH>
static stats_fn pick_stats_rows_kernel(const Problem &pb)
{
    const bool arb = pb.mask == STREAM_MASK_ARRAY, bk32 = pb.bk == 32, ns1 = pb.b == 32;
    if (pb.dtype == STREAM_BF16) {
        if (pb.d == 128) return ns1 ? pick_stats_rows<true, 128, 1, SCRATCH>(arb, bk32) : pick_stats_rows<true, 128, 2, SCRATCH>(arb, bk32);
        return ns1 ? pick_stats_rows<true, 64, 1, SCRATCH>(arb, bk32) : pick_stats_rows<true, 64, 2, SCRATCH>(arb, bk32);
    }
    if (pb.d == 128) return ns1 ? pick_stats_rows<false, 128, 1, SCRATCH>(arb, bk32) : pick_stats_rows<false, 128, 2, SCRATCH>(arb, bk32);
    return ns1 ? pick_stats_rows<false, 64, 1, SCRATCH>(arb, bk32) : pick_stats_rows<false, 64, 2, SCRATCH>(arb, bk32);
}

}  // namespace stream

using namespace stream;

extern "C" {

size_t stream_receiver_stats_workspace_bytes(const stream_shape *shape)
{
    Problem pb;
    if (make_problem(shape, 0, nullptr, 0, &pb) != STREAM_OK) return 0;
    return stats_layout(pb).total;
}

stream_status stream_receiver_stats(const void *Q, const void *K, const stream_shape *shape, float scale,
                                    float *block_mean, float *col_mean, float *col_kurt,
                                    float *head_stats, void *workspace, size_t workspace_bytes,
                                    void *hip_stream)
{
    if (!Q || !K || !shape || !col_mean || !col_kurt || !head_stats) return STREAM_EINVAL;
    if (!(scale > 0.f) || !isfinite(scale)) return STREAM_EINVAL;
    Problem pb;
    stream_status rc = make_problem(shape, 0, nullptr, 0, &pb);
    if (rc != STREAM_OK) return rc;
    const long long q_sh = shape->q_stride_h ? shape->q_stride_h : pb.T * pb.d;
    const long long q_st = shape->q_stride_t ? shape->q_stride_t : pb.d;
    const long long k_sh = shape->k_stride_h ? shape->k_stride_h : pb.T * pb.d;
    const long long k_st = shape->k_stride_t ? shape->k_stride_t : pb.d;
    if (q_st < pb.d || k_st < pb.d || q_sh < 0 || k_sh < 0) return STREAM_EINVAL;
    if (((uintptr_t)Q | (uintptr_t)K) & 15) return STREAM_EINVAL;
    if ((q_sh * pb.esize | q_st * pb.esize | k_sh * pb.esize | k_st * pb.esize) & 15) return STREAM_EINVAL;
    if (pb.dtype == STREAM_F32 && pb.d == 128 && pb.bk == 128) return STREAM_EUNSUPPORTED;
    const bool arb = pb.mask == STREAM_MASK_ARRAY;
    const StatsWorkspace w = stats_layout_in(pb, workspace_bytes);
    if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < w.total) return STREAM_EWORKSPACE;
    hipStream_t st = (hipStream_t)hip_stream;
    char *ws = (char *)workspace;

    rc = launch_pack(K, k_sh, k_st, ws + w.kp, pb, st);
    if (rc != STREAM_OK) return rc;

    StatsParams p;
    p.Q = (const char *)Q;
    p.q_sh_b = q_sh * pb.esize; p.q_st_b = q_st * pb.esize;
    p.Kp = ws + w.kp;
    p.scratch = w.scratch_rows ? (float *)(ws + w.scratch) : nullptr; p.scratch_wave = w.scratch_wave;
    p.sums = (float *)(ws + w.sums);
    p.queue = (int *)(ws + w.queue);
    p.state = w.chunk < pb.NB ? (double *)(ws + w.state) : nullptr;
    p.block_mean = block_mean;
    p.col_mean = col_mean; p.col_kurt = col_kurt; p.head_stats = head_stats;
    p.c = scale * 1.4426950408889634f;
    p.H = pb.H; p.g = pb.g; p.NB = pb.NB; p.b = pb.b;
    p.bk = pb.bk; p.NBk = (int)((long long)pb.NB * pb.b / pb.bk);
    p.mask = pb.mask; p.window = pb.window;
    p.cbits = pb.cbits; p.cpitch = pb.cpitch;
    p.cany = (const unsigned *)(ws + w.cany);
    p.cw = arb ? block_bitmap_words(pb) : 0;
    p.col_n = (int *)(ws + w.coln);
    p.seqs = pb.seqs;
    if (arb) {
        rc = launch_block_bitmaps(pb, (unsigned *)(ws + w.cany), (unsigned *)(ws + w.call), st);
        if (rc != STREAM_OK) return rc;
    }

    if (block_mean) {
        // entries no kernel writes (blocks the mask hides, pairs of different sequences) are zero
        const long long n = (long long)pb.H * pb.NB * p.NBk;
        const long long wgs = (n + 255) / 256;
        hipLaunchKernelGGL(stats_zero_kernel, dim3((unsigned)(wgs < 8192 ? wgs : 8192)), dim3(256), 0, st,
                           block_mean, n);
        if (hipGetLastError() != hipSuccess) return STREAM_EDEVICE;
    }

    hipLaunchKernelGGL(stats_zero_kernel, dim3(1), dim3(64), 0, st, (float *)p.queue, (long long)kXcds);
    if (hipGetLastError() != hipSuccess) return STREAM_EDEVICE;

    const int qt = pb.b == 32 ? 32 : 64;
    stats_fn rows = w.scratch_rows ? pick_stats_rows_kernel<true>(pb) : pick_stats_rows_kernel<false>(pb);
    for (int qb0 = 0; qb0 < pb.NB; qb0 += w.chunk) {
        p.qb0 = qb0;
        p.qb1 = qb0 + w.chunk < pb.NB ? qb0 + w.chunk : pb.NB;
        const long long row_items = (long long)(p.qb1 - p.qb0) * (pb.b / qt) * pb.g;
        if ((row_items + 3) / 4 * pb.Hkv + 64 > 0x7fffffffLL) return STREAM_EUNSUPPORTED;
        p.map = make_wg_map(pb.Hkv, (int)((row_items + 3) / 4));
        const int full = (p.map.grid + kXcds - 1) / kXcds * kXcds;
        hipLaunchKernelGGL(rows, dim3((unsigned)(full < w.wgs ? full : w.wgs)), dim3(256), 0, st, p);
        if (hipGetLastError() != hipSuccess) return STREAM_EDEVICE;
        const dim3 grid((unsigned)((p.NBk + 63) / 64), (unsigned)pb.H);
        if (arb) hipLaunchKernelGGL(stats_cols_kernel<true>, grid, dim3(256), 0, st, p);
        else hipLaunchKernelGGL(stats_cols_kernel<false>, grid, dim3(256), 0, st, p);
        if (hipGetLastError() != hipSuccess) return STREAM_EDEVICE;
    }
    hipLaunchKernelGGL(stats_heads_kernel, dim3((unsigned)(pb.H * pb.batch)), dim3(64), 0, st, p);
    return hipGetLastError() == hipSuccess ? STREAM_OK : STREAM_EDEVICE;
}

}  // extern "C"
