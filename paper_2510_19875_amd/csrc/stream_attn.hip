// stream_sparse_attn: Eq. (2) of the paper on the retained key blocks, gfx950.
//
// A wavefront owns up to 64 query tokens of one (head, query block) and walks the block's
// retained key blocks: the first 32 keys of the list, then the rest in order from a place of its own on
// and around the end; where rows are few the four wavefronts of a workgroup share a row.  K tiles come from the same
// packed layout the pruning kernels use; V tiles are packed transposed so that a lane's 16
// bytes hold one feature of the 8 (bf16) or 4 (fp32) keys its MFMA contraction slots cover.
//
// Pass 1 computes S^T = K Q^T with 32x32 MFMAs: a lane then owns one query column and 16 key
// rows per accumulator, so the softmax statistics are per lane (plus one exchange between the
// two lane halves) and the probabilities already sit in B-operand order for O^T += V^T P^T.
// Pass 2 (only when the received mass is requested) recomputes S = Q K^T, where a lane owns one
// key column, turns it into probabilities with the final row normalisers and adds the column
// sums to mass[] with atomics.
#include "stream_mfma.h"
#include "stream_pack.h"

#include <math.h>

namespace stream {

// ---------------------------------------------------------------------------------------------
// Preparation, one launch: K and V packed and the received mass cleared, a workgroup per 32-key group of K
// or V or per kZeroPerWg values.  Bound: memory, or the launch itself: 1 k tokens, 12/2 heads 4.3 us (a
// launch each: 3.3 + 3.9 + 1.8, and two launches more for the host), 32 k tokens, 8 kv heads 43 us
// (25 + 24), 131 k tokens 166 us = 6.6 TB/s (82 + 88 + 7).
//
// V: per 32-key group and per 32-feature block db, fragment vf holds for lane
// (mrow = lane % 32, gh = lane / 32) the values V[key][db*32 + mrow] of the keys
//     bf16: element e of fragment vf (2 per group): key = (2*vf + e/4)*8 + gh*4 + e%4
//     fp32: element e of fragment vf (4 per group): key = vf*8 + gh*4 + e
// which are exactly the key rows a lane's S^T accumulator elements cover, in order.
// Layout: [kv_head][global block][group][db][vf][lane] x 16 bytes.
// ---------------------------------------------------------------------------------------------
struct PrepParams {
    const char *K, *V;
    char *Kp, *Vp;
    long long k_sh_b, k_st_b, v_sh_b, v_st_b;
    int d, esize, b, NB;
    unsigned groups;             // 32-key groups of K (and of V)
    unsigned first;              // workgroups of the launches before this one
    float *mass;                 // nullable
    long long mass_n;
    SeqTable seqs;
};

constexpr int kZeroPerWg = 2048;
// (a launch holds fewer than 2^32 threads, 2^24 workgroups: from half of that on the preparation takes several)
constexpr long long kPrepWgsPerLaunch = 1LL << 23;

__global__ void __launch_bounds__(256) attn_prep_kernel(PrepParams p)
{
    const unsigned wg = p.first + blockIdx.x;
    if (wg < p.groups) {
        pack_group(p.K, p.Kp, p.k_sh_b, p.k_st_b, p.d * p.esize, p.b, p.NB, 0, p.seqs, wg);
        return;
    }
    if (wg >= 2u * p.groups) {
        const long long i0 = (long long)(wg - 2u * p.groups) * kZeroPerWg;
        for (long long i = i0 + threadIdx.x; i < i0 + kZeroPerWg && i < p.mass_n; i += 256) p.mass[i] = 0.f;
        return;
    }
    const int groups = p.b / 32;
    const int ndb = p.d / 32;
    const int nvf = p.esize == 2 ? 2 : 4;
    const long long grp = wg - p.groups;
    const int gi = (int)(grp % groups);
    const long long t = grp / groups;
    const int gb = (int)(t % p.NB);
    const int kvh = (int)(t / p.NB);
    const int s = seq_of_block(p.seqs, gb);
    const SeqDesc sd = p.seqs.d[s];
    const int tok0 = (gb - sd.blk0) * p.b + gi * 32;
    char *dst = p.Vp + grp * (32LL * p.d * p.esize);
    const char *src = p.V + kvh * p.v_sh_b;
    for (int c = threadIdx.x; c < ndb * nvf * 64; c += blockDim.x) {
        const int lane = c & 63, vf = (c >> 6) % nvf, db = (c >> 6) / nvf;
        const int mrow = lane & 31, gh = lane >> 5;
        uint4 out = make_uint4(0, 0, 0, 0);
        // (tokens past the end of the sequence read its last one and are cleared afterwards: no branch
        // around a load, all of them in flight together)
        const char *col = src + sd.tok0 * p.v_st_b + (db * 32 + mrow) * p.esize;
        const int last = sd.len - 1;
        if (p.esize == 2) {
            unsigned v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
                const int tok = tok0 + (2 * vf + (e >> 2)) * 8 + gh * 4 + (e & 3);
                v[e] = *reinterpret_cast<const unsigned short *>(col + (tok < last ? tok : last) * p.v_st_b);
            }
#pragma unroll
            for (int e = 0; e < 8; ++e)
                if (tok0 + (2 * vf + (e >> 2)) * 8 + gh * 4 + (e & 3) > last) v[e] = 0u;
            out = make_uint4(v[0] | (v[1] << 16), v[2] | (v[3] << 16), v[4] | (v[5] << 16), v[6] | (v[7] << 16));
        } else {
            unsigned v[4];
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const int tok = tok0 + vf * 8 + gh * 4 + e;
                v[e] = *reinterpret_cast<const unsigned *>(col + (tok < last ? tok : last) * p.v_st_b);
            }
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (tok0 + vf * 8 + gh * 4 + e > last) v[e] = 0u;
            out = make_uint4(v[0], v[1], v[2], v[3]);
        }
        *reinterpret_cast<uint4 *>(dst + (long long)c * 16) = out;
    }
}

struct AttnParams {
    const char *Q;
    const char *Kp, *Vp;
    char *O;
    long long q_sh_b, q_st_b, o_sh_b, o_st_b;
    const int *idx, *cnt;
    float *lse, *mass;           // nullable
    float *lse2;                 // workspace [H, T]: base-2 log-sum-exp, written by pass 1 for pass 2
    long long T;
    int H, g, NB, kmax;
    int b, qsub, ksh;            // b_q; wavefronts (of 32 * NQ queries) per query block; log2(b_k / 32)
    float scale_log2e;           // scale * log2(e): softmax runs in base 2
    int mask, window;            // the mask rule C (stream_mask) and its window
    // STREAM_MASK_ARRAY (ARB kernels): the bit array C, its "wholly visible" block summary
    // [NB, cw] and the words per row of the summary
    const unsigned *cbits, *call;
    long long cpitch;
    int cw;
    unsigned sweep;              // workgroups an XCD starts while a row walks its list (rows of their own): see phase_sweep
    WgMap map;
    WgMap map_own;               // few rows: the mapping with a row per wavefront
    int share_from;              // few rows: entries at which sharing pays, 64 times the mean of a list
    SeqTable seqs;
};
static_assert(sizeof(AttnParams) <= 4096, "kernel arguments are limited to 4 KB");

typedef float floatx8 __attribute__((ext_vector_type(8)));

template <bool BF16>
__device__ __forceinline__ floatx16 mfma16(const uint4 &a, const uint4 &b, floatx16 c)
{
    if constexpr (BF16) {
        return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a),
                                                       __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    } else {
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, a.x), __builtin_bit_cast(float, b.x), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, a.y), __builtin_bit_cast(float, b.y), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, a.z), __builtin_bit_cast(float, b.z), c, 0, 0, 0);
        c = __builtin_amdgcn_mfma_f32_32x32x2f32(__builtin_bit_cast(float, a.w), __builtin_bit_cast(float, b.w), c, 0, 0, 0);
        return c;
    }
}

// Bit pattern of a float taken BY VALUE.  (__builtin_bit_cast applied directly to an element of
// an ext_vector_type lvalue reads element 0 whatever the index, with this compiler.)
__device__ __forceinline__ unsigned f2u(float v) { return __builtin_bit_cast(unsigned, v); }

// Eight probabilities -> one bf16 B-operand fragment (round to nearest even, v_cvt_pk_bf16_f32).
__device__ __forceinline__ uint4 to_bf16_frag(float a, float b, float c, float d, float e, float f,
                                               float g, float h)
{
    floatx8 t = {a, b, c, d, e, f, g, h};
    return __builtin_bit_cast(uint4, __builtin_convertvector(t, bf16x8));
}

__device__ __forceinline__ unsigned pack_bf16x2(float lo, float hi)
{
    typedef float floatx2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    floatx2 t = {lo, hi};
    return __builtin_bit_cast(unsigned, __builtin_convertvector(t, bf16x2));
}

// acc + lo + hi of a packed bf16 pair (v_dot2c_f32_bf16 against (1, 1)).
__device__ __forceinline__ float dot2_ones(unsigned pair, float acc)
{
    typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2_t, pair),
                                           __builtin_bit_cast(bf16x2_t, 0x3f803f80u), acc, false);
}

// One (head, query block, query sub-tile) row of the launch: what both passes derive from the
// workgroup number, the sequence table and the row's list.
// ARB: the mask C is an explicit bit array (STREAM_MASK_ARRAY).  WIDE: lists of more than 64 entries
// (up to kMaxTopkWide) sit in LDS instead of one register.  SHIFT: the walk over the list is shifted (rows in
// phase, see attn_row).  A wavefront has a row of its own, or the four of a workgroup share one, wavefront w
// taking the sub-tiles w, w + 4, ...
template <bool ARB, bool WIDE, bool SHIFT>
struct AttnRow {
    int lane, wave;
    int h, kvh, gb, q, L, qtok0, qt;            // head, kv head, global / local query block, length, first query, queries
    int blk0, nblk;
    long long tok0;
    const int *idx;                             // the row's list in memory
    int kmax, bq;
    int mask, window, ksh;
    int my_blk;                                 // lane j holds list entry j (not WIDE)
    int n_blk;                                  // entries of the list
    int *blk;                                   // this wavefront's list in LDS (WIDE)
    int n_tiles;                                // 32-key sub-tiles of the row's list that can hold a visible key
    int rot;                                    // sub-tiles by which the walk behind the list's first one is shifted (< n_tiles)
    bool plain_list;                            // not what stream_prune writes: every sub-tile is masked token by token
    unsigned long long allmask;                 // ARB: bit j = list entry j is wholly visible to the query block

    // List position of the t-th sub-tile the row visits (past the last one: the last one).
    __device__ __forceinline__ int place(int t) const
    {
        int ts = __builtin_amdgcn_readfirstlane(t);
        ts = ts < n_tiles ? ts : n_tiles - 1;
        if constexpr (!SHIFT) return ts;
        // the head of the list first, then from `rot` on and around the end
        const int tr = ts + rot;
        return ts == 0 ? 0 : (tr < n_tiles ? tr : tr - (n_tiles - 1));
    }
    // A long list sits in LDS: the loops fetch the entry of a sub-tile two sub-tiles ahead of its use, so that
    // the read is not waited for.  (A list in a register is read where it is needed: fetched ahead like this
    // it cost pass 2 2.71 instead of 2.41 ms at 131 k tokens.)
    __device__ __forceinline__ int fetch(int t) const
    {
        if constexpr (WIDE) return blk[place(t) >> ksh];
        else return 0;
    }
    // 32-key group of the sequence that the t-th sub-tile covers, `raw` being its entry (WIDE: fetched before)
    __device__ __forceinline__ int group(int t, int raw) const
    {
        const int ts = place(t);
        const int e = WIDE ? __builtin_amdgcn_readfirstlane(raw) & 0x7fffffff : __builtin_amdgcn_readlane(my_blk, ts >> ksh);
        return (e << ksh) + (ts & ((1 << ksh) - 1));
    }
    // does the mask C (or the end of the sequence) cut through sub-tile t, which starts at key k0?
    __device__ __forceinline__ bool masked(int t, int k0, int raw) const
    {
        if (plain_list) return true;
        if constexpr (ARB && WIDE) return __builtin_amdgcn_readfirstlane(raw) < 0;
        else if constexpr (ARB) return !((allmask >> (place(t) >> ksh)) & 1ull);
        else {
            bool m = k0 + 32 > L;
            if (mask != STREAM_MASK_FULL) m = m | (k0 + 31 > qtok0);                                 // keys after a query
            if (mask == STREAM_MASK_SLIDING) m = m | (k0 <= qtok0 + qt - 1 - window);                // keys before a window
            return m;
        }
    }
};

// Fills in the row and issues the loads of its list; false: nothing to do.  (shared: the same answer in all
// four wavefronts.)
template <bool ARB, bool WIDE, bool SHIFT>
__device__ __forceinline__ bool attn_row(const AttnParams &p, const WgMap &map, bool shared, int qt, int *lds_list, AttnRow<ARB, WIDE, SHIFT> &r)
{
    r.lane = threadIdx.x & 63;
    r.wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);   // wave-uniform: keep it scalar
    // The arguments a wavefront needs before its first tile, fetched together: left to itself the
    // compiler loads each where it is first used and waits for it there - a dozen round trips to
    // the scalar cache one after the other, at the start of every row.  (The empty asm makes them
    // live here.)
    WgMap a_map = map;
    int a_NB = p.NB, a_g = p.g, a_kmax = p.kmax, a_nseq = p.seqs.n, a_b = p.b, a_qsub = p.qsub;
    r.mask = p.mask; r.window = p.window; r.ksh = p.ksh;
    unsigned long long u_idx = (unsigned long long)p.idx, u_cnt = (unsigned long long)p.cnt;
    asm volatile("" : "+s"(a_map.mode), "+s"(a_map.per_kv), "+s"(a_map.kv_heads), "+s"(a_NB), "+s"(a_g),
                      "+s"(a_kmax), "+s"(a_nseq), "+s"(a_b), "+s"(a_qsub), "+s"(u_idx), "+s"(u_cnt),
                      "+s"(r.mask), "+s"(r.window), "+s"(r.ksh));
    // (the two pointers that are dereferenced come back as pointers to global memory: through
    // the asm the compiler no longer knows where they point and would use flat loads, whose
    // completion it can only wait for together with every other load in flight)
    typedef const int __attribute__((address_space(1))) *global_int_ptr;
    const int *a_idx = (const int *)(global_int_ptr)u_idx, *a_cnt = (const int *)(global_int_ptr)u_cnt;
    int slot;
    if (!wg_decode(a_map, blockIdx.x, r.kvh, slot)) return false;
    const long long items_per_kv = (long long)a_NB * a_g * a_qsub;
    const long long it = shared ? (long long)slot : (long long)slot * 4 + r.wave;
    if (it >= items_per_kv) return false;
    int qs, rk_blk, rk_head;
    if (items_per_kv <= 0x7fffffffLL) {           // (a 64-bit division is ~100 instructions)
        const unsigned rk = a_qsub == 2 ? (unsigned)it >> 1 : (unsigned)it;
        qs = a_qsub == 2 ? (int)((unsigned)it & 1u) : 0;
        rk_blk = (int)(rk / (unsigned)a_g);
        rk_head = (int)(rk - (unsigned)rk_blk * (unsigned)a_g);
    } else {
        const long long rk = it / a_qsub;
        qs = (int)(it % a_qsub);
        rk_blk = (int)(rk / a_g);
        rk_head = (int)(rk % a_g);
    }
    const int gb = a_NB - 1 - rk_blk;             // long rows first
    r.gb = gb;
    r.h = r.kvh * a_g + rk_head;
    int sq = 0;
    while (sq + 1 < a_nseq && gb >= p.seqs.d[sq + 1].blk0) ++sq;
    const SeqDesc sd = p.seqs.d[sq];
    r.blk0 = sd.blk0; r.nblk = sd.nblk; r.tok0 = sd.tok0; r.L = sd.len;
    r.q = gb - sd.blk0;
    r.qt = qt;
    r.qtok0 = r.q * a_b + qs * qt;                // first query token (sequence-local) of this row
    if (r.qtok0 >= r.L) return false;
    const long long row = (long long)r.h * a_NB + gb;
    r.idx = a_idx + row * a_kmax;
    r.kmax = a_kmax; r.bq = a_b;
    // (the list is fetched for every slot of the row, whatever its count, so that the load does
    // not wait for the count)
    r.my_blk = !WIDE && r.lane < a_kmax ? r.idx[r.lane] : 0;
    r.n_blk = a_cnt[row];
    r.blk = lds_list;
    return true;
}

// Second half, after the kernel has issued its loads of Q: this waits for the list.  (In one piece the wait
// came ahead of the loads of Q: pass 1 378 instead of 369 us at 10 k tokens and k = 256, pass 2 2.39 instead of
// 2.37 ms at 131 k.)
template <bool ARB, bool WIDE, bool SHIFT>
__device__ __forceinline__ void attn_list(const AttnParams &p, AttnRow<ARB, WIDE, SHIFT> &r)
{
    __builtin_amdgcn_sched_barrier(0);
    const int a_kmax = r.kmax, a_b = r.bq, qt = r.qt, gb = r.gb, nblk = r.nblk;
    const int *my_idx = r.idx;
    int *lds_list = r.blk;
    const int n_blk = r.n_blk < 0 ? 0 : (r.n_blk > a_kmax ? a_kmax : r.n_blk);   // never read past the row's list
    if (r.lane >= n_blk) r.my_blk = 0;
    // ARB: "every pair of this query block and that key block is real and set in C", per key block
    const unsigned *allrow = ARB ? p.call + (long long)gb * p.cw : nullptr;
    auto all_bit = [&](int e) -> bool {           // (an entry outside the block range reads as "cut")
        return (unsigned)e < (unsigned)p.cw * 32u && ((allrow[e >> 5] >> (e & 31)) & 1u);
    };
    // The loops assume what stream_prune writes: strictly ascending ids of key blocks of the
    // sequence.  A list that is anything else (not ascending, a repeated id, an id outside the
    // sequence) is still handled safely: `plain_list` sends every sub-tile through the
    // token-level mask (so no key after a query, and no key outside the sequence, ever
    // counts), and the trimming of the last block is skipped.
    const int bk = 32 << r.ksh, ksub = 1 << r.ksh;
    const int nkb = (int)((long long)nblk * a_b / bk);            // key blocks of the sequence
    bool entry_bad = false;
    if constexpr (WIDE) {
        for (int i = r.lane; i < n_blk; i += 64) {
            int v = my_idx[i];
            const int before = i > 0 ? my_idx[i - 1] : -1;
            entry_bad = entry_bad | ((unsigned)v >= (unsigned)nkb) | (v <= before);
            // (with a mask array the top bit of an entry says that C cuts through the block)
            if constexpr (ARB) v |= all_bit(v) ? 0 : (int)0x80000000;
            lds_list[i] = v;
        }
        wave_sync();
    } else {
        const int before = __shfl_up(r.my_blk, 1);
        entry_bad = (r.lane < n_blk) & (((unsigned)r.my_blk >= (unsigned)nkb) | ((r.lane > 0) & (r.my_blk <= before)));
    }
    r.plain_list = __ballot(entry_bad) != 0ull;                   // wave-uniform
    // key sub-tiles to visit: all of every listed block, except that under a causal rule the
    // sub-tiles of the diagonal block lying entirely after this row's queries are dropped
    // (lists are ascending, so the diagonal block, if present, is the last one)
    int n_tiles = n_blk << r.ksh;
    if (!ARB && !r.plain_list && n_blk > 0 && r.mask != STREAM_MASK_FULL) {
        const int last_r = WIDE ? my_idx[n_blk - 1] : __builtin_amdgcn_readlane(r.my_blk, n_blk - 1);
        if (last_r * bk + (ksub - 1) * 32 > r.qtok0 + qt - 1) {
            int vis = ((r.qtok0 + qt - 1 - last_r * bk) >> 5) + 1;
            vis = vis < 0 ? 0 : (vis > ksub ? ksub : vis);
            n_tiles = ((n_blk - 1) << r.ksh) + vis;
        }
    }
    r.n_tiles = __builtin_amdgcn_readfirstlane(n_tiles);
    // An XCD works on the keys of one kv head at a time, far more than its L2 holds, and what a row
    // finds there is what other rows in flight have just read.  Rows start one after the other, so if each
    // began at the head of its list they would be spread over the whole key axis at any moment.
    // Instead workgroup i of the R that an XCD starts while a row lasts goes, after the first sub-tile, to
    // i/R of the way through its list and wraps around: a full sweep takes as long as R workgroups take to be
    // started, so all rows in flight pass the same keys at the same time (phase_sweep says what R is and what
    // it measured).  The first sub-tile of the list stays the first one visited: it usually holds the heaviest key (the sink), whose probability is then 1 before it is rounded to
    // bf16.  (From i/R on without it: error of O against 64 bits 1.85e-3 instead of 1.81e-3 at 10 k tokens, of the
    // mass 4.1e-7 instead of 3.1e-7; time the same.)  The order of the sums depends on the row's place in
    // the launch: O and lse repeat from call to call, not from one number of heads or packing to another.
    // The mass is added up with atomics, in no fixed order.
    r.rot = 0;
    if constexpr (SHIFT) {
        const unsigned phase = (blockIdx.x / kXcds) % p.sweep;
        const int rot = (int)(((unsigned)n_blk * phase / p.sweep) << r.ksh);
        r.rot = __builtin_amdgcn_readfirstlane(rot < n_tiles ? rot : (n_tiles > 0 ? n_tiles - 1 : 0));
    }
    // ARB: one lane per entry looks its block up once, the loops then test a scalar bit per sub-tile
    r.allmask = 0;
    if constexpr (ARB && !WIDE) r.allmask = __ballot(r.lane < n_blk && all_bit(r.my_blk));
}

// ---------------------------------------------------------------------------------------------
// Pass 1: O and the log-sum-exps.  NQ: 32-query groups per wavefront.
//
// Per 32-key sub-tile: S^T = K Q^T, softmax, O^T += V^T P^T.  What a wavefront does alone (the
// matrix products, then ~160 vector instructions, then the products again) and what surrounds a
// row (its decode, Q, the list, the normalisation and the stores: as long as 20-30 sub-tiles' matrix
// work) only overlaps with another wavefront's work, so the tile has to leave room for two
// wavefronts on a SIMD, 256 registers each: 128 hold O, 32 the K and V fragments on their way, 32 the
// scores; the Q fragments are read from LDS for every sub-tile (a lane reads back the 16 bytes it
// wrote itself, so no barrier is involved; 16 KB per sub-tile is half of what LDS delivers in the
// matrix time).  K and V fragments take turns in their registers.
//
// The reference exponent of the softmax is set by the first sub-tile in which every query sees a
// key and then kept: probabilities are 2^(s - m_ref), any magnitude fp32 and bf16 represent,
// and the final normalisation makes the choice of reference immaterial.  That saves the maximum,
// the reference update and the accumulator rescale of all other sub-tiles.  It cannot be wrong
// silently: a probability beyond 2^127 shows as a non-finite normaliser / output, and then the row is
// computed again with the maximum tracked in every sub-tile (`safe`).
//
// SPLIT: the four wavefronts share a row, in launches with too few rows to fill the chip; the wavefronts' partial results are merged
// through LDS at the end.
// ---------------------------------------------------------------------------------------------
template <bool BF16, int D, int NQ>
struct FwdLds {
    // staging of the output: 32 query rows of at most 256 bytes at a time (the pad of 16 bytes per row
    // spreads the rows over the banks); partial results of shared rows are staged in fp32
    static constexpr int ndbu(int es) { return D / 32 < 256 / (32 * es) ? D / 32 : 256 / (32 * es); }   // feature blocks per staged unit
    static constexpr int row(int es) { return ndbu(es) * 32 * es; }
    static constexpr int ES = BF16 ? 2 : 4;
    static constexpr int Q = NQ == 1 ? 0 : NQ * D * ES / 32 * 1024;
    static constexpr int bytes(bool few) { int o = 32 * (row(few ? 4 : ES) + 16); return Q > o ? Q : o; }   // per wavefront
};

template <bool BF16, int D, int NQ, bool ARB, bool WIDE, bool SPLIT, bool SHIFT>
__device__ __forceinline__ void attn_fwd_rows(const AttnParams &p, const WgMap &map, char *s_q, int wave_lds,
                                              int (*s_blk)[WIDE ? kMaxTopkWide : 1], float (*s_ml)[3][SPLIT ? 32 * NQ : 1])
{
    constexpr int ES = BF16 ? 2 : 4;
    constexpr int FR = D * ES / 32;            // K/Q fragments per 32-token group
    constexpr int NDB = D / 32;                // 32-feature blocks of the output
    constexpr int NVF = BF16 ? 2 : 4;          // V fragments per (group, feature block)
    constexpr int QT = 32 * NQ;                // queries per wavefront
    constexpr int GROUP_BYTES = 32 * D * ES;
    constexpr int TS = SPLIT ? 4 : 1;
    // 32-query rows: half the output accumulators, room for Q and for V fragments of their own (10 k
    // tokens, 12/2 heads, k = 64 / 256: 160 / 421 us with shared registers and Q in LDS, 158 / 409 us so)
    constexpr bool QREG = NQ == 1, OWNV = NQ == 1;
    constexpr int OES = SPLIT ? 4 : ES;
    constexpr int O_NDBU = FwdLds<BF16, D, NQ>::ndbu(OES), O_URB = FwdLds<BF16, D, NQ>::row(OES), O_URS = O_URB + 16;

    AttnRow<ARB, WIDE, SHIFT> r;
    const int wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (!attn_row(p, map, SPLIT, QT, s_blk[WIDE ? wave_id : 0], r)) return;
    const int lane = r.lane, wave = r.wave;
    const int col = lane & 31, gh = lane >> 5;
    const int L = r.L, qtok0 = r.qtok0;
    char *my_lds = s_q + wave * wave_lds;
    const unsigned lane_off = lane * 16;

    // packed K and V of this (kv head, sequence)
    const long long qblk_bytes = (long long)p.b * D * ES;
    const unsigned region_bytes = (unsigned)((long long)r.nblk * qblk_bytes);
    const __amdgpu_buffer_rsrc_t krs =
        make_tile_rsrc(p.Kp + ((long long)r.kvh * p.NB + r.blk0) * qblk_bytes, region_bytes);
    const __amdgpu_buffer_rsrc_t vrs =
        make_tile_rsrc(p.Vp + ((long long)r.kvh * p.NB + r.blk0) * qblk_bytes, region_bytes);

    // Q fragments (B operand): lane (col, gh), fragment fr -> chunk 2*fr+gh of row col, to LDS
    // (through a resource that starts at the row's first query and spans its real queries: rows past
    // the end of the sequence read as zeros, no branch around any load)
    uint4 qreg[QREG ? NQ : 1][QREG ? FR : 1];
    {
        const long long q_st = p.q_st_b;
        const int qrows = L - qtok0 < QT ? L - qtok0 : QT;
        const __amdgpu_buffer_rsrc_t qrs = make_tile_rsrc(
            p.Q + (long long)r.h * p.q_sh_b + (r.tok0 + qtok0) * q_st, (unsigned)((long long)(qrows - 1) * q_st + D * ES));
        u32x4_t v[NQ][FR];
#pragma unroll
        for (int cq = 0; cq < NQ; ++cq) {
            const unsigned voff = (unsigned)(cq * 32 + col) * (unsigned)q_st + gh * 16;
#pragma unroll
            for (int fr = 0; fr < FR; ++fr) v[cq][fr] = __builtin_amdgcn_raw_buffer_load_b128(qrs, voff + fr * 32, 0, 0);
        }
        attn_list(p, r);
#pragma unroll
        for (int cq = 0; cq < NQ; ++cq)
#pragma unroll
            for (int fr = 0; fr < FR; ++fr) {
                if constexpr (QREG) qreg[cq][fr] = make_uint4(v[cq][fr][0], v[cq][fr][1], v[cq][fr][2], v[cq][fr][3]);
                else *reinterpret_cast<u32x4_t *>(my_lds + (fr * NQ + cq) * 1024 + lane_off) = v[cq][fr];
            }
    }
    auto q_frag = [&](int fr, int cq) -> uint4 {
        if constexpr (QREG) return qreg[cq][fr];
        else return *reinterpret_cast<const uint4 *>(my_lds + (fr * NQ + cq) * 1024 + lane_off);
    };

    const float c2 = p.scale_log2e;
    const int n_tiles = r.n_tiles, t0 = SPLIT ? wave : 0;
    floatx16 acc_o[NDB][NQ];
    float m_run[NQ], l_run[NQ];
    // bf16: the PV product uses the probabilities rounded to bf16, so O is normalised by the sum
    // of those same rounded values (lr_run): a row dominated by one key then gets that key's V
    // exactly, whatever the rounding of its probability.  lse uses the unrounded sum (l_run).
    float lr_run[NQ];
    float l_tot[NQ], lr_tot[NQ];
    bool safe = false;
    for (;;) {
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int cq = 0; cq < NQ; ++cq)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc_o[db][cq][i] = 0.f;
#pragma unroll
        for (int cq = 0; cq < NQ; ++cq) { m_run[cq] = -INFINITY; l_run[cq] = 0.f; lr_run[cq] = 0.f; }
        // The K and the V fragments of a sub-tile (there are as many) take turns in one set of registers:
        // a fragment's registers are refilled right after its last use, K's with V of the same
        // sub-tile, V's with K of the next.  (With a set of their own each the 64-query tile spills;
        // half shared and half not measured 2-4 % slower than this.)
        uint4 kv[FR], vreg[OWNV ? FR : 1];
        static_assert(FR == NDB * NVF, "as many fragments of V as of K");
        if (t0 < n_tiles) {
            // same order as the refills inside the loop: waits count loads in issue order
            const unsigned off0 = (unsigned)r.group(t0, r.fetch(t0)) * (unsigned)GROUP_BYTES;
#pragma unroll
            for (int fr = 0; fr < FR; ++fr) {
                kv[fr] = load_frag(krs, lane_off, off0, fr);
                __builtin_amdgcn_sched_barrier(0);
            }
            if constexpr (OWNV)
#pragma unroll
                for (int g = 0; g < FR; ++g) {
                    vreg[g] = load_frag(vrs, lane_off, off0, (g % NDB) * NVF + g / NDB);
                    __builtin_amdgcn_sched_barrier(0);
                }
        }
        bool track = true;                      // wave-uniform: some query has no reference yet (or `safe`)
        int raw = 0, raw_next = 0, grp = 0;
        if (t0 < n_tiles) { raw = r.fetch(t0); raw_next = r.fetch(t0 + TS); grp = r.group(t0, raw); }
        for (int t = t0; t < n_tiles; t += TS) {
            const int k0 = grp * 32;
            const unsigned cur = (unsigned)grp * (unsigned)GROUP_BYTES;
            const bool masked = r.masked(t, k0, raw);
            raw = raw_next;
            grp = r.group(t + TS, raw);
            raw_next = r.fetch(t + 2 * TS);
            const unsigned next = (unsigned)grp * (unsigned)GROUP_BYTES;
            // ARB: the word of this lane's queries that holds keys k0 .. k0 + 31 (a word wholly past the
            // end of the row is not read), fetched ahead of the refills so that it is not waited for behind them
            unsigned cwd[NQ];
            if constexpr (ARB) {
#pragma unroll
                for (int cq = 0; cq < NQ; ++cq) {
                    cwd[cq] = ~0u;
                    const int tq = qtok0 + cq * 32 + col;
                    if (masked) cwd[cq] = ((tq < L) & ((unsigned)k0 < (unsigned)L)) ? p.cbits[(long long)tq * p.cpitch + (k0 >> 5)] : 0u;
                }
            }
            floatx16 acc_s[NQ];
#pragma unroll
            for (int cq = 0; cq < NQ; ++cq)
#pragma unroll
                for (int i = 0; i < 16; ++i) acc_s[cq][i] = 0.f;
            constexpr int QP = 1;               // Q fragments are read this many steps ahead
            uint4 qb[FR][NQ];
#pragma unroll
            for (int fr = 0; fr < QP && fr < FR; ++fr)
#pragma unroll
                for (int cq = 0; cq < NQ; ++cq) qb[fr][cq] = q_frag(fr, cq);
#pragma unroll
            for (int fr = 0; fr < FR; ++fr) {
                if (fr + QP < FR)
#pragma unroll
                    for (int cq = 0; cq < NQ; ++cq) qb[fr + QP < FR ? fr + QP : fr][cq] = q_frag(fr + QP, cq);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int cq = 0; cq < NQ; ++cq) acc_s[cq] = mfma16<BF16>(kv[fr], qb[fr][cq], acc_s[cq]);
                __builtin_amdgcn_sched_barrier(0);
                kv[fr] = OWNV ? load_frag(krs, lane_off, next, fr) : load_frag(vrs, lane_off, cur, (fr % NDB) * NVF + fr / NDB);
                __builtin_amdgcn_sched_barrier(0);
            }
            if (masked) {                       // the rule C inside the sub-tile, padded keys
#pragma unroll
                for (int cq = 0; cq < NQ; ++cq)
#pragma unroll
                    for (int i = 0; i < 16; ++i) {
                        const int kr = (i >> 2) * 8 + gh * 4 + (i & 3);
                        bool visible = (unsigned)(k0 + kr) < (unsigned)L;
                        if constexpr (ARB) visible = visible & ((cwd[cq] >> kr) & 1u);
                        else visible = visible & mask_token(r.mask, r.window, qtok0 + cq * 32 + col, k0 + kr);
                        // (a select, not a conditional store: `if (!visible) acc[..][i] = -inf` on a
                        // vector element was dropped by this compiler inside a lambda)
                        acc_s[cq][i] = visible ? acc_s[cq][i] : -INFINITY;
                    }
            }
            if (track) {
                float alpha[NQ];
                bool grew = false, unset = false;
#pragma unroll
                for (int cq = 0; cq < NQ; ++cq) {
                    float mx = -INFINITY;
#pragma unroll
                    for (int i = 0; i < 16; ++i) mx = fmaxf(mx, acc_s[cq][i]);
                    mx = fmaxf(mx, __shfl_xor(mx, 32)) * c2;
                    // the reference follows the running maximum lazily: it moves only when the
                    // maximum has grown by more than 2^8
                    const float m_new = mx > m_run[cq] + 8.f ? mx : m_run[cq];
                    grew = grew || (m_new > m_run[cq] && m_run[cq] != -INFINITY);
                    unset = unset || m_new == -INFINITY;
                    alpha[cq] = __builtin_amdgcn_exp2f(m_run[cq] - (m_new == -INFINITY ? 0.f : m_new));
                    m_run[cq] = m_new;
                }
                if (__any(grew)) {
#pragma unroll
                    for (int cq = 0; cq < NQ; ++cq) {
                        l_run[cq] *= alpha[cq];
                        lr_run[cq] *= alpha[cq];
#pragma unroll
                        for (int db = 0; db < NDB; ++db)
#pragma unroll
                            for (int i = 0; i < 16; ++i) acc_o[db][cq][i] *= alpha[cq];
                    }
                }
                track = safe || __any(unset);
            }
            // probabilities in base 2: p = 2^(raw * c2 - m); O^T += V^T P^T
            uint4 pf[NVF][NQ];
#pragma unroll
            for (int cq = 0; cq < NQ; ++cq) {
                const float m_use = m_run[cq] == -INFINITY ? 0.f : m_run[cq];
                float sum = 0.f;
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const float pr = __builtin_amdgcn_exp2f(fmaf(acc_s[cq][i], c2, -m_use));
                    acc_s[cq][i] = pr;
                    sum += pr;
                }
                l_run[cq] += sum;                 // per-lane partial; the lane halves are added at the end
#pragma unroll
                for (int vf = 0; vf < NVF; ++vf) {
                    if constexpr (BF16) {
                        const int o = vf * 8;
                        pf[vf][cq] = to_bf16_frag(acc_s[cq][o + 0], acc_s[cq][o + 1], acc_s[cq][o + 2], acc_s[cq][o + 3],
                                                  acc_s[cq][o + 4], acc_s[cq][o + 5], acc_s[cq][o + 6], acc_s[cq][o + 7]);
                        lr_run[cq] = dot2_ones(pf[vf][cq].w, dot2_ones(pf[vf][cq].z, dot2_ones(pf[vf][cq].y, dot2_ones(pf[vf][cq].x, lr_run[cq]))));
                    } else {
                        const int o = vf * 4;
                        pf[vf][cq] = make_uint4(f2u(acc_s[cq][o + 0]), f2u(acc_s[cq][o + 1]), f2u(acc_s[cq][o + 2]), f2u(acc_s[cq][o + 3]));
                    }
                }
            }
#pragma unroll
            for (int vf = 0; vf < NVF; ++vf)
#pragma unroll
                for (int db = 0; db < NDB; ++db) {
                    const int g = vf * NDB + db;
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int cq = 0; cq < NQ; ++cq) acc_o[db][cq] = mfma16<BF16>(OWNV ? vreg[OWNV ? g : 0] : kv[g], pf[vf][cq], acc_o[db][cq]);
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (OWNV) vreg[g] = load_frag(vrs, lane_off, next, db * NVF + vf);
                    else kv[g] = load_frag(krs, lane_off, next, g);
                }
            __builtin_amdgcn_sched_barrier(0);
        }
        // normalisers; in the first attempt also the check that nothing overflowed
        bool bad = false;
#pragma unroll
        for (int cq = 0; cq < NQ; ++cq) {
            l_tot[cq] = l_run[cq] + __shfl_xor(l_run[cq], 32);
            lr_tot[cq] = BF16 ? lr_run[cq] + __shfl_xor(lr_run[cq], 32) : l_tot[cq];
            if (!safe) {
                // (a query that has seen no key has nothing to check)
                const bool any_key = m_run[cq] != -INFINITY;
                bad = bad | (any_key & (!(l_tot[cq] > 1e-30f) | !(l_tot[cq] < 3e38f) | !(lr_tot[cq] > 1e-30f) | !(lr_tot[cq] < 3e38f)));
                // (0 * x summed over the accumulators is NaN as soon as one of them is not finite)
                float chk = 0.f;
#pragma unroll
                for (int db = 0; db < NDB; ++db)
#pragma unroll
                    for (int i = 0; i < 16; ++i) chk = fmaf(acc_o[db][cq][i], 0.f, chk);
                bad = bad | !(chk == 0.f);
            }
        }
        if (safe || !__any(bad)) break;
        safe = true;
    }

    int l_exp[NQ];                                // the sum is l_tot * 2^l_exp (0 unless merged)
#pragma unroll
    for (int cq = 0; cq < NQ; ++cq) l_exp[cq] = 0;
    if constexpr (SPLIT) {
        // the wavefronts' references, sums and outputs: one reference per query, everything scaled to it.
        // A sum may lie anywhere from 1 to 3e38 times 2^reference, so a wavefront's weight is its reference
        // plus the exponent of its sum: the largest of those is what the others are scaled to, and the sums
        // enter with their exponent taken out.  (Scaled by the references alone, a sum of 2^127 whose
        // reference lies 127 octaves below another's would be lost, and sums of 2^127 each would overflow.)
        if (gh == 0) {
#pragma unroll
            for (int cq = 0; cq < NQ; ++cq) {
                s_ml[wave][0][cq * 32 + col] = m_run[cq];
                s_ml[wave][1][cq * 32 + col] = l_tot[cq];
                s_ml[wave][2][cq * 32 + col] = lr_tot[cq];
            }
        }
        __syncthreads();                          // (also: every wavefront is done with its Q fragments)
        float own[NQ];
        int own_exp[NQ];
#pragma unroll
        for (int cq = 0; cq < NQ; ++cq) {
            const int qi = cq * 32 + col;
            float m = -INFINITY, top = -INFINITY;
            int e = 0;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float mw = s_ml[w][0][qi];
                const int ew = __builtin_amdgcn_frexp_expf(s_ml[w][1][qi]);
                const float key = mw + (float)ew;
                if (key > top) { top = key; m = mw; e = ew; }
            }
            const float m_use = m == -INFINITY ? 0.f : m;
            own_exp[cq] = __builtin_amdgcn_frexp_expf(l_tot[cq]);
            own[cq] = __builtin_amdgcn_exp2f((m_run[cq] - m_use) + (float)(own_exp[cq] - e));
            float l = 0.f, lr = 0.f;
#pragma unroll
            for (int w = 0; w < 4; ++w) {
                const float lw = s_ml[w][1][qi];
                const int ew = __builtin_amdgcn_frexp_expf(lw);
                const float f = __builtin_amdgcn_exp2f((s_ml[w][0][qi] - m_use) + (float)(ew - e));
                l += __builtin_amdgcn_ldexpf(lw, -ew) * f;
                lr += __builtin_amdgcn_ldexpf(s_ml[w][2][qi], -ew) * f;
            }
            m_run[cq] = m; l_tot[cq] = l; l_exp[cq] = e;
            own[cq] *= lr > 0.f ? 1.f / lr : 0.f;
        }
        constexpr int LPR = 8, FPL = O_URB / 4 / LPR;          // lanes per row, features per lane
        static_assert(O_URB % (LPR * 16) == 0, "whole 16-byte chunks per lane");
#pragma unroll
        for (int cq = 0; cq < NQ; ++cq)
#pragma unroll
            for (int u = 0; u < NDB / O_NDBU; ++u) {
#pragma unroll
                for (int dbu = 0; dbu < O_NDBU; ++dbu)
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4) {
                        const int db = u * O_NDBU + dbu;
                        float4 v;
                        v.x = __builtin_amdgcn_ldexpf(acc_o[db][cq][i4 * 4 + 0], -own_exp[cq]) * own[cq];
                        v.y = __builtin_amdgcn_ldexpf(acc_o[db][cq][i4 * 4 + 1], -own_exp[cq]) * own[cq];
                        v.z = __builtin_amdgcn_ldexpf(acc_o[db][cq][i4 * 4 + 2], -own_exp[cq]) * own[cq];
                        v.w = __builtin_amdgcn_ldexpf(acc_o[db][cq][i4 * 4 + 3], -own_exp[cq]) * own[cq];
                        *reinterpret_cast<float4 *>(my_lds + col * O_URS + (dbu * 32 + i4 * 8 + gh * 4) * 4) = v;
                    }
                __syncthreads();
                // wavefront w adds up and stores the rows 8w .. 8w + 7
                const int rr = wave * 8 + lane / LPR, tok = qtok0 + cq * 32 + rr;
                float o[FPL];
#pragma unroll
                for (int e = 0; e < FPL; ++e) o[e] = 0.f;
#pragma unroll
                for (int w = 0; w < 4; ++w)
#pragma unroll
                    for (int e4 = 0; e4 < FPL / 4; ++e4) {
                        const float4 v = *reinterpret_cast<const float4 *>(s_q + w * wave_lds + rr * O_URS + ((lane % LPR) * FPL + e4 * 4) * 4);
                        o[e4 * 4 + 0] += v.x; o[e4 * 4 + 1] += v.y; o[e4 * 4 + 2] += v.z; o[e4 * 4 + 3] += v.w;
                    }
                if (tok < L) {
                    char *dst = p.O + (long long)r.h * p.o_sh_b + (r.tok0 + tok) * p.o_st_b +
                                (u * O_NDBU * 32 + (lane % LPR) * FPL) * ES;
#pragma unroll
                    for (int e = 0; e < FPL; e += 16 / ES) {
                        uint4 v;
                        if constexpr (BF16)
                            v = make_uint4(pack_bf16x2(o[e], o[e + 1]), pack_bf16x2(o[e + 2], o[e + 3]),
                                           pack_bf16x2(o[e + 4], o[e + 5]), pack_bf16x2(o[e + 6], o[e + 7]));
                        else
                            v = make_uint4(f2u(o[e]), f2u(o[e + 1]), f2u(o[e + 2]), f2u(o[e + 3]));
                        *reinterpret_cast<uint4 *>(dst + e * ES) = v;
                    }
                }
                __syncthreads();
            }
        if (wave != 0) return;
    } else {
        // O^T accumulator: lane holds query `col`; element i of block db is feature
        // db*32 + 8*(i/4) + 4*gh + (i%4): four consecutive features per group of 4.  Written from
        // here a store instruction would touch 32 rows with 8 or 16 bytes each; the normalised tile
        // goes through LDS instead, 32 rows at a time, and leaves as whole rows (16 bytes per lane).
        constexpr int LPR = O_URB / 16, RPI = 64 / LPR;        // lanes per staged row, rows per store
        float inv[NQ];
#pragma unroll
        for (int cq = 0; cq < NQ; ++cq) inv[cq] = lr_tot[cq] > 0.f ? 1.f / lr_tot[cq] : 0.f;
#pragma unroll
        for (int cq = 0; cq < NQ; ++cq)
#pragma unroll
            for (int u = 0; u < NDB / O_NDBU; ++u) {
#pragma unroll
                for (int dbu = 0; dbu < O_NDBU; ++dbu)
#pragma unroll
                    for (int i4 = 0; i4 < 4; ++i4) {
                        const int db = u * O_NDBU + dbu;
                        const int feat = dbu * 32 + i4 * 8 + gh * 4;      // within the unit
                        const float a = acc_o[db][cq][i4 * 4 + 0] * inv[cq], b = acc_o[db][cq][i4 * 4 + 1] * inv[cq];
                        const float c = acc_o[db][cq][i4 * 4 + 2] * inv[cq], d = acc_o[db][cq][i4 * 4 + 3] * inv[cq];
                        if constexpr (BF16)
                            *reinterpret_cast<uint2 *>(my_lds + col * O_URS + feat * 2) = make_uint2(pack_bf16x2(a, b), pack_bf16x2(c, d));
                        else
                            *reinterpret_cast<float4 *>(my_lds + col * O_URS + feat * 4) = make_float4(a, b, c, d);
                    }
                // (LDS serves a wavefront's instructions in order: the reads below see these writes,
                // and the next unit's writes come after these reads; the barrier only keeps the
                // compiler from moving them across each other)
                __builtin_amdgcn_wave_barrier();
                // (all reads of the unit first, then its stores: one LDS latency per unit, not per store)
                uint4 ov[32 / RPI];
#pragma unroll
                for (int j = 0; j < 32 / RPI; ++j)
                    ov[j] = *reinterpret_cast<const uint4 *>(my_lds + (j * RPI + lane / LPR) * O_URS + (lane % LPR) * 16);
#pragma unroll
                for (int j = 0; j < 32 / RPI; ++j) {
                    const int rr = j * RPI + lane / LPR, ch = lane % LPR;
                    const int tok = qtok0 + cq * 32 + rr;
                    if (tok < L)
                        *reinterpret_cast<uint4 *>(p.O + (long long)r.h * p.o_sh_b + (r.tok0 + tok) * p.o_st_b +
                                                   u * O_URB + ch * 16) = ov[j];
                }
                __builtin_amdgcn_wave_barrier();
            }
    }
#pragma unroll
    for (int cq = 0; cq < NQ; ++cq) {
        const int tok = qtok0 + cq * 32 + col;
        const float lse2 = l_tot[cq] > 0.f ? m_run[cq] + (log2f(l_tot[cq]) + (float)l_exp[cq]) : -INFINITY;
        if (tok < L && gh == 0) {
            if (p.lse) p.lse[(long long)r.h * p.T + r.tok0 + tok] = lse2 * 0.6931471805599453f;
            if (p.lse2) p.lse2[(long long)r.h * p.T + r.tok0 + tok] = lse2;
        }
    }
}

// ---------------------------------------------------------------------------------------------
// Pass 2: received mass.  S = Q K^T: a lane owns key column `col`; element i of row block rq is query
// rq*32 + 8*(i/4) + 4*gh + (i%4).  No output accumulators: Q stays in registers, two wavefronts per
// SIMD so that one's exponentials overlap the other's MFMAs.
// ---------------------------------------------------------------------------------------------
template <bool BF16, int D, int NQ, bool ARB, bool WIDE, bool SHIFT>
__device__ __forceinline__ void attn_mass_rows(const AttnParams &p, const WgMap &map, bool shared, int (*s_blk)[WIDE ? kMaxTopkWide : 1])
{
    constexpr int ES = BF16 ? 2 : 4;
    constexpr int FR = D * ES / 32;
    constexpr int QT = 32 * NQ;
    constexpr int GROUP_BYTES = 32 * D * ES;
    const int TS = shared ? 4 : 1;
    AttnRow<ARB, WIDE, SHIFT> r;
    const int wave_id = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (!attn_row(p, map, shared, QT, s_blk[WIDE ? wave_id : 0], r)) return;
    const int lane = r.lane;
    const int col = lane & 31, gh = lane >> 5;
    const int L = r.L, qtok0 = r.qtok0;
    const unsigned lane_off = lane * 16;
    const int qrows = L - qtok0 < QT ? L - qtok0 : QT;
    // Q fragments (A operand): lane (col, gh), fragment fr -> chunk 2*fr+gh of row col
    uint4 qf[NQ][FR];
    {
        const long long q_st = p.q_st_b;
        const __amdgpu_buffer_rsrc_t qrs = make_tile_rsrc(
            p.Q + (long long)r.h * p.q_sh_b + (r.tok0 + qtok0) * q_st, (unsigned)((long long)(qrows - 1) * q_st + D * ES));
#pragma unroll
        for (int cq = 0; cq < NQ; ++cq) {
            const unsigned voff = (unsigned)(cq * 32 + col) * (unsigned)q_st + gh * 16;
#pragma unroll
            for (int fr = 0; fr < FR; ++fr) {
                const u32x4_t v = __builtin_amdgcn_raw_buffer_load_b128(qrs, voff + fr * 32, 0, 0);
                qf[cq][fr] = make_uint4(v[0], v[1], v[2], v[3]);
            }
        }
    }
    const long long qblk_bytes = (long long)p.b * D * ES;
    const __amdgpu_buffer_rsrc_t krs =
        make_tile_rsrc(p.Kp + ((long long)r.kvh * p.NB + r.blk0) * qblk_bytes, (unsigned)((long long)r.nblk * qblk_bytes));
    const float c2 = p.scale_log2e;
    // normalisers, through a resource over the row's real queries: queries past the end of the sequence
    // read as zeros, and no load sits behind a branch
    float lq[NQ][16];
    {
        const __amdgpu_buffer_rsrc_t lrs =
            make_tile_rsrc(p.lse2 + (long long)r.h * p.T + r.tok0 + qtok0, (unsigned)qrows * 4u);
#pragma unroll
        for (int rq = 0; rq < NQ; ++rq)
#pragma unroll
            for (int i = 0; i < 16; ++i) {
                const unsigned voff = (unsigned)(rq * 32 + (i >> 2) * 8 + gh * 4 + (i & 3)) * 4u;
                lq[rq][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(lrs, voff, 0, 0));
            }
    }
    attn_list(p, r);
    float *mass_h = p.mass + (long long)r.h * p.T + r.tok0;
    const int n_tiles = r.n_tiles, t0 = shared ? r.wave : 0;
    uint4 kreg[FR];
    if (t0 < n_tiles) {
        const unsigned off0 = (unsigned)r.group(t0, r.fetch(t0)) * (unsigned)GROUP_BYTES;
#pragma unroll
        for (int fr = 0; fr < FR; ++fr) {
            kreg[fr] = load_frag(krs, lane_off, off0, fr);
            __builtin_amdgcn_sched_barrier(0);
        }
    }
    int raw = 0, raw_next = 0, grp = 0;
    if (t0 < n_tiles) { raw = r.fetch(t0); raw_next = r.fetch(t0 + TS); grp = r.group(t0, raw); }
    for (int t = t0; t < n_tiles; t += TS) {
        const int k0 = grp * 32;
        const bool masked = r.masked(t, k0, raw);
        raw = raw_next;
        grp = r.group(t + TS, raw);
        raw_next = r.fetch(t + 2 * TS);
        const unsigned next = (unsigned)grp * (unsigned)GROUP_BYTES;
        floatx16 acc_s[NQ];
#pragma unroll
        for (int rq = 0; rq < NQ; ++rq)
#pragma unroll
            for (int i = 0; i < 16; ++i) acc_s[rq][i] = 0.f;
#pragma unroll
        for (int fr = 0; fr < FR; ++fr) {
#pragma unroll
            for (int rq = 0; rq < NQ; ++rq) acc_s[rq] = mfma16<BF16>(qf[rq][fr], kreg[fr], acc_s[rq]);
            __builtin_amdgcn_sched_barrier(0);
            kreg[fr] = load_frag(krs, lane_off, next, fr);
            __builtin_amdgcn_sched_barrier(0);
        }
        const int tk = k0 + col;
        float colsum = 0.f;
        if (!(masked | (qtok0 + QT > L))) {   // wave-uniform: most sub-tiles are fully visible
#pragma unroll
            for (int rq = 0; rq < NQ; ++rq)
#pragma unroll
                for (int i = 0; i < 16; ++i)
                    colsum += __builtin_amdgcn_exp2f(fmaf(acc_s[rq][i], c2, -lq[rq][i]));
        } else {
            // (the empty asm keeps this a real branch: merged into the path above, the mask
            // arithmetic would run on every sub-tile)
            asm volatile("" ::: "memory");
            // ARB: lane j fetches the mask word of query row j for this 32-key group; an
            // element takes its row's word from the lane that fetched it
            unsigned rowword = 0u;
            if constexpr (ARB) {
                const int tqr = qtok0 + lane;
                if (lane < QT && tqr < L && (unsigned)k0 < (unsigned)L)     // (no read of a word wholly past the end of the row)
                    rowword = p.cbits[(long long)tqr * p.cpitch + (k0 >> 5)];
            }
#pragma unroll
            for (int rq = 0; rq < NQ; ++rq)
#pragma unroll
                for (int i = 0; i < 16; ++i) {
                    const int qi = rq * 32 + (i >> 2) * 8 + gh * 4 + (i & 3), tq = qtok0 + qi;
                    const float e = __builtin_amdgcn_exp2f(fmaf(acc_s[rq][i], c2, -lq[rq][i]));
                    bool visible = tq < L;
                    if constexpr (ARB) {
                        const unsigned cwd = (unsigned)__shfl((int)rowword, qi);
                        visible = visible & ((cwd >> col) & 1u);
                    } else {
                        visible = visible & mask_token(r.mask, r.window, tq, tk);
                    }
                    colsum += visible ? e : 0.f;
                }
        }
        colsum += __shfl_xor(colsum, 32);
        if (gh == 0 && (unsigned)tk < (unsigned)L && colsum != 0.f) atomicAdd(mass_h + tk, colsum);
    }
}

// Do the lists of a launch pay for sharing the rows?  Every wavefront looks at the same 16 counts, spread over
// the heads and over the length of the sequences, and comes to the same answer.  (The host knows the slots of
// the lists only: a sweep's or a packed batch's may be nearly empty.)
__device__ __forceinline__ bool share_rows(const AttnParams &p)
{
    const int s = threadIdx.x & 15, most = p.kmax;
    const long long h = ((long long)p.H * s) >> 4, q = (2LL * ((s * 7) & 15) + 1) * p.NB >> 5;
    const int c = min(max(p.cnt[h * p.NB + q], 0), most);
    return __builtin_amdgcn_readfirstlane((int)wave_sum((float)c)) >= p.share_from;
}

// Who works on a row: its own wavefront, the four of a workgroup, or as the lists say.
enum AttnMode { kOwnRow = 0, kSharedRow = 1, kByLists = 2 };

template <bool BF16, int D, int NQ, int OCC, bool ARB, bool WIDE, int MODE>
__global__ void __launch_bounds__(256, OCC) attn_fwd_kernel(const AttnParams p)
{
    constexpr int WAVE_LDS = FwdLds<BF16, D, NQ>::bytes(MODE != kOwnRow);     // Q fragments, then the output staging
    __shared__ __align__(16) char s_q[4 * WAVE_LDS];
    __shared__ int s_blk[WIDE ? 4 : 1][WIDE ? kMaxTopkWide : 1];
    if constexpr (MODE == kOwnRow) {
        attn_fwd_rows<BF16, D, NQ, ARB, WIDE, false, true>(p, p.map, s_q, WAVE_LDS, s_blk, nullptr);
    } else {
        __shared__ float s_ml[4][3][32 * NQ];                     // reference, sum, sum of rounded per query
        if (MODE == kSharedRow || share_rows(p))
            attn_fwd_rows<BF16, D, NQ, ARB, WIDE, true, false>(p, p.map, s_q, WAVE_LDS, s_blk, s_ml);
        else if ((int)blockIdx.x < p.map_own.grid)
            attn_fwd_rows<BF16, D, NQ, ARB, WIDE, false, false>(p, p.map_own, s_q, WAVE_LDS, s_blk, nullptr);
    }
}

template <bool BF16, int D, int NQ, int OCC, bool ARB, bool WIDE, int MODE>
__global__ void __launch_bounds__(256, OCC) attn_mass_kernel(const AttnParams p)
{
    __shared__ int s_blk[WIDE ? 4 : 1][WIDE ? kMaxTopkWide : 1];
    if constexpr (MODE == kOwnRow) {
        attn_mass_rows<BF16, D, NQ, ARB, WIDE, NQ == 1>(p, p.map, false, s_blk);        // (64-query rows gain nothing from a shift here)
    } else if constexpr (MODE == kSharedRow) {
        attn_mass_rows<BF16, D, NQ, ARB, WIDE, false>(p, p.map, true, s_blk);
    } else {
        const bool shared = share_rows(p);
        if (!shared && (int)blockIdx.x >= p.map_own.grid) return;
        attn_mass_rows<BF16, D, NQ, ARB, WIDE, false>(p, shared ? p.map : p.map_own, shared, s_blk);
    }
}

typedef void (*attn_fn)(const AttnParams);

// A kernel and the workgroups of it that a CU runs at a time.
struct AttnKernel {
    attn_fn fn;
    int (*per_cu)();
};

// What the kernel's registers and LDS leave room for (a workgroup is one wavefront per SIMD): asked of the
// runtime once per kernel, a property of the compiled code.  Pass 1 bf16 with 32-query rows fits two at d = 128
// and four at d = 64, pass 2 up to five, fp32 with d = 128 one.
template <attn_fn FN>
static int attn_per_cu()
{
    static const int n = [] {
        int wgs = 0;
        if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&wgs, FN, 256, 0) != hipSuccess || wgs < 1) {
            (void)hipGetLastError();
            wgs = 2;
        }
        return wgs;
    }();
    return n;
}

// R of the rows in phase (see attn_row).  A launch starts with all its workgroups at once, in phase without any
// shift, and drifts apart, because of the wavefronts of a SIMD one is served first: once the starts are
// spread evenly R is what an XCD has in flight, before that a shift of 1/R puts rows out of phase that were in
// it, and with one wavefront per SIMD they stay in it.  Pass 1, us, without shift / R in flight / this rule:
// two per SIMD, 32/8 heads, 131 k tokens at k = 32 5523 / 4800 / 4800 (2048 workgroups per XCD; requests that
// miss the L2 55 % -> 38 %), 80 k 2841 / 2758 / 2760 (1280), 12/2 heads 60 k at k = 64 1473 / 1585 / 1466 (703),
// blocks of 32, 30 k at k = 256 1516 / 1725 / 1512 (352); four per SIMD (d = 64), 60 k at k = 64 1414 / 1333 / 1333
// (1875), 120 k 5443 / 4337 / 4337 (1407); one per SIMD, 60 k at k = 256 3506 / 6982 / 3321 (703), 131 k, k = 64
// 6824 / 10596 / 6801 (4096).  Where the keys fit the L2 nothing changes.  In pass 2, 131 k tokens:
// 64-query rows 2.37 ms with the shift, 2.34 without, 32-query rows (k = 64) 3.5 and 3.9.  fp32 is walked without a shift: its
// products take eight times as long per byte (d = 64, 60 k at k = 256 10336 / 11201 / 10950, at k = 64 2827 / 2911 /
// 2870; 30 k the same either way).
static unsigned phase_sweep(bool bf16, int per_cu, int grid)
{
    if (!bf16) return 1;
    const unsigned started = (unsigned)(grid + kXcds - 1) / kXcds;        // workgroups of an XCD
    const unsigned in_flight = per_cu > 1 ? 32u * (unsigned)per_cu : 192u;
    const unsigned early = (1u << 17) / (started ? started : 1u);
    return early > in_flight ? early : in_flight;
}

// Long lists of 32-query rows over more keys than the L2 holds a good part of: one workgroup per CU, by way of
// LDS that nobody uses.  Two wavefronts on a SIMD drift apart and with them the rows that should pass the same
// keys together; half as many, in step, read less from beyond the L2.  Pass 1 (bf16, d = 128), us, two / one:
// 12/2 heads, 60 k tokens at k = 256 5022 / 3321, at k = 64 1046 / 994, 40 k at k = 256 2234 / 2067, at k = 64 671 /
// 677, 32/8 heads, 131 k at k = 64 7295 / 6791; the other way round 30 k at k = 256 1540 / 1567, at k = 64 478 / 497,
// 32/8 heads 60 k at k = 32 1549 / 1611, 40 k at k = 16 583 / 641; 64-query rows 1466 / 1601 (60 k at k = 64),
// d = 64 1372 / 1455.
constexpr unsigned kOneWgPerCuLds = 48 << 10;             // (with the kernel's own 34 KB: more than half of 160 KB)

static bool one_wg_per_cu(const Problem &pb, int topk_max)
{
    return pb.b == 32 && pb.d == 128 && pb.dtype == STREAM_BF16 && topk_max >= 64 &&
           2LL * pb.T * pb.d * pb.esize / pb.batch >= 20000000;
}

template <attn_fn FN>
static AttnKernel attn_kernel() { return AttnKernel{FN, attn_per_cu<FN>}; }

// Wavefronts own 64 queries of a row (32 for query block 32).  fp32 with d = 128 fits one wavefront per
// SIMD only.
template <bool BF16, int D, int NQ, bool ARB, bool WIDE>
static AttnKernel pick_attn(int pass, AttnMode mode)
{
    constexpr int OCC = BF16 || D == 64 ? 2 : 1;
    if (pass == 1)
        return mode == kOwnRow      ? attn_kernel<attn_fwd_kernel<BF16, D, NQ, OCC, ARB, WIDE, kOwnRow>>()
               : mode == kSharedRow ? attn_kernel<attn_fwd_kernel<BF16, D, NQ, OCC, ARB, WIDE, kSharedRow>>()
                                    : attn_kernel<attn_fwd_kernel<BF16, D, NQ, OCC, ARB, WIDE, kByLists>>();
    return mode == kOwnRow      ? attn_kernel<attn_mass_kernel<BF16, D, NQ, OCC, ARB, WIDE, kOwnRow>>()
           : mode == kSharedRow ? attn_kernel<attn_mass_kernel<BF16, D, NQ, OCC, ARB, WIDE, kSharedRow>>()
                                : attn_kernel<attn_mass_kernel<BF16, D, NQ, OCC, ARB, WIDE, kByLists>>();
}

template <bool BF16, int D, int NQ>
static AttnKernel pick_attn_list(int pass, AttnMode mode, bool arb, bool wide)
{
    if (arb) return wide ? pick_attn<BF16, D, NQ, true, true>(pass, mode) : pick_attn<BF16, D, NQ, true, false>(pass, mode);
    return wide ? pick_attn<BF16, D, NQ, false, true>(pass, mode) : pick_attn<BF16, D, NQ, false, false>(pass, mode);
}

static AttnKernel pick_attn_kernel(const Problem &pb, int pass, AttnMode mode)
{
    const bool arb = pb.mask == STREAM_MASK_ARRAY;
    const bool wide = pb.kmax > kMaxTopk;              // lists longer than one register of entries
    const bool nq1 = pb.b == 32;
    if (pb.dtype == STREAM_BF16) {
        if (pb.d == 128) return nq1 ? pick_attn_list<true, 128, 1>(pass, mode, arb, wide) : pick_attn_list<true, 128, 2>(pass, mode, arb, wide);
        return nq1 ? pick_attn_list<true, 64, 1>(pass, mode, arb, wide) : pick_attn_list<true, 64, 2>(pass, mode, arb, wide);
    }
    if (pb.d == 128) return nq1 ? pick_attn_list<false, 128, 1>(pass, mode, arb, wide) : pick_attn_list<false, 128, 2>(pass, mode, arb, wide);
    return nq1 ? pick_attn_list<false, 64, 1>(pass, mode, arb, wide) : pick_attn_list<false, 64, 2>(pass, mode, arb, wide);
}

// When the four wavefronts of a workgroup share one row: few rows, per sub-tile of a full list, and for
// pass 1 few rows altogether.  A launch of few rows leaves SIMDs idle and lasts as long as its longest row;
// sharing costs every row four decodes and, in pass 1, a merge through LDS, which long lists pay for
// sooner.  Both passes, us, own row / shared row (bf16, d = 128, 12/2 heads unless said): 384 rows x 16
// sub-tiles 39.7 / 26.9, 768 x 32 78.8 / 69.1, 1024 x 32 (32/8 heads) 78.0 / 75.1, 1536 x 64 196 / 173,
// 2256 x 64 166 / 152; the other way round 1536 x 16 54.8 / 55.5, 1024 x 16 (fp32, d = 64) 131 / 135,
// 2048 x 32 122 / 140, 3072 x 16 77 / 92.  At 3756 rows x 64 and 3840 x 256 pass 1 is 158 / 163 and 409 /
// 445, pass 2 101 / 102 and 279 / 264.
// The host knows the slots of the lists; from kShareAlways rows on the kernels go by the lists themselves
// (share_rows; 84 instead of 60, since the mean lies below the slots also where the lists are full: the first
// rows of a sequence).  By the slots alone, 64 of them holding 1 entry, pass 1 took 26.5 us instead of 16.1 for
// 1500 rows and 42.5 instead of 24.2 for 3000; 756 rows of 16 slots 18.8 either way.
constexpr long long kSplitRowsPerTile = 60, kSplitRows = 3000, kShareAlways = 800, kShareRowsPerTile = 84;

struct AttnWorkspace {
    size_t kp, vp, lse2, cany, call, total;
};

static AttnWorkspace attn_layout(const Problem &pb)
{
    AttnWorkspace w;
    const size_t tile = align_up((size_t)pb.Hkv * pb.NB * pb.b * pb.d * pb.esize, 256);
    w.kp = 0;
    w.vp = tile;
    w.lse2 = 2 * tile;
    size_t off = 2 * tile + align_up((size_t)pb.H * pb.T * 4, 256);
    // block-level summaries of an explicit mask array
    const size_t bm = pb.mask == STREAM_MASK_ARRAY ? align_up((size_t)pb.NB * block_bitmap_words(pb) * 4, 256) : 0;
    w.cany = off; off += bm;
    w.call = off; off += bm;
    w.total = off;
    return w;
}

}  // namespace stream

using namespace stream;

extern "C" {

size_t stream_sparse_attn_workspace_bytes(const stream_shape *shape, int topk_max)
{
    Problem pb;
    if (topk_max < 1) return 0;
    if (make_problem(shape, 0, nullptr, 0, &pb) != STREAM_OK) return 0;
    return attn_layout(pb).total;
}

stream_status stream_sparse_attn(const void *Q, const void *K, const void *V,
                                 const stream_shape *shape,
                                 const int *idx, const int *cnt, int topk_max, float scale,
                                 void *O, float *lse, float *mass,
                                 void *workspace, size_t workspace_bytes, void *hip_stream)
{
    if (!Q || !K || !V || !shape || !idx || !cnt || !O) return STREAM_EINVAL;
    if (topk_max < 1 || !(scale > 0.f) || !isfinite(scale)) return STREAM_EINVAL;
    Problem pb;
    stream_status rc = make_problem(shape, 0, nullptr, 0, &pb);
    if (rc != STREAM_OK) return rc;
    pb.kmax = topk_max;
    if (topk_max > kMaxTopkWide) return STREAM_EUNSUPPORTED;
    const long long dflt_h = pb.T * pb.d;
    const long long q_sh = shape->q_stride_h ? shape->q_stride_h : dflt_h;
    const long long q_st = shape->q_stride_t ? shape->q_stride_t : pb.d;
    const long long k_sh = shape->k_stride_h ? shape->k_stride_h : dflt_h;
    const long long k_st = shape->k_stride_t ? shape->k_stride_t : pb.d;
    const long long v_sh = shape->v_stride_h ? shape->v_stride_h : dflt_h;
    const long long v_st = shape->v_stride_t ? shape->v_stride_t : pb.d;
    const long long o_sh = shape->o_stride_h ? shape->o_stride_h : dflt_h;
    const long long o_st = shape->o_stride_t ? shape->o_stride_t : pb.d;
    if (q_st < pb.d || k_st < pb.d || v_st < pb.d || o_st < pb.d) return STREAM_EINVAL;
    if (((uintptr_t)Q | (uintptr_t)K | (uintptr_t)V | (uintptr_t)O) & 15) return STREAM_EINVAL;
    if (((q_sh | q_st | k_sh | k_st | v_sh | v_st | o_sh | o_st) * pb.esize) & 15) return STREAM_EINVAL;
    // the kernels address a wavefront's query rows with 32-bit offsets from its first row
    if (q_st * pb.esize * 128 >= (1LL << 31)) return STREAM_EUNSUPPORTED;
    const AttnWorkspace w = attn_layout(pb);
    if (!workspace || ((uintptr_t)workspace & 255) || workspace_bytes < w.total) return STREAM_EWORKSPACE;
    hipStream_t st = (hipStream_t)hip_stream;
    char *ws = (char *)workspace;

    {
        PrepParams pp;
        pp.K = (const char *)K; pp.V = (const char *)V;
        pp.Kp = ws + w.kp; pp.Vp = ws + w.vp;
        pp.k_sh_b = k_sh * pb.esize; pp.k_st_b = k_st * pb.esize;
        pp.v_sh_b = v_sh * pb.esize; pp.v_st_b = v_st * pb.esize;
        pp.d = pb.d; pp.esize = pb.esize; pp.b = pb.b; pp.NB = pb.NB;
        pp.seqs = pb.seqs;
        pp.mass = mass;
        pp.mass_n = mass ? (long long)pb.H * pb.T : 0;
        const long long groups = (long long)pb.Hkv * pb.NB * (pb.b / 32);
        const long long grid = 2 * groups + (pp.mass_n + kZeroPerWg - 1) / kZeroPerWg;
        if (grid > 0x7fffffffLL) return STREAM_EUNSUPPORTED;
        pp.groups = (unsigned)groups;
        for (long long first = 0; first < grid; first += kPrepWgsPerLaunch) {
            const long long n = grid - first < kPrepWgsPerLaunch ? grid - first : kPrepWgsPerLaunch;
            pp.first = (unsigned)first;
            hipLaunchKernelGGL(attn_prep_kernel, dim3((unsigned)n), dim3(256), 0, st, pp);
            if (hipGetLastError() != hipSuccess) return STREAM_EDEVICE;
        }
    }
    AttnParams p;
    p.Q = (const char *)Q;
    p.Kp = ws + w.kp;
    p.Vp = ws + w.vp;
    p.O = (char *)O;
    p.q_sh_b = q_sh * pb.esize; p.q_st_b = q_st * pb.esize;
    p.o_sh_b = o_sh * pb.esize; p.o_st_b = o_st * pb.esize;
    p.idx = idx; p.cnt = cnt; p.lse = lse; p.mass = mass;
    p.T = pb.T; p.H = pb.H; p.g = pb.g; p.NB = pb.NB; p.kmax = topk_max;
    p.scale_log2e = scale * 1.4426950408889634f;
    p.mask = pb.mask; p.window = pb.window;
    p.cbits = pb.cbits; p.cpitch = pb.cpitch;
    p.call = (const unsigned *)(ws + w.call);
    p.cw = pb.mask == STREAM_MASK_ARRAY ? block_bitmap_words(pb) : 0;
    if (pb.mask == STREAM_MASK_ARRAY) {
        rc = launch_block_bitmaps(pb, (unsigned *)(ws + w.cany), (unsigned *)(ws + w.call), st);
        if (rc != STREAM_OK) return rc;
    }
    p.seqs = pb.seqs;
    p.lse2 = mass ? (float *)(ws + w.lse2) : nullptr;
    p.b = pb.b; p.qsub = pb.b == 128 ? 2 : 1;
    p.ksh = pb.bk == 32 ? 0 : (pb.bk == 64 ? 1 : 2);
    const long long items_per_kv = (long long)pb.NB * pb.g * p.qsub;
    const long long rows = items_per_kv * pb.Hkv;
    for (int pass = 1; pass <= (mass ? 2 : 1); ++pass) {
        const bool split = rows <= kSplitRowsPerTile * ((long long)topk_max << p.ksh) && (pass == 2 || rows <= kSplitRows);
        const long long per_kv = split ? items_per_kv : (items_per_kv + 3) / 4;
        if (per_kv * pb.Hkv + 64 > 0x7fffffffLL) return STREAM_EUNSUPPORTED;
        p.map = make_wg_map(pb.Hkv, (int)per_kv);
        p.map_own = make_wg_map(pb.Hkv, (int)((items_per_kv + 3) / 4));
        p.share_from = (int)((rows * 64 + (kShareRowsPerTile << p.ksh) - 1) / (kShareRowsPerTile << p.ksh));
        const AttnKernel k = pick_attn_kernel(pb, pass, split ? (rows <= kShareAlways ? kSharedRow : kByLists) : kOwnRow);
        const bool one = pass == 1 && !split && one_wg_per_cu(pb, topk_max);
        p.sweep = split ? 1u : phase_sweep(pb.dtype == STREAM_BF16, one ? 1 : k.per_cu(), p.map.grid);
        hipLaunchKernelGGL(k.fn, dim3((unsigned)p.map.grid), dim3(256), one ? kOneWgPerCuLds : 0u, st, p);
        if (hipGetLastError() != hipSuccess) return STREAM_EDEVICE;
    }
    return STREAM_OK;
}

}  // extern "C"
