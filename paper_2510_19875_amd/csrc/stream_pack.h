// Device side of the tile packing, shared by the packing kernel and the attention's preparation kernel.
#pragma once

#include "stream_common.h"

namespace stream {

// ---------------------------------------------------------------------------------------------
// Tile packing.
//
// A 32x32 MFMA reads, per lane, 16 contiguous bytes of one operand row: lane (n = lane % 32,
// g = lane / 32) supplies row n, and the g-th half of the fragment's slice of the contraction
// axis.  Reading those 16 bytes straight from a row-major [token, d] tensor makes every lane of
// a load instruction touch a different row.  The packer therefore rewrites each group of 32
// tokens so that the 64 lanes' chunks of fragment `fr` are contiguous (1 KiB per fragment):
//
//     dst chunk (fr * 64 + g * 32 + n)  <-  src row n, 16-byte chunk (2 * fr + g)
//
// A block of b tokens is b/32 consecutive groups; tokens past the end of a sequence are zero
// (they are masked out wherever they could matter).  Layout: [kv_head][global block][b * d].
// The permutation is per 32-token group, so the same packed tensor serves every block size.
// With kPackFrag16 (operands of the 16x16x32 bf16 MFMA: lane (g = lane / 16, n = lane % 16) supplies
// row n and the g-th 16-byte chunk of the fragment's 64-byte slice) the group is cut into
// fragments of 16 rows x 64 bytes instead:
//
//     dst chunk ((n / 16 * (row_bytes / 64) + cc / 4) * 64 + (cc % 4) * 16 + n % 16)  <-  src row n, chunk cc
// ---------------------------------------------------------------------------------------------
// One group of 32 tokens (grp = (kv head * NB + global block) * (b / 32) + group), by the threads of a workgroup.
__device__ __forceinline__ void pack_group(const char *src_base, char *dst_base, long long stride_h_bytes,
                                           long long stride_t_bytes, int row_bytes, int b, int NB, int frag16,
                                           const SeqTable &seqs, long long grp)
{
    const int cpr = row_bytes / 16;           // 16-byte chunks per row
    const int groups = b / 32;
    const int gi = (int)(grp % groups);
    const long long t = grp / groups;
    const int gb = (int)(t % NB);
    const int kvh = (int)(t / NB);
    const int s = seq_of_block(seqs, gb);
    const SeqDesc sd = seqs.d[s];
    const int r = gb - sd.blk0;
    const int tok_in_seq0 = r * b + gi * 32;
    char *dst = dst_base + grp * (32LL * row_bytes);
    for (int c = threadIdx.x; c < 32 * cpr; c += blockDim.x) {
        const int n = c / cpr, cc = c % cpr;
        const int fr = cc >> 1, g = cc & 1;
        uint4 v = make_uint4(0, 0, 0, 0);
        const int tok = tok_in_seq0 + n;
        if (tok < sd.len)
            v = *reinterpret_cast<const uint4 *>(src_base + kvh * stride_h_bytes +
                                                 (sd.tok0 + tok) * stride_t_bytes + cc * 16);
        int chunk = fr * 64 + g * 32 + n;
        if (frag16) {
            // fragment (16-row group n / 16, 64-byte slice cc / 4), lane (chunk cc % 4 of the slice, row n % 16)
            const int kf = cpr >> 2;
            chunk = ((n >> 4) * kf + (cc >> 2)) * 64 + (cc & 3) * 16 + (n & 15);
        }
        *reinterpret_cast<uint4 *>(dst + chunk * 16) = v;
    }
}

}  // namespace stream
