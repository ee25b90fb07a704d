// Layout of the cross kernels' partial sums, shared by the cross kernels
// (kernels_cross.hip) and the scoring kernel that reads them
// (kernels_score.hip): the support ranges of the direct (VALU) kernel and of
// the batch-stationary MFMA kernel, and their launch shapes.
#pragma once

#include "mbkk_internal.h"

namespace mbkk {

// Ranges of the direct kernel: the concatenated support is cut into nranges
// ranges of RR rows (RR from the support size, so the scoring kernel derives
// the same cut); a run is a range's stretch of one center's segment.  Run id:
// the center j for the run that starts at the center's first row, k + r for
// the run that starts at the start of range r inside a center.
// Small supports (direct_min_rows): a range holds at least kDirectMinRows
// entries, whose terms are then summed in FP64 before the partial is stored.
// The scoring reads a partial per range, and with b = 256, k = 3 (2-D blobs)
// one-entry ranges gave it 340 per center to read, 65 us; with 8 it is 8 us and
// the cross kernel no slower.
constexpr int kDirectMinRows = 8;
__host__ __device__ inline int direct_range_rows(int M, int nranges, int min_rows)
{
    const int r = (M + nranges - 1) / nranges;
    return r > min_rows ? r : min_rows;
}

// Batch rows per lane of the direct kernel: two for FP32 rows of at most 32
// coordinates (each broadcast support row then feeds two evaluations).
inline int direct_rpl(int d, bool fp64) { return !fp64 && d <= 32 ? 2 : 1; }

// Ranges of the direct kernel for nb batch rows: about kDirectWGs workgroups
// (one round at 8 waves per SIMD), 3/4 of that with two rows per lane (whose
// registers allow 6 waves per SIMD).  In FP64 a row of 33 to 64 coordinates
// takes 168 registers, 3 waves per SIMD, one of 17 to 32 takes 106, 4 waves: one
// round of workgroups there while the ranges are short (b = 1024, M = 4096,
// d = 64: nine entries per range, behind a start of two load round trips, took
// 99 us; 22 entries take 63 us), and kDirectWGs again from 128 entries of a full
// support per range on, where the starts weigh less than what the last workgroups
// keep waiting (d = 64, one round against kDirectWGs: M = 8242, b = 2048, 86 entries
// 174 and 184 us; M = 12308, b = 2048, 129 entries 260 and 261 us; M = 16404,
// b = 4096, 342 entries 618 and 572 us; d = 32: 64 entries 96 and 97 us, 128
// entries 170 and 162 us).
inline int direct_nranges(const Layout &L, int nb, bool fp64)
{
    const int rpl = direct_rpl(L.d, fp64);
    const int tiles = (nb + 256 * rpl - 1) / (256 * rpl);
    int wgs = rpl == 2 ? kDirectWGs * 3 / 4 : kDirectWGs;
    if (fp64 && L.d > 16 && L.d <= 64) {
        const int one = L.d > 32 ? kDirectWGs * 3 / 8 : kDirectWGs / 2;
        if (L.Mcap * tiles / one < 128)
            wgs = one;
    }
    const int r = wgs / tiles;
    return r < 1 ? 1 : r;
}

// Fewest entries per range: kDirectMinRows where the fullest support has no
// more per range anyway (so that every larger one keeps its cut), else 1; also
// 1 past 64 coordinates, where a lane reads its batch row again for every
// entry and the cross kernel needs the workgroups (Laplacian, b = 64, 784
// coordinates: 78 us in ranges of one entry, 549 us of 8; 100 coordinates, b = 256:
// 51 and 104 us).
inline int direct_min_rows(const Layout &L, int nranges)
{
    return L.d <= 64 && (L.Mcap + nranges - 1) / nranges <= kDirectMinRows ? kDirectMinRows : 1;
}

constexpr int kBsStageBlocks = 4;  // support blocks (32 rows) per stage of the MFMA kernel

// Blocks per range for Mb support blocks split over nranges ranges (the
// kernel's last stage of a range skips the blocks past it).
__host__ __device__ inline int bs_range_blocks(int Mb, int nranges) { return (Mb + nranges - 1) / nranges; }

// Waves per SIMD: two in the BF16X3 form with row stride above 64, whose
// two waves on a SIMD take turns, one issuing MFMAs while the other runs its
// exp epilogue or waits on LDS; one elsewhere (the FP32 MFMAs are twice as
// long, and at stride 64 the register file holds four N-blocks per wave).
__host__ __device__ constexpr int bs_wps(int mode, int dp) { return mode == 1 && dp > 64 ? 2 : 1; }
// Batch rows held in registers per wave, in 32-row N-blocks: as many as the
// register file allows (one wave per SIMD: 256 VGPRs + 256 AGPRs; two waves:
// half each) with two accumulator sets (the pipelined epilogue) and few
// copies between the two register kinds.  FP32 fragments are 2x larger and
// each FP32 MFMA is 2x longer, so two N-blocks already amortise the support
// reads.
__host__ __device__ constexpr int bs_nbk(int mode, int dp) { return mode == 0 ? 2 : (mode == 1 && dp > 64 ? 1 : 4); }
inline int bs_tile_rows(int mode, int dp) { return 4 * bs_wps(mode, dp) * 32 * bs_nbk(mode, dp); }
inline int bs_mode(int precision) { return precision == MBKK_FP32 ? 0 : (precision == MBKK_BF16X3 ? 1 : 2); }
// Ranges for nb batch rows: one round of workgroups (kBsOcc per compute unit).
inline int bs_nranges(int nb, int mode, int dp)
{
    const int tr = bs_tile_rows(mode, dp);
    const int nbt = (nb + tr - 1) / tr;
    const int r = kNumCU * kBsOcc / nbt;
    return r < 1 ? 1 : r;
}

// A center's cross term from the partials of the MFMA kernels, summed in FP32.
// LAYOUT 1: one partial per run of a center's blocks inside a range of RB
// blocks, at the run's first block: the center's first block and every range
// start inside the center.
// LAYOUT 2 (packed segments, which may start inside a block): two slots per
// block, 2 b for the run from block b's first row (a range start, or a center
// starting there) and 2 b + 1 for a center starting inside block b; a
// center's partials are its first slot and slot 2 b of every range start b
// after its first block and inside its segment.
template <typename T, int LAYOUT>
__device__ __forceinline__ double cross_of(const T *__restrict__ part, int ldp, int row, int j,
                                           const int32_t *__restrict__ seg_off, int RB)
{
    if constexpr (LAYOUT == 1) {
        const int bs = seg_off[j] / 32, be = seg_off[j + 1] / 32;
        if (bs >= be)
            return 0.0;
        float s = part[(int64_t)bs * ldp + row];
        for (int blk = (bs / RB + 1) * RB; blk < be; blk += RB)
            s += part[(int64_t)blk * ldp + row];
        return (double)s;
    } else {
        const int s0 = seg_off[j], s1 = seg_off[j + 1];
        if (s0 >= s1)
            return 0.0;
        const int b0 = s0 / 32;
        float s = part[(int64_t)(2 * b0 + (s0 % 32 != 0)) * ldp + row];
        for (int blk = (b0 / RB + 1) * RB; 32 * blk < s1; blk += RB)
            s += part[(int64_t)(2 * blk) * ldp + row];
        return (double)s;
    }
}

}  // namespace mbkk
