// The kernel variant space: the knobs the per-layer tuner chooses from, the
// counterpart of the paper's tile-size / LMUL template parameters (section 3.3).
//   NBLK 16-pixel MFMA blocks per wavefront   WP  wavefronts along the pixel axis
//        (pixels per workgroup BP = 16*NBLK*WP)
//   NJ  16-channel row blocks per wavefront
//   CK  im2col rows per LDS chunk      SPC k-steps (4 kept columns each) per chunk
//   VEC 1: chunks are channel runs of one tap fetched 16 bytes at a time
//       0: chunks are cut on the flat k axis, fetched element-wise (Cin % 4 != 0)
#pragma once

// X(NBLK, WP, NJ)
#define NM_SHAPES(X) \
    X(8, 1, 2) X(8, 1, 4) X(4, 2, 4) X(4, 2, 2) X(8, 2, 2) X(4, 4, 4) \
    X(4, 1, 2) X(4, 1, 4) X(4, 1, 1)                                  \
    X(1, 4, 1) X(1, 4, 2) X(2, 1, 1) X(2, 1, 2) X(2, 2, 1) X(2, 2, 2) \
    X(3, 1, 1) X(3, 1, 2) X(5, 1, 1) X(6, 1, 1) X(6, 1, 2) X(7, 1, 1) \
    X(7, 1, 2) X(7, 2, 1) X(8, 1, 1) X(10, 1, 1) X(12, 1, 1)          \
    X(13, 1, 1) X(13, 1, 2) X(14, 1, 1) X(16, 1, 1) X(16, 1, 2)

// Y(NBLK, WP, NJ, CK, SPC, VEC)
#define NM_VEC_CHUNKS(Y, NB, WP, NJ)                                              \
    Y(NB, WP, NJ, 32, 2, 1) Y(NB, WP, NJ, 32, 4, 1) Y(NB, WP, NJ, 32, 8, 1)       \
    Y(NB, WP, NJ, 64, 2, 1) Y(NB, WP, NJ, 64, 4, 1) Y(NB, WP, NJ, 64, 8, 1)

// fp32 kernel with a per-(tile, chunk) number of k-steps: for kept sets that are not
// spread evenly over the chunks (group size M larger than a chunk).  SPC = CK / 4 is
// the width of the operand table, not the work done.
// X(NBLK, WP, NJ)
#define NMVAR_SHAPES(X)                                                             \
    X(2, 1, 1) X(3, 1, 1) X(4, 1, 1) X(5, 1, 1) X(6, 1, 1) X(7, 1, 1) X(8, 1, 1)    \
    X(10, 1, 1) X(13, 1, 1) X(2, 1, 2) X(4, 1, 2) X(8, 1, 2) X(2, 2, 1) X(4, 2, 2)
// Y(NBLK, WP, NJ, CK, SPC)
#define NMVAR_CHUNKS(Y, NB, WP, NJ) Y(NB, WP, NJ, 32, 8) Y(NB, WP, NJ, 64, 16)

#define NM_SCALAR_VARIANTS(Y) Y(4, 4, 4, 32, 8, 0) Y(4, 2, 2, 32, 8, 0) Y(4, 1, 1, 32, 8, 0)

// bf16 matrix-core kernel (bf16 activations, bf16-rounded weights):
//   SHARE row blocks of one column tile are fed from the same gathered operand (2 for T = 32)
//   a k-step is 32 kept columns; CK channels per chunk hold SPC k-steps
// X(NBLK, WP, NJ, SHARE)
#define NM16_SHAPES(X)                                                              \
    X(8, 1, 2, 1) X(8, 1, 1, 1) X(4, 1, 2, 1) X(4, 1, 1, 1) X(4, 2, 2, 1) X(2, 1, 2, 1) \
    X(2, 1, 1, 1) X(5, 1, 1, 1) X(6, 1, 1, 1) X(12, 1, 1, 1) X(16, 1, 1, 1)            \
    X(8, 1, 2, 2) X(4, 1, 2, 2) X(4, 2, 2, 2) X(2, 1, 2, 2) X(4, 1, 4, 2)
// Y(NBLK, WP, NJ, SHARE, CK, SPC)
#define NM16_CHUNKS(Y, NB, WP, NJ, SH)                                              \
    Y(NB, WP, NJ, SH, 32, 1) Y(NB, WP, NJ, SH, 64, 1) Y(NB, WP, NJ, SH, 128, 1)     \
    Y(NB, WP, NJ, SH, 64, 2) Y(NB, WP, NJ, SH, 128, 2) Y(NB, WP, NJ, SH, 256, 1)

// bf16 kernels that contract the dense strip without a gather: the sparse
// matrix instruction (SP = 1: N <= 2 kept of every aligned 4 columns) or the
// dense one on zero-filled weights (SP = 0).  A chunk is CK channels of one tap.
// X(NBLK, WP, NJ)
#define NMSP_SHAPES(X)                                                          \
    X(4, 1, 2) X(4, 1, 4) X(2, 1, 2) X(2, 1, 4) X(4, 2, 2) X(4, 2, 4) X(8, 1, 2) \
    X(8, 1, 1) X(4, 1, 1) X(2, 1, 1) X(2, 2, 2) X(6, 1, 2) X(3, 1, 2) X(2, 2, 4)
// Y(NBLK, WP, NJ, CK, SP)
#define NMSP_CHUNKS(Y, NB, WP, NJ)                                   \
    Y(NB, WP, NJ, 64, 1) Y(NB, WP, NJ, 128, 1) Y(NB, WP, NJ, 256, 1) \
    Y(NB, WP, NJ, 64, 0) Y(NB, WP, NJ, 128, 0) Y(NB, WP, NJ, 256, 0)

// The same kernels with four producer wavefronts that issue the loads (512 threads).
// X(NBLK, WP, NJ)
#define NMSPW_SHAPES(X) X(8, 1, 2) X(4, 1, 2) X(4, 2, 4) X(4, 1, 4) X(4, 2, 2) X(6, 1, 2) X(2, 1, 2) X(2, 2, 4)
// Y(NBLK, WP, NJ, CK, SP)
#define NMSPW_CHUNKS(Y, NB, WP, NJ)                                  \
    Y(NB, WP, NJ, 64, 1) Y(NB, WP, NJ, 128, 1) Y(NB, WP, NJ, 256, 1) \
    Y(NB, WP, NJ, 64, 0) Y(NB, WP, NJ, 128, 0) Y(NB, WP, NJ, 256, 0)

// Producer wavefronts, and the weights loaded straight into the contracting wavefronts'
// registers (the LDS stages hold the strip alone).  112 pixels for images of 7, 14 and 28 pixels a row, whose tiles of 128 fill one
// round of workgroups or two by 77 %, those of 112 by 88: batch 256, T = 32, out of cache, the fastest with 128 and with 112, 14x14
// 1024 -> 256 36.2 and 34.9 us, 1024 -> 512 4:8 73.6 and 66.2, 512 -> 512 3x3 stride 2 4:8 55.1 and 50.6, 7x7 2048 -> 512 4:8 29.0 and
// 27.1; batch 64 14x14 1024 -> 256 9.8 and 9.4.  (224 x 128 was first on none of them.)
// X(NBLK, WP, NJ)
#define NMSPR_SHAPES(X) X(7, 1, 4) X(7, 1, 2) X(4, 2, 4) X(8, 1, 2) X(4, 1, 4) X(2, 2, 4) X(8, 2, 4) X(4, 2, 2) X(8, 1, 4) X(6, 1, 2)
// Y(NBLK, WP, NJ, CK, SP)
#define NMSPR_CHUNKS(Y, NB, WP, NJ)             \
    Y(NB, WP, NJ, 64, 1) Y(NB, WP, NJ, 128, 1) \
    Y(NB, WP, NJ, 64, 0) Y(NB, WP, NJ, 128, 0)

// k x k layers whose output is as large as the input: a tile's input staged once for all taps, 64 channels at a time;
// sparse instruction and dense one.  (64 x 256 and 128 x 128 tiles, 96 x 256 and 192 x 128 were first on no layer.)
// X(NBLK, WP, NJ)
#define NMTAPS1_SHAPES(X) X(4, 1, 2) X(5, 2, 4) X(7, 2, 4) X(8, 2, 4) X(8, 1, 4) X(7, 4, 4) X(8, 4, 4)
#define NMTAPS0_SHAPES(X) X(5, 2, 4) X(7, 2, 4) X(7, 4, 4)
// the same with eight contracting wavefronts (512 x 64, 320 x 128, 128 x 256 and, dense, 256 x 128 were first on no layer)
#define NMTAPSW1_SHAPES(X) X(7, 2, 4) X(8, 2, 4)
#define NMTAPSW0_SHAPES(X) X(7, 2, 4) X(7, 2, 2)

// 1x1 layers of up to 256 input channels: the input of 16 NBLK pixels stays, the output channels pass
// X(NBLK); Y(NBLK, chunks of 64 input channels)
#define NMCOLS_SHAPES(X) X(4) X(2)
#define NMCOLS_CHUNKS(Y, NB) Y(NB, 1) Y(NB, 2) Y(NB, 3) Y(NB, 4)

// bf16 kernel for layers with very few input channels (contiguous kernel-row
// runs, one chunk of KS 64-element k-steps): where output pixels are not whole
// 16-byte granules or the staged rows do not fit the CU, and for very few pixels.
// X(NBLK, WP, NJ)
#define NMRUN_SHAPES(X) \
    X(4, 1, 1) X(8, 1, 1) X(2, 1, 1) X(2, 2, 2) X(4, 2, 2) X(2, 4, 4) X(4, 4, 4) X(1, 4, 4) X(3, 4, 4) X(7, 1, 1)
// Y(NBLK, WP, NJ, KS)
#define NMRUN_CHUNKS(Y, NB, WP, NJ) Y(NB, WP, NJ, 1) Y(NB, WP, NJ, 2) Y(NB, WP, NJ, 3) Y(NB, WP, NJ, 4)

// fp8 through the staged kernel of the gather-free bf16 form (LDS ring, optional producer
// wavefronts and register-held weights): CK E4M3 channels of one tap per chunk.  (112 pixels as in bf16: 14x14 1024 -> 256 at batch 64
// 8.2 and 7.8 us, 256 -> 256 3x3 11.5 and 10.7.)
// X(NBLK, WP, NJ)
#define NMF8S_SHAPES(X) X(7, 1, 2) X(8, 1, 2) X(4, 1, 2) X(4, 1, 1) X(6, 1, 2) X(4, 2, 2) X(8, 1, 4) X(4, 2, 4) X(4, 1, 4) X(2, 1, 2)
// Y(NBLK, WP, NJ, CK)
#define NMF8S_CHUNKS(Y, NB, WP, NJ) Y(NB, WP, NJ, 64) Y(NB, WP, NJ, 128) Y(NB, WP, NJ, 256)

// fp8 (E4M3 activations and weights, bf16 output): both operands streamed from global memory
// into registers, 64-channel k-steps.
// X(NBLK, WP, NJ)
#define NMF8_SHAPES(X) \
    X(4, 1, 4) X(4, 2, 4) X(4, 4, 4) X(2, 1, 4) X(2, 2, 4) X(2, 4, 4) X(4, 1, 2) X(4, 2, 2) X(8, 1, 2) X(8, 2, 2)

// fp32 tensors as three bf16 planes (64-channel chunks, four producer and four contracting wavefronts):
// the sparse instruction and the dense one.  (128-pixel tiles were tried: their two stages leave a CU one
// workgroup, and they were first on no layer of the ResNet-50 stack.)
// X(NBLK, WP, NJ)
#define NMSS_SHAPES(X) X(4, 1, 2) X(4, 1, 4) X(3, 1, 2) X(2, 1, 2) X(2, 2, 2) X(4, 1, 1) X(2, 1, 1)
#define NMSD_SHAPES(X) X(4, 1, 2) X(2, 1, 2) X(2, 2, 2) X(4, 1, 1) X(2, 1, 1)

// k x k layers of the same whose output is as large as the input: a tile's input staged and cut once for all taps, eight
// contracting wavefronts in KG groups that take the chunks in turn (128-pixel tiles were first on no layer)
// X(NBLK, WP, NJ, KG)
#define NMST1_SHAPES(X) X(4, 1, 4, 2) X(4, 1, 4, 4)
#define NMST0_SHAPES(X) X(4, 1, 2, 2) X(4, 1, 2, 4)

// few input channels out of staged input rows: R output rows a workgroup, 64 channels, KS 64-element k-steps
// Y(NJ, KS); X(R, NJ, KS)
#define NMROWB_CHUNKS(Y) Y(4, 1) Y(4, 2) Y(4, 3) Y(4, 4)
#define NMROWF_CHUNKS(Y) Y(1, 1) Y(1, 2) Y(1, 3) Y(1, 4) Y(2, 1) Y(2, 2) Y(2, 3)
#define NMROW_HEIGHTS(X, NJ, KS) X(1, NJ, KS) X(2, NJ, KS) X(4, NJ, KS) X(8, NJ, KS)

// small fp32 layers: the K axis over up to NW wavefronts of a workgroup of 16 PB pixels x 16 NJ channels (as many as
// leave each the registers of two chunks).  (64-channel chunks and 32 pixels x 16 channels were first on no layer by
// more than 3 %.)
// X(PB, NJ); Y(PB, NJ, CK, SPC, NW)
#define NMWAVE_SHAPES(X) X(1, 1) X(1, 2) X(2, 2) X(1, 4)
#define NMWAVE_1_1(Y) Y(1, 1, 32, 2, 16) Y(1, 1, 32, 4, 16) Y(1, 1, 32, 8, 16)
#define NMWAVE_1_2(Y) Y(1, 2, 32, 2, 16) Y(1, 2, 32, 4, 16) Y(1, 2, 32, 8, 16)
#define NMWAVE_2_2(Y) Y(2, 2, 32, 2, 16) Y(2, 2, 32, 4, 12) Y(2, 2, 32, 8, 12)
#define NMWAVE_1_4(Y) Y(1, 4, 32, 2, 16) Y(1, 4, 32, 4, 16) Y(1, 4, 32, 8, 8)
