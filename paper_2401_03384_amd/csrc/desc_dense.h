// Descriptors of the dense-kernel path: a layer (or step) evaluated as one
// 2-D convolution with its merged kernel W[t][s][kh][kw].  Host-only types,
// shared by the planner and the HIP kernels.
#pragma once

#include <cstdint>

namespace ce {

// Pixel tile of the dense convolution kernels: NI images x TH output rows x
// all OW columns, staged with its halo in LDS as HP x WP slots an image.
// Input position of output row p, tap i: sth * p + zh0 + zhs * i (columns the
// same with stw, zw0, zws), zero outside the plane.
struct DTile {
    int32_t B, H, W, OH, OW, KH, KW;
    int32_t zh0, zhs, zw0, zws, sth, stw;
    int32_t NI, TH, HP, WP, slots;     // slots = NI * HP * WP
    int32_t nth, npt;                  // row tiles of an image group, pixel tiles
};

// Y[b][m][p] = sum_c sum_taps W[m][c][tap] X[b][c][pos(p, tap)] with W packed
// in the order the wavefronts read it: [m / 32][c chunk][tap][2][64 lanes][16
// bytes], lane l of a k step holding row l % 32 and the 16 bytes of channels
// that its half l / 32 multiplies (bf16: 8, fp32: 4; a chunk is 32 / 16).
struct DConvDesc {
    DTile t;
    int32_t C, M, nch, mblk, cfg;
    uint32_t lds_bytes;
    int64_t x_sb, x_sc;                // input strides (rows of a plane contiguous)
    int64_t y_sb, y_sm, y_sh, y_sw;    // output strides
    int64_t blocks;
};

// P[split][tap][t][s] = sum over the split's pixel tiles of
// G[b][t][p] X[b][s][pos(p, tap)]  (fp32 partials of the kernel's gradient)
struct DWgradDesc {
    DTile t;
    int32_t T, S, ntb, nsb, cfg, nsplit, PP, pad_;
    uint32_t lds_bytes, o_x, o_tab;    // LDS: G tile at 0, X tile at o_x, slot table at o_tab (bytes)
    int64_t x_sb, x_sc, g_sb, g_sc;
    int64_t blocks;
};

// The packed kernel of F (strides in elements: row, channel, taps).
struct DPackDesc {
    int32_t M, C, KH, KW, mt, nch;     // mt: tiles of 32 rows, nch: channel chunks
    int64_t sm, sc, sh, sw;
};

// Ordered sum of dwgrad's partials into C (strides in elements).
struct DWredDesc {
    int32_t T, S, KH, KW, nsplit, pad_;
    int64_t st, ss, sh, sw;
};

// Reshaped CP: W[t1 t2 t3][s1 s2 s3][j] = sum_r W1[r][t1][s1] W2[r][t2][s2]
// W3[r][t3][s3] W0[r][j], packed for the forward (rows t) or for the input
// gradient (rows s); and the factor gradients from the partials of dW.
struct DRcpDesc {
    int32_t R, T1, T2, T3, S1, S2, S3, KT;
    int32_t NJ, jper;                  // tap groups and taps a group
    int32_t transposed;                // merge: rows s, channels t
    int32_t nch;                       // merge: channel chunks of the packed kernel
    int32_t nsplit;                    // gradient: partials of dW
    int32_t nrc;                       // chunks of 64 ranks
    int64_t blocks;
};

// The reshaped-CP forward as one launch: each block merges the kernel rows it
// needs on chip.  A block: one t1 (rows t2 t3) x one pixel tile.
struct RcpDfwdDesc {
    DTile t;
    int32_t R, RK, T1, S1, S2, S3, T2, T3;   // RK: steps of 16 ranks
    int32_t nch, pad_;                       // chunks of 16 channels (all s1 of 16 / S1 (s2, s3) pairs)
    uint32_t o_f, o_w2, o_w3, o_w, o_x, lds_bytes;   // LDS bytes: rank tables, merged values, X buffers
    int64_t blocks;
};

}  // namespace ce
