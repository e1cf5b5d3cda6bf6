// Launch geometry of the group kernels on the 16x16 matrix instructions (gconv_gemm.hip), made once a call.
#pragma once
#include <stddef.h>

namespace dwc {

// How the 256 lanes of a block copy a tile into LDS where FAST holds: lane t takes item t % per of row t / per, so that the divisions
// are done once and an item costs a few additions; `rows` rows in nrit steps of RPI, for every `cols` columns of a wider tile again.
// NHWC: an item is 16 bytes of channels of a pixel, a row one of the tile (all images); NCHW: four channels of four columns, a row one
// of a channel quad.
struct StageGeom {
    int LH, LW, pitch;               // the tile: rows of an image, columns, elements between pixels
    int imrows, rows, cols, per, nv; // imrows: rows of all images; nv: items of a pixel (NHWC)
    int width;                       // items of a row
    int RPI, nrit, iters;
    float rper, rnv, rLH, rimrows;
};

// One launch: the convolution from `in` (CI channels, Hi x Wi) to `out` (CO channels, Ho x Wo).  Position (a, b) of a tile
// reads input row IS*a - ip + roff and writes output row OS*a + f - op; roff = kh forward, -k for tap kh = f + OS*k backward.
struct GemmGeom {
    int N, CI, CO, Hi, Wi, Ho, Wo;
    int Cgi, Cgo;          // channels per group, input and output side
    int K, IS, OS, ip, op;
    int a0, na, b0, nb;    // positions of the whole image
    int bwd;
    int pairs, shift;      // E = 2: a position's outputs are columns 2b - 2*(op/2) and the next one; shift: odd op, the second one is class 0 of position b + 1
    // tile
    int TN, TA, TB;        // images, rows and columns of positions
    int tn, ta, tb;        // tiles in each direction
    int LH, LW;            // input pixels of a tile, per image
    int lo;                // lowest roff (backward: -(taps per class - 1))
    int NS, nk, CL, pitch; // 16-channel output blocks, 16-channel input chunks of each, channels in LDS, elements between pixels
    int nchb;              // channel blocks
    int packed;            // output blocks span groups
    int FO, FCg;           // filter dims: output channels, input channels per group (of the forward layer)
    float rCgi, rCgo, rKK, rnk, rTA, rTB, rta, rtb;         // reciprocals for fdiv
};

// lds: bytes of a block; npair: pairs of channel blocks of a block (filter gradient); fast: form of the staging; quad: fragments between quads of the filter
struct GemmPlan { GemmGeom g; StageGeom sg, sy; size_t lds; int nparts; unsigned nblocks; int npair, CLy, pitchy, fast, quad; };

}  // namespace dwc
