// Rules that choose a conv's kernel and tile by its sizes (host).
#pragma once

#include <cstdint>

namespace sg {

// Tile of the forward and data-gradient GEMM of M pixels (nz times: the parity classes) and N channels.  A compute
// unit runs its share of the blocks one after the other (256 units), so a tile's time goes up in steps: a block of
// 128 x 128 has the most products per fetched operand, but below 190 of them too many units stand idle, and 64 x 64
// ones are as fast as long as they come to two or three rounds (two share a unit almost for free).  us with 128 x 128 /
// 128 x 64 / 64 x 64 / 32 x 64 tiles, [blocks] of the first:
//   512 -> 512 channels 3x3, 2976 pixels [96]     43 /  33 /  27 /  31     14880 [468]   94 / 154 / 175 / 242
//   512 -> 136 3x3,          8928 pixels [140]    49 /  39 /  35 /  49     14880 [234]   50 /  58 /  61 /  78
//   1024 -> 256 1x1,         6944 pixels [110]    15 /  13 /  12 /  17     32550 [510]   27 /  43 /  44 /  57
// A second round of a few 128 x 128 blocks is worse than two of 128 x 64 (96 -> 192 3x3, 17670 pixels: [278] 18.2,
// [417] 13.8).  Over 691 such layers the rule is on average 1.4 % slower than the best tile of each; the largest tile
// that gives two blocks per unit would be 8.8 % slower, 128 x 128 always 15 %.  Up to 64 channels the same line is
// between 64 x 64 and 128 x 64 (256 -> 64 3x3: 32550 pixels 19.9 and 21.4, 65100 pixels 44 and 34), up to 32 and 16 the tall
// tiles pay from 350 blocks on (256 -> 32 3x3, 56730 pixels [444]: 26.5 against 29.5; 72 -> 8 130200 [509]: 15.9 against
// 17.8).
struct GemmTile {
    int bm, bn;
};
inline GemmTile gemm_tile(int64_t M, int64_t N, int nz)
{
    auto blocks = [&](int bm, int bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn) * nz; };
    if (N <= 16) return blocks(256, 16) >= 350 ? GemmTile{256, 16} : GemmTile{64, 16};
    if (N <= 32) return blocks(128, 32) >= 350 ? GemmTile{128, 32} : GemmTile{64, 32};
    const int64_t b64 = blocks(64, 64);
    if (N <= 64) {
        if (b64 > 640) return GemmTile{128, 64};
    } else {
        const int64_t b128 = blocks(128, 128);
        if (b128 > 256 && blocks(128, 64) <= 512) return GemmTile{128, 64};
        if (b128 >= 190 || b64 > 640) return GemmTile{128, 128};
    }
    return b64 >= 128 ? GemmTile{64, 64} : GemmTile{32, 64};
}

// Blocks of the halo kernel: 16 x 16 output pixels of an image for 64 channels, each computed whole.
constexpr int kHaloT = 16, kHaloN = 64;
inline int64_t halo_blocks(int Co, int64_t images, int Ho, int Wo)
{
    return (int64_t)((Ho + kHaloT - 1) / kHaloT) * ((Wo + kHaloT - 1) / kHaloT) * images * (Co / kHaloN);
}
// Whether that kernel is faster than the GEMM (C input channels, those of dy as data gradient).  Below one block per
// compute unit (256) the GEMM's smaller tiles are as fast (128 -> 64 upsampled, 128 blocks 13.4 against 12.9 us).  Its time
// goes with the rounds of 256 blocks, the GEMM's with the output pixels, so what decides is the share of useful pixels in
// whole rounds: half of them up to two rounds, 0.64 beyond (us, halo against GEMM; 64 -> 64: 256 images of 16 x 16, one
// round, 10.3 and 12.0, 72 of 24 x 24, two rounds, 0.32, 11.8 and 10.2, 130 of them, three rounds, 0.38, 17.6 and 14.1;
// 128 -> 64: 16 of 50 x 50, one round, 0.61, 12.8 and 14.8, 32 of 40 x 40, two rounds, 0.39, 22.9 and 15.8; 256 -> 64
// upsampled: 16 of 50 x 50 19.4 and 23.8, 72 of 18 x 18, two rounds, 0.18, 28.7 and 18.9; 128 -> 64 upsampled, 4200 blocks 140
// and 182).  128 channels not upsampled take 107 KB of LDS, one block per compute unit: with 128 outputs and more, where
// the GEMM has its 128 x 128 tiles, one round or two nearly full ones (128 -> 128: 256 blocks 13.8 and 17.7, 330 23.9 and
// 22.2, 504 of 0.94 24.2 and 27.3, 800 46.6 and 44.2), with 64 up to 1024 blocks.  As data gradient it takes whole tiles only and wins at any share
// (128 -> 128, 290 blocks 26.2 and 27.4; 64 -> 64, 580 blocks 15.6 and 19.3).
inline bool halo_pays(bool dgrad, int C, int Co, bool up, int64_t images, int Ho, int Wo)
{
    const int64_t blocks = halo_blocks(Co, images, Ho, Wo), rounds = (blocks + 255) / 256;
    const bool wide = C == 128 && !up;
    if (blocks < 256 || (wide && blocks >= 1024)) return false;
    if (dgrad) return true;
    const int64_t useful = images * Ho * Wo * (Co / kHaloN), whole = rounds * 256 * kHaloT * kHaloT;
    if (wide && Co > kHaloN && rounds > 1) return rounds == 2 && 5 * useful >= 4 * whole;
    return rounds <= 2 ? 2 * useful >= whole : 25 * useful >= 16 * whole;
}

}  // namespace sg
