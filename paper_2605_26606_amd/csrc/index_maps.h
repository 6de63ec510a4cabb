// Index maps shared by kernels and host code (plain integer arithmetic, usable on either side; the host
// build of the tests checks them exhaustively on the CPU).
#pragma once

#include <stdint.h>

#if defined(__HIPCC__) || defined(__CUDACC__)
#define PC_HD __host__ __device__
#else
#define PC_HD
#endif

namespace pc {

// ---- KV cache, operand-fragment order (head_dim a multiple of 32, block_size a multiple of 32).
// Element offset of K[token tin][dim d] inside the K half of one (block, kv head) region: tiles of 32 tokens,
// a tile = 2 x (head_dim / 32) fragments [u][kk] of 512 elements; lane (i, g) of fragment (u, kk) holds dims
// 32 kk + 8 g .. + 7 of token 8 (i / 4) + i % 4 + 4 u of the tile, at element (16 g + i) * 8 of the fragment.
PC_HD inline int kv_k_index_frag(int tin, int d, int head_dim) {
    const int tt = tin & 31, u = (tt >> 2) & 1, i = ((tt >> 3) << 2) | (tt & 3);
    const int frag = ((tin >> 5) * 2 + u) * (head_dim >> 5) + (d >> 5);
    return (frag << 9) + (((((d & 31) >> 3) << 4) + i) << 3) + (d & 7);
}
// Element offset of V[token tin][dim d] inside the V half: tiles of 32 tokens, a tile = head_dim / 16 fragments
// [nn]; lane (i, g) of fragment nn holds tokens 8 g .. 8 g + 7 of dim 16 nn + i.
PC_HD inline int kv_v_index_frag(int tin, int d, int head_dim) {
    const int frag = (tin >> 5) * (head_dim >> 4) + (d >> 4);
    return (frag << 9) + (((((tin & 31) >> 3) << 4) + (d & 15)) << 3) + (tin & 7);
}

// ---- Weight matrices [N][K] of the 16-bit projections.  lg = 0: plain rows.  lg = WEIGHT_SLAB: slabs of 32 rows x 64 k (4 KB), a
// row's 128 bytes behind the previous row's, the slabs of 32 rows one after another along K: the eight rows x 64 k that a
// wave-wide load of the GEMMs takes are one contiguous kilobyte, the loads that follow it the same slab's and the next one's.  Both orders
// timed in turn, several passes side by side: 16 decode steps of 256 sequences x 28 layers of the 1.5B shape 31.17 -> 30.14 ms, of 1024 x 4 layers 17.74
// -> 17.19, 32 of three x 8 layers 9.44 -> 9.18, 16 of 168 x 3 layers of the 14B shape in bfloat16 (whose lm_head stays in plain rows) 16.83 ->
// 16.64, 8B steps and prefills as before; gate/up alone 26.2 -> 23.5 us (19.3 in either order if the weights lie in the last-level cache), the head
// 149 -> 142.
// weight_row: element offset of the first 64 k of row r; the next 64 lie 64 << lg elements on.
constexpr int WEIGHT_SLAB = 5;
PC_HD inline int64_t weight_row(int64_t r, int64_t K, int lg) { return ((r >> lg) << lg) * K + (r & ((1 << lg) - 1)) * 64; }
PC_HD inline int64_t weight_at(int64_t r, int64_t k, int64_t K, int lg) { return weight_row(r, K, lg) + ((k >> 6) << (6 + lg)) + (k & 63); }

// ---- GEMM, many row blocks (a multiple of 8): workgroup id -> output tile.  Workgroup i runs on die i % 8.
// Every die owns mb / 8 row blocks and walks all column blocks in groups of 8, patch by patch of `ph` row
// blocks x 8 column blocks (ph = 4 where mb / 8 allows), so that the 32 blocks a die runs at a time share few
// activation and weight slabs.  Returns false for ids past the last tile.
PC_HD inline bool gemm_patch_tile(int id, int mb, int nb, int *bm, int *bn) {
    const int die = id % 8, j = id / 8;
    const int rows_per = mb / 8;
    if (j >= rows_per * nb) return false;
    const int ph = (rows_per % 4 == 0) ? 4 : ((rows_per % 2 == 0) ? 2 : 1);
    const int full = rows_per * 8;                        // tiles of a full group of 8 column blocks
    const int last = (nb - 1) / 8;
    const int cg = (j / full < last) ? j / full : last;
    const int w = (nb - 8 * cg < 8) ? nb - 8 * cg : 8;
    const int jj = j - cg * full;
    const int sg = jj / (ph * w), r = jj % (ph * w);
    *bm = die * rows_per + sg * ph + r % ph;
    *bn = 8 * cg + r / ph;
    return true;
}

// ---- GEMM in runs of tiles: workgroup -> its i-th output tile (of `run`), K slice included.  The mb x nb x S tiles are walked
// in bands of `bh` row blocks (the last one may be lower), a band column by column; every die takes one eighth of that walk
// and its workgroups, 32 at a time (one per CU), neighbouring places of it: they share bh activation and 32 / bh weight slabs
// through the die's L2.  False: no such tile.
PC_HD inline bool gemm_band_tile(int block, int i, int run, int mb, int nb, int S, int bh, int *bm, int *bn, int *z) {
    const int die = block % 8, j = block / 8;
    const int64_t total = (int64_t)mb * nb * S, share = (total + 7) / 8;
    const int64_t pos = (int64_t)(j / 32) * 32 * run + 32 * i + j % 32, p = die * share + pos;
    if (pos >= share || p >= total) return false;
    const int nu = nb * S, band = (int)(p / ((int64_t)bh * nu));
    const int h = (mb - band * bh < bh) ? mb - band * bh : bh;
    const int r = (int)(p - (int64_t)band * bh * nu);
    *bm = band * bh + r % h;
    *bn = (r / h) % nb;
    *z = (r / h) / nb;
    return true;
}
// Grid, band height and run length for it.  A run costs its first tile's wait for memory once; up to six tiles, so that a
// workgroup which comes late (another stream's kernel on its CU) does not hold the rest up for long.
inline unsigned gemm_band_grid(int mb, int nb, int S, int *bh, int *run) {
    const int64_t share = ((int64_t)mb * nb * S + 7) / 8;         // tiles per die
    const int64_t rounds = (share + 31) / 32, parts = (rounds + 5) / 6;
    *run = (int)((rounds + parts - 1) / parts);
    const int bands = (mb + 7) / 8;
    *bh = (mb + bands - 1) / bands;
    const int64_t groups = (share + 32 * *run - 1) / (32 * *run);    // groups of 32 workgroups per die
    return (unsigned)(groups > 1 ? groups * 256 : 8 * (share < 32 ? share : 32));
}

}   // namespace pc
