// kf_route.h -- which kernel variant a call runs: rules on its sizes alone.
// Without HIP types, so that a host compiler can test the rules.
#pragma once

namespace kf {

// Training-mask attention: query rows per wavefront (32: 128-row workgroups, or
// 16: 64-row ones) and how a head's query rows are cut into workgroups.
struct TrainingRoute {
  bool rows32;
  int prow;      // rows that are cut into blocks by themselves: all nq, or half of them
  int blocks32;  // 128-row workgroups of a head
};

// 32 rows share each tile's transfer among twice the rows; 16 give twice the
// workgroups, half the serial work of each and less padding of the last block.
// Times of the 32-row kernel over the 16-row one (3529 shapes: both masks, 8 to 4096
// heads, N from 1 to 1000, k = 1, 2, 4, 8), by the number of 128-row workgroups
// ("grid"), blocks per part, and rows in the last one ("last"):
//   d_head 128  grid of 384 and more 0.82 on average; from 288 on with three blocks
//               and last > 64 0.9.  One block of 64 rows and less 1.04 to 1.22, two
//               blocks with last <= 32 from grid 1024 on up to 1.10, smaller grids
//               1.05 to 1.35
//   d_head 64   0.90 where last > 64 and the grid is of 512 and more and fills whole
//               rounds of 768 (three workgroups per CU) by 85 % (M_S: N under 256,
//               beyond it up to 1.06), or is of 3072, or the head is one block, or two
//               with last <= 96, or N is of 80 to 255 on a grid of 1024 (self-forcing
//               rollouts); on 3072 also where the padding of the last block is under
//               1/24 of the rows.  Else up to 1.40
//   d_head 32   0.85 where last > 64 on 768 and more (one block: 512), last >= 32 in
//               six blocks and more on 3072, or little padding on 1024.  Else up to 1.40
// The most among the shapes that the rule gives to the 32-row kernel is 1.07.
//
// M_D has two halves of N k rows.  A block across their border would walk nearly
// all Future-1 keys (the last groups see the last ones, the first groups the
// first): from 512 rows a half on, each half is cut by itself (8 heads, N = 600, k
// = 8, d_head 128: 67 -> 32 us; below that the block more costs up to 28 %).
inline TrainingRoute training_route(int dh, long long BH, bool two_parts, long long N, long long k,
                                    long long nq) {
  const bool cut = two_parts && N * k >= 512;
  const long long prow = cut ? nq / 2 : nq;
  const long long b32 = (prow + 127) / 128 * (cut ? 2 : 1), b16 = (nq + 63) / 64;
  const long long grid = BH * b32, blocks = (prow + 127) / 128, last = prow - 128 * (blocks - 1);
  const bool full = last > 64, whole = 48 * b32 <= 25 * b16;
  bool r32;
  if (dh == 128)
    r32 = (grid >= 384 && prow > 64 && !(blocks == 2 && last <= 32 && grid >= 1024)) ||
          (grid >= 288 && full && blocks >= 3);
  else if (dh == 64)
    r32 = (whole && grid >= 3072) ||
          (full && grid >= 512 &&
           (grid >= 3072 || blocks == 1 ||
            ((two_parts || N < 256) && 20 * grid >= 17 * 768 * ((grid + 767) / 768)) ||
            (blocks == 2 && last <= 96) || (N >= 80 && N < 256 && grid >= 1024)));
  else
    r32 = (whole && grid >= 1024) || (full && grid >= (blocks == 1 ? 512 : 768)) ||
          (blocks >= 6 && last >= 32 && grid >= 3072);
  return {r32, (int)prow, (int)b32};
}

// Block attention of a step over the paged KV cache (bf16).  Three kernels:
//   split  one workgroup of four wavefronts (two for contexts of at most 128 keys)
//          per 16 query rows and key split, ns splits, and a merge kernel if ns > 1
//   wide   eight wavefronts per 16 query rows, no split
//   tiled  128 query rows (d_head 128: 64) share each key tile and walk all keys
struct AttentionRoute {
  int ns;
  bool wide, tiled;
};

// B sequences, H heads, query rows [qoff, R) of each, T keys of capacity; entries:
// partial states that the split may write (0: none); empty: the step starts at an
// empty context (a prefill), so that its rows see R keys at most.
inline AttentionRoute attention_route(int dh, int B, int H, int R, int qoff, int T,
                                      long long entries, bool empty) {
  // key splits: enough workgroups for ~512 in flight, each split at least 128
  // keys of the full context, within the partial-state workspace
  const long long base = (long long)B * H * ((R - qoff + 15) / 16);
  int ns = 1;
  if (entries > 0 && base < 256) {
    ns = (int)(512 / base);
    ns = ns < T / 128 ? ns : T / 128;
    ns = ns < 16 ? ns : 16;
    while (ns > 1 && (long long)B * H * R * ns > entries) --ns;
    if (ns < 1) ns = 1;
  }
  // Decode grids of 64 to 255 query blocks at d_head 64 (batch 6 to 21 at 12
  // heads): measured on the OWT-shaped model at batch 16, attention 43.2 -> 31.0
  // ms per generate (the generate 139.6 -> 130.5 ms).  Smaller grids keep the
  // splits (batch 1 lost 4 % with eight wavefronts and no split), and grids of 256
  // blocks and more keep four wavefronts (batch 24 and 32 lost 5 %, batch 64 9 %,
  // batch 256 15 % with eight).
  const bool wide = dh == 64 && ns > 1 && base >= 64;
  // The tiled kernel reads each key R / 128 times where the others read it R / 16
  // times, but in fewer workgroups, each of which walks every tile.  Its time over
  // theirs (12 heads, 1 to 64 sequences, 32 to 1000 rows, T = 128 to 1024):
  //   few keys (a prefill, or T = 128)
  //     splits in their place         0.65 to 0.95: it saves the merge kernel
  //     no split, d_head 64           0.28 to 1.06 from 864 query blocks, or 576 of
  //                                   128 rows and more; fewer 0.91 to 1.18
  //     no split, d_head 32           0.48 to 0.95 from 1000 blocks; fewer 0.90 to 1.25
  //     no split, d_head 128          0.28 to 0.97 from 257 blocks; fewer 1.14 to 1.37
  //   a context of up to T keys (decode blocks of 32 rows and more)
  //     splits in their place         T = 256 0.69 to 1.05, d_head 32 at 512 0.69 to
  //                                   1.02, d_head 128 at two splits 0.74 to 0.94;
  //                                   else up to 2.0 (one sequence, T = 1024)
  //     no split                      d_head 64 0.26 to 1.04, d_head 128 0.28 to 0.87,
  //                                   d_head 32 0.34 to 1.04 from 576 blocks (fewer 1.26)
  bool tiled = qoff == 0 && R >= 32 && !wide;
  if (tiled && ns > 1)
    tiled = empty || T <= (dh == 32 ? 512 : 256) || (dh == 128 && ns == 2);
  else if (tiled && (empty || T <= 128))
    tiled = dh == 64 ? base >= 864 || (R >= 128 && base >= 576) : base >= (dh == 32 ? 1000 : 257);
  else if (tiled)
    tiled = base >= (dh == 32 ? 576 : 256);
  return {ns, wide, tiled};
}

// Plain GEMMs (out-projection, MLP-down, noise encoder): two K groups per workgroup
// on a grid of `tiles` tiles of at most 64 x 64 with nk K steps each.  Half to one
// workgroup per CU: two groups.  Fewer: two groups where K is too short to be split
// across workgroups; in fp32 also at nk = 24, whose split does not pay either
// (out-projection, K = 768, up to 144 rows: 9.6 -> 8.8 us).  Longer K splits: in
// fp32 two groups took 1.04 to 1.34 times as long there (K = 1024 1.17, K = 2048
// 1.21, K = 3072 1.19, K = 4096 1.34 at most; 1 to 64 sequences of 2 to 8 rows).
inline bool two_groups(bool fp32, int tiles, int nk) {
  return tiles >= 128 ? tiles <= 256 : nk < 24 || (fp32 && nk == 24);
}

// MLP-up (16 bits, K columns) in 128 x 128 tiles: four wavefronts where K is long
// enough for their lighter LDS reads to pay for a longer epilogue (K = 1024, 3500 to
// 8200 rows: 0.96 to 1.01 of eight wavefronts' time).  Eight below, and always for
// QKV, whose epilogue, the KV append, is the longer one: K = 1024, 1400 to 19800 rows
// 1.05 to 1.32 times as long in four (4096 x 3072 37 -> 45 us).
inline bool mlp_up_four_waves(int tiles, int K) { return tiles >= 256 && K >= 1024 && K % 128 == 0; }

// The time of `tiles` tiles at two workgroups per CU, in fifths of a round: a
// last round of one workgroup per CU or less takes about three.
inline int tile_rounds(int tiles) {
  const int rest = tiles % 512;
  return tiles / 512 * 5 + (rest == 0 ? 0 : rest <= 256 ? 3 : 5);
}

// Plain GEMMs (16 bits, K columns) of 256 tiles of 128 x 128 and more, t160 of 160 x
// 128: rows of the four-wavefront tile to run, two workgroups per CU, or 0 for 128
// rows in eight wavefronts.  160 where they save more rounds than their tiles are
// larger: 0.66 to 0.98 of eight wavefronts' time (residual 11808 x 768, K = 3072 83 ->
// 61 us; K = 768 34 -> 27; 16896 x 1024, K = 4096 178 -> 166); at 8 fifths against
// 10, an equal sum, they took 0 to 9 % longer than 128.  128 rows in four wavefronts:
// 0.92 to 1.02 of eight on one round (K = 4096 up to 1.08), and at K = 2048 and more
// beyond; at K = 768 and 1024 on more than one round 1.00 to 1.06.
inline int plain_tile_rows(int t128, int t160, int K) {
  if (t128 < 256 || K % 128 != 0) return 0;
  if (5 * tile_rounds(t160) < 4 * tile_rounds(t128)) return 160;
  return t128 <= 512 || K > 1024 ? 128 : 0;
}

// QKV value tiles of M rows, R a sequence: by column (a lane stores runs of 4 slots)
// or by row.  By column the time depends on whether the rows fall into whole 4-slot
// blocks, which the committed length decides as well as R, and the host rule does not
// know it (asking on the device costs every launch a load: one sequence, 11.00 ->
// 11.08 ms a generate).  QKV at K = 768, k = 4, us by row against by column, contexts
// of 16 | 17:  M = 48 6.8, 7.1 | 7.1, 8.8;  192 8.0, 8.0 | 8.8, 10.1;  256 8.9, 8.9 |
// 9.8, 11.2;  384 9.3, 9.0 | 10.4, 11.3;  512 11.6, 11.0 | 12.7, 15.2 (K = 1024 at 512
// 13.5, 12.0 | 14.8, 16.1); through a page table 192 8.8, 8.8 | 9.5, 11.7;  256 9.7, 9.3
// | 10.5, 12.6.  fp32: 512 28.4, 27.6 | 29.7, 32.4.
constexpr bool value_columns(bool fp32, int M, int R) {
  return M > 512 || (!fp32 && M > 224 && R % 4 == 0);
}

}  // namespace kf
