// kf_route.h -- which attention kernel a call runs: rules on its sizes alone.
// Host code without HIP types, so that a host compiler can test the rules.
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
// Times of the 32-row kernel over the 16-row one, both masks, 8 to 4096 heads, N
// from 1 to 1000, k = 1, 2, 4, 8, against the number of 128-row workgroups:
//   d_head 128  384 and more 0.81 on average, 1.04 at most; fewer 1.05 to 1.35
//   d_head 64   3072 and more 0.91, 1.05 at most; 1024 and more at N of 80 to 255
//               likewise (self-forcing rollouts); else up to 1.35
//   d_head 32   1024 and more 0.84, 1.07 at most; fewer up to 1.13
// where a head's last workgroup is nearly whole: the rows padded to 128 a block may
// exceed those padded to 64 by 1/24 (d_head 128: 1/5).  Beyond that 1.05 to 1.26.
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
  const long long grid = BH * b32;
  const bool whole = 48 * b32 <= 25 * b16;
  bool r32;
  if (dh == 128) r32 = grid >= 384 && 10 * b32 <= 6 * b16;
  else if (dh == 64) r32 = (whole && grid >= 3072) || (2 * b32 == b16 && grid >= 1024 && N >= 80 && N < 256);
  else r32 = whole && grid >= 1024;
  return {r32, (int)prow, (int)b32};
}

}  // namespace kf
