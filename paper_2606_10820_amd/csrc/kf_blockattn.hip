// kf_blockattn.hip -- block-sparse attention of the training masks on gfx950.
//
// Appendix C.2 defines two masks over a sequence of N context tokens and k
// tokens per context position:
//   SingleForward M_S, queries and keys [context N | noise N*k]:
//     context row i sees context 0..i; noise token j of group t (t = 0..N-1)
//     sees context 0..t and tokens 0..j of its own group;
//   DoubleForward M_D, queries [Future-1 N*k | Future-2 N*k], keys
//     [context N | Future-1 N*k | Future-2 N*k]:
//     Future-1 token j of group t sees context 0..t and Future-1 tokens 0..j
//     of its group; Future-2 token j of group t sees context 0..t, all k
//     Future-1 tokens of its group and Future-2 tokens 0..j of its group.
// Every query row therefore sees at most three key intervals, one in each of
// the disjoint key regions (context, first noise block, second noise block).
// A workgroup owns 128 consecutive query rows (32 per wavefront) and walks only
// the union of their intervals, region by region, in 64-key tiles that travel
// from HBM straight into an S-stage LDS ring (buffer loads with the lds
// modifier; keys past the interval read as zero) and are shared by its four
// wavefronts.  A wavefront skips a tile that misses all of its rows and
// applies the per-element mask only on tiles that are not fully visible to
// all of them.  The work is O(|M|), not O((N + Nk)^2).
//
//   S^T = K Q^T on v_mfma_f32_32x32x16_bf16, keys as the A operand; a lane
//   ends up with one query (lane % 32) and half of the tile's keys.
//   Online softmax in fp32, base 2 with the scale folded into one FMA; the
//   running maximum is raised only when it grows by more than 2^8.
//   O^T += V^T P^T: eight of the lane's probabilities are the B operand of one
//   MFMA directly, and the A operand comes from the natural [key][d_head] value
//   tile through transposing LDS reads (ds_read_b64_tr_b16) whose row addresses
//   put keys in that same order.
//
// The same walk over the paged KV cache with the causal interval is the
// attention of a prefill (prefill_attention_kernel).
#include <limits.h>
#include <math.h>

#include <type_traits>
#include <utility>

#include "kforcing.h"
#include "kf_internal.h"
#include "kf_lds.h"
#include "kf_route.h"

namespace kf {
namespace {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));
typedef short s16x2_t __attribute__((ext_vector_type(2)));

constexpr int kKT = 64;  // keys per tile

// Visible key intervals [lo, hi) of one query row, one per key region
// (empty: lo >= hi).
struct Intervals {
  int lo[3], hi[3];
};

__device__ inline Intervals no_intervals() {
  Intervals v;
#pragma unroll
  for (int s = 0; s < 3; ++s) v.lo[s] = v.hi[s] = 0;
  return v;
}

// q / k for 0 <= q with q * k < 2^32, from km = ceil(2^32 / k) (km = 0 for
// k = 1): the rounded-up reciprocal errs by less than one in q / k there.
__device__ inline int div_k(int q, uint32_t km) {
  return km ? (int)__umulhi((uint32_t)q, km) : q;
}

__device__ inline Intervals row_intervals(int mask, int N, int k, uint32_t km, int row) {
  Intervals v = no_intervals();
  if (mask == KF_MASK_SINGLE) {
    if (row < N) {
      v.hi[0] = row + 1;
    } else {
      const int q = row - N, t = div_k(q, km), j = q - t * k;
      v.hi[0] = t + 1;
      v.lo[1] = N + t * k;
      v.hi[1] = N + t * k + j + 1;
    }
  } else {
    const int nk1 = N * k;
    const bool f2 = row >= nk1;
    const int q = f2 ? row - nk1 : row, t = div_k(q, km), j = q - t * k;
    v.hi[0] = t + 1;
    v.lo[1] = N + t * k;
    v.hi[1] = f2 ? N + (t + 1) * k : N + t * k + j + 1;
    if (f2) {
      v.lo[2] = N + nk1 + t * k;
      v.hi[2] = N + nk1 + t * k + j + 1;
    }
  }
  return v;
}

// Union [ulo, uhi) and intersection [ilo, ihi) per region of the intervals
// of query rows [a, b) (a < b <= rows).  Within each part of the query rows
// (single: context, noise; double: Future-1, Future-2) every endpoint is a
// non-decreasing function of the row and a region is either empty for all
// rows of the part or for none, so the first and last row of each part
// decide.  An empty union is [0, 0); an empty intersection has ilo > ihi.
__device__ inline void row_bounds(int mask, int N, int k, uint32_t km, int a, int b, int (&ulo)[3],
                                  int (&uhi)[3], int (&ilo)[3], int (&ihi)[3]) {
  const int split = mask == KF_MASK_SINGLE ? N : N * k;
#pragma unroll
  for (int s = 0; s < 3; ++s) {
    ulo[s] = INT_MAX;
    uhi[s] = INT_MIN;
    ilo[s] = INT_MIN;
    ihi[s] = INT_MAX;
  }
  const int pa[2] = {a, max(a, split)}, pb[2] = {min(b, split), b};
#pragma unroll
  for (int part = 0; part < 2; ++part) {
    if (pa[part] >= pb[part]) continue;
    const Intervals f = row_intervals(mask, N, k, km, pa[part]);
    const Intervals l = row_intervals(mask, N, k, km, pb[part] - 1);
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      if (f.lo[s] < f.hi[s]) {
        ulo[s] = min(ulo[s], f.lo[s]);
        uhi[s] = max(uhi[s], l.hi[s]);
        ilo[s] = max(ilo[s], l.lo[s]);
        ihi[s] = min(ihi[s], f.hi[s]);
      } else {
        ilo[s] = INT_MAX;
        ihi[s] = INT_MIN;
      }
    }
  }
#pragma unroll
  for (int s = 0; s < 3; ++s)
    if (ulo[s] >= uhi[s]) ulo[s] = uhi[s] = 0;
}

// a[s] for a runtime s in 0..2 without indexing a register array
__device__ inline int pick(const int (&a)[3], int s) { return s == 0 ? a[0] : (s == 1 ? a[1] : a[2]); }

template <int... I, typename F>
__device__ inline void static_for_impl(std::integer_sequence<int, I...>, F&& f) {
  (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ inline void static_for(F&& f) {
  static_for_impl(std::make_integer_sequence<int, N>{}, f);
}

// IEEE maximum (v_maximum3_f32): no NaN-quieting copies of the operands, and,
// unlike an instruction in inline asm, visible to the compiler, which keeps the
// distance that a read of an MFMA result needs.
__device__ inline float max2(float a, float b) { return __builtin_elementwise_maximum(a, b); }
__device__ inline float max3(float a, float b, float c) { return max2(max2(a, b), c); }
// Maximum over the two lane halves (a permlane swap: VALU, no LDS traffic).
__device__ inline float max_xor32(float x) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return max2(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Tile geometry.  A stage holds the K tile then the V tile.  K, and V of a
// training call, are [64 keys][DH] bf16 in natural layout with 16-byte chunks
// permuted within each row: logical chunk c of key row r sits at chunk
// c ^ swz(r), swz the bit reversal of the row's 256-byte line index (the 64
// LDS banks).  That makes both readers conflict-free: the K reads (16
// consecutive rows, one logical chunk: all lines differ) and the transposing V
// reads (4 consecutive rows, four adjacent chunks: neighbouring lines differ
// in the top bits).  V of a paged cache is [16 blocks][DH][4 keys] as it lies
// in its page: a lane's 4 keys of one value row are 8 bytes, 32 lanes read 256
// consecutive bytes.
template <int DH, int S_, int NW>
struct Geo {
  static constexpr int ROWB = DH * 2;           // bytes per key row
  static constexpr int TILEB = kKT * ROWB;      // bytes of one K or V tile
  static constexpr int SEGW = TILEB / 1024 / NW; // 1 KB DMA segments per wavefront per tensor
  static constexpr int S = S_;                  // pipeline stages
  static constexpr int PER = 2 * SEGW;          // DMA instructions per wavefront per tile
  static constexpr int STAGEB = 2 * TILEB;
};

template <int DH>
__device__ inline int swz(int r) {
  constexpr int NCH = DH / 8, RP = 128 / DH;  // chunks per row, rows per line
  const int m = (r / RP) % NCH;
  if constexpr (NCH == 4) return ((m & 1) << 1) | (m >> 1);
  else if constexpr (NCH == 8) return ((m & 1) << 2) | (m & 2) | (m >> 2);
  else return ((m & 1) << 3) | ((m & 2) << 1) | ((m >> 1) & 2) | (m >> 3);
}

// Scalar geometry of one work item -- a head and a QB-row query block: the
// workgroup's key ranges as a tile sequence.  Tiles run over region 0, 1, 2,
// each from its union's first key in steps of 64; tile ti lies in region
// (ti >= b1) + (ti >= b2).
struct Item {
  int bh, q0, qe, ntiles, b1, b2, lo0, dt1, dt2, hi0, de1, de2;  // query rows [q0, qe)
  __device__ int t0(int ti) const {
    return lo0 + kKT * ti + (ti >= b1 ? dt1 : 0) + (ti >= b2 ? dt2 : 0);
  }
  __device__ int end(int ti) const { return hi0 + (ti >= b1 ? de1 : 0) + (ti >= b2 ? de2 : 0); }
};

// Item t of the (head, query block) list: head t / nqb, its blocks heaviest
// (latest rows) first.  A head's rows are cut into blocks from row 0 on (prow =
// nq), or each half of them by itself (prow = nq / 2: see launch_ta).
__device__ inline Item make_item(int t, int qb, int nqb, int mask, int N, int k, uint32_t km,
                                 int nq, int prow) {
  Item it;
  it.bh = t / nqb;
  int j = nqb - 1 - (t - it.bh * nqb), r0 = 0;
  if (prow < nq && 2 * j >= nqb) {
    r0 = prow;
    j -= nqb / 2;
  }
  it.q0 = r0 + j * qb;
  it.qe = min(it.q0 + qb, r0 + prow);
  int lo[3], hi[3], ilo[3], ihi[3], nt[3];
  row_bounds(mask, N, k, km, it.q0, it.qe, lo, hi, ilo, ihi);
#pragma unroll
  for (int s = 0; s < 3; ++s) nt[s] = (hi[s] - lo[s] + kKT - 1) / kKT;
  it.ntiles = nt[0] + nt[1] + nt[2];
  it.b1 = nt[0];
  it.b2 = nt[0] + nt[1];
  it.lo0 = lo[0];
  it.dt1 = lo[1] - lo[0] - kKT * nt[0];
  it.dt2 = lo[2] - lo[1] - kKT * nt[1];
  it.hi0 = hi[0];
  it.de1 = hi[1] - hi[0];
  it.de2 = hi[2] - hi[1];
  return it;
}

// Where a workgroup's key tiles come from.  tile(t0, rows): the tile of keys
// t0 .. t0 + rows - 1, as buffer ranges that end with its last key (value
// block), so that keys past the interval read as zero.
template <int DH>
struct SeqKeys {  // K, V [ldk][DH] of one head
  static constexpr bool kPaged = false;
  const bf16 *K, *V;
  __device__ void tile(int t0, int rows, __amdgpu_buffer_rsrc_t& rk,
                       __amdgpu_buffer_rsrc_t& rv) const {
    rk = make_rsrc(K + (size_t)t0 * DH, rows * DH * 2);
    rv = make_rsrc(V + (size_t)t0 * DH, rows * DH * 2);
  }
};
template <int DH>
struct PagedKeys {  // one sequence, layer and head of the KV cache
  static constexpr bool kPaged = true;
  const bf16* kv;
  const KfKvGeom& kg;
  int seq;
  unsigned ko, vo;  // the head's keys and values within a page
  int written;      // keys that hold data: value slots past them are stale
  __device__ void tile(int t0, int rows, __amdgpu_buffer_rsrc_t& rk,
                       __amdgpu_buffer_rsrc_t& rv) const {
    static_assert(kPage % kKT == 0, "a tile lies in one page");
    const bf16* page = kv + kg.page_base(seq, t0) + (t0 % kPage) * DH;
    rk = make_rsrc(page + ko, rows * DH * 2);
    rv = make_rsrc(page + vo, (rows + kVBlk - 1) / kVBlk * (kVBlk * DH * 2));
  }
};

// The visible key intervals of a wavefront and of this lane's query row.
struct RowSets {
  int wlo[3], whi[3];  // union over the wavefront's rows
  int ilo[3], ihi[3];  // intersection over them
  int lo[3], hi[3];    // this lane's row
  int glo, ghi;        // keys inside a union that no row of the wavefront sees
};

// One work item: the unnormalised O^T and row sum of this lane's query row
// (row lane & 31 of its wavefront's 32), lane half h = lane >> 5 holding d_head
// indices 32 eg + 8 (i / 4) + 4 h + i % 4 of o[eg][i].
//
// What bounds it: per 64-key tile a wavefront issues 16 MFMAs of 32 cycles at
// d_head 64 and about 140 VALU instructions (32 of them exponentials of 8
// cycles: about 690 cycles), and on sustained launches the clock: it falls to
// 1.7-2.1 GHz under this mix.  32 query rows per wavefront rather than 16: a
// tile's K and V cross LDS once per wavefront and DMA once per workgroup, and
// half of that traffic bought 10 % (sustained: M_S at B = 16, H = 12, N = 1024,
// k = 4, d_head 64 300 -> 270 us; N = 600, k = 3, d_head 128 75 -> 60 us).
// Scores of the next tile formed under the softmax of this one (two score
// blocks, 239 registers, two wavefronts per SIMD instead of three) took 342 us;
// four wavefronts per SIMD spill (324 us); a third stage changes nothing.
template <int DH, int S, int NW, class Keys>
__device__ __forceinline__ void attend(unsigned char* smem, const Item& C, const Keys& keys,
                                       const RowSets& rs_, const bf16x8_t (&qf)[DH / 16], float c2,
                                       f32x16_t (&o)[DH / 32], float& ls) {
  using G = Geo<DH, S, NW>;
  constexpr int NC = DH / 16, NE = DH / 32;
  const int lane = threadIdx.x & 63, half = lane >> 5;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // DMA: segment w + NW i of a tile is LDS bytes [1024 (w + NW i), +1024); lane L
  // fills 16 of them, the chunk that the swizzle puts there
  uint32_t koff[G::SEGW], voff[G::SEGW];
#pragma unroll
  for (int i = 0; i < G::SEGW; ++i) {
    const int byte = (w + NW * i) * 1024 + 16 * lane;
    const int r = byte / G::ROWB, pc = (byte % G::ROWB) / 16;
    koff[i] = r * G::ROWB + ((pc ^ swz<DH>(r)) * 16);
    voff[i] = Keys::kPaged ? byte : koff[i];
  }
  // LDS read offsets of this lane within a tile.  K (MFMA A of S^T): key row
  // 32 g + lane % 32, logical chunk 2c + half.  V (MFMA A of O^T): step j takes
  // keys 16j .. 16j + 15 in the order in which the lanes hold their
  // probabilities, slots 4 r2 .. 4 r2 + 3 of half h being keys 16j + 8 r2 + 4h ..
  // + 3; value row 32 eg + lane % 32.
  uint32_t kofs[NC], vofs[Keys::kPaged ? 1 : NE][2];
#pragma unroll
  for (int c = 0; c < NC; ++c)
    kofs[c] = (lane & 31) * G::ROWB + (((2 * c + half) ^ swz<DH>(lane & 31)) * 16);
  if constexpr (Keys::kPaged) {
    vofs[0][0] = half * (DH * 8) + (lane & 31) * 8;
  } else {
#pragma unroll
    for (int r2 = 0; r2 < 2; ++r2) {
      const int r = 8 * r2 + 4 * half + ((lane & 15) >> 2);
#pragma unroll
      for (int eg = 0; eg < NE; ++eg)
        vofs[eg][r2] = r * G::ROWB + (lane & 1) * 8 +
                       (((4 * eg + 2 * ((lane >> 4) & 1) + ((lane & 3) >> 1)) ^ swz<DH>(r)) * 16);
    }
  }
  const bf16x2_t one2 = {1.f, 1.f};

  // Tiles past the last one load nothing, so every wavefront issues the same
  // number of loads per tile.
  auto issue = [&](int ti, int stage) {
    const bool live = ti < C.ntiles;
    const int t0 = live ? C.t0(ti) : 0;
    const int rows = live ? min(C.end(ti) - t0, kKT) : 0;
    __amdgpu_buffer_rsrc_t rk, rv;
    keys.tile(t0, rows, rk, rv);
    unsigned char* st = smem + stage * G::STAGEB;
#pragma unroll
    for (int i = 0; i < G::SEGW; ++i) dma16(rk, koff[i], 0, st + (w + NW * i) * 1024);
#pragma unroll
    for (int i = 0; i < G::SEGW; ++i) dma16(rv, voff[i], 0, st + G::TILEB + (w + NW * i) * 1024);
  };
#pragma unroll
  for (int j = 0; j < S - 1; ++j) issue(j, j);

  // running max m (log2 units); o = the unnormalised O^T; ls = this lane's part
  // of the row sum: over the bf16 probabilities that o uses, or, in a model's step
  // over the cache, over the fp32 ones as in the other kernels of block attention
  float m_run = -INFINITY;
  ls = 0.f;
#pragma unroll
  for (int eg = 0; eg < NE; ++eg)
#pragma unroll
    for (int i = 0; i < 16; ++i) o[eg][i] = 0.f;

  // per-region values of the current tile's region, updated where a region starts
  int cwlo = 0, cwhi = 0, cilo = 0, cihi = 0, rlo = 0, width = 0, stage = 0;
  for (int ti = 0; ti < C.ntiles; ++ti) {
    vm_wait<(S - 2) * G::PER>();  // this wavefront's part of tile ti has landed
    __builtin_amdgcn_s_barrier();  // ... and everyone's; stage (ti - 1) % S is free
    issue(ti + S - 1, stage == 0 ? S - 1 : stage - 1);
    if (ti == 0 || ti == C.b1 || ti == C.b2) {
      const int rs = (ti >= C.b1) + (ti >= C.b2);
      cwlo = pick(rs_.wlo, rs);
      cwhi = pick(rs_.whi, rs);
      cilo = pick(rs_.ilo, rs);
      cihi = pick(rs_.ihi, rs);
      rlo = pick(rs_.lo, rs);
      width = max(pick(rs_.hi, rs) - rlo, 0);
    }
    const int t0 = C.t0(ti);
    const uint32_t kb = lds_addr(smem + stage * G::STAGEB), vb = kb + G::TILEB;
    stage = stage + 1 == S ? 0 : stage + 1;
    if (t0 >= cwhi || t0 + kKT <= cwlo || (t0 >= rs_.glo && t0 + kKT <= rs_.ghi))
      continue;  // no row of this wavefront sees the tile
    // S^T = K Q^T: lane holds query lane % 32, keys 32g + 8 (i / 4) + 4 half + i % 4
    u32x4 a[2][NC];
    static_for<2>([&](auto g) {
#pragma unroll
      for (int c = 0; c < NC; ++c) a[g][c] = ds_read16_off<g * 32 * G::ROWB>(kb + kofs[c]);
    });
    f32x16_t sc[2];
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int i = 0; i < 16; ++i) sc[g][i] = 0.f;
    lgkm_wait0();
#pragma unroll
    for (int g = 0; g < 2; ++g)
#pragma unroll
      for (int c = 0; c < NC; ++c) pin(a[g][c]);
#pragma unroll
    for (int c = 0; c < NC; ++c)
#pragma unroll
      for (int g = 0; g < 2; ++g)
        sc[g] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8_t, a[g][c]), qf[c],
                                                        sc[g], 0, 0, 0);
    // value fragments of all 64 keys, in flight during the softmax
    u32x2 va[4][NE][2];
    static_for<4>([&](auto j) {
      static_for<NE>([&](auto eg) {
        static_for<2>([&](auto r2) {
          if constexpr (Keys::kPaged)
            va[j][eg][r2] = ds_read8_off<(4 * j + 2 * r2) * DH * 8 + eg * 256>(vb + vofs[0][0]);
          else
            va[j][eg][r2] = ds_read_tr16_off<j * 16 * G::ROWB>(vb + vofs[eg][r2]);
        });
      });
    });
    // mask: a tile serves its own region's interval only (its last keys may
    // spill into the next region, which has tiles of its own)
    if (!(t0 >= cilo && t0 + kKT <= cihi)) {
      const int base = t0 + 4 * half - rlo;
#pragma unroll
      for (int g = 0; g < 2; ++g)
#pragma unroll
        for (int i = 0; i < 16; ++i)
          sc[g][i] = (unsigned)(base + 32 * g + 8 * (i >> 2) + (i & 3)) < (unsigned)width ? sc[g][i] : -INFINITY;
    }
    float mx = max2(sc[0][0], sc[1][0]);
#pragma unroll
    for (int i = 1; i < 16; ++i) mx = max3(mx, sc[0][i], sc[1][i]);
    mx = max_xor32(mx) * c2;
    // rescale only when the row maximum grows by more than 2^8: probabilities
    // stay below 256, and the same reference serves numerator and denominator
    const bool grow = mx > m_run + 8.f;
    if (__builtin_amdgcn_ballot_w64(grow)) {
      const float mn = grow ? mx : m_run;
      const float alpha = __builtin_amdgcn_exp2f(m_run - mn);
      ls *= alpha;
#pragma unroll
      for (int eg = 0; eg < NE; ++eg)
#pragma unroll
        for (int i = 0; i < 16; ++i) o[eg][i] *= alpha;
      m_run = mn;
    }
    const float mref = m_run == -INFINITY ? 0.f : m_run;
    bf16x8_t pf[4];
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 8; r += 2) {
        const f32x2_t e = {
            __builtin_amdgcn_exp2f(__builtin_fmaf(sc[j >> 1][8 * (j & 1) + r], c2, -mref)),
            __builtin_amdgcn_exp2f(__builtin_fmaf(sc[j >> 1][8 * (j & 1) + r + 1], c2, -mref))};
        const bf16x2_t h = __builtin_convertvector(e, bf16x2_t);
        pf[j][r] = h[0];
        pf[j][r + 1] = h[1];
        if constexpr (Keys::kPaged)
          ls += e[0] + e[1];
        else
          ls = __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(s16x2_t, h),
                                               __builtin_bit_cast(s16x2_t, one2), ls, false);
      }
    // O^T += V^T P^T, 16 keys a step
    lgkm_wait0();
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int eg = 0; eg < NE; ++eg) {
        pin(va[j][eg][0]);
        pin(va[j][eg][1]);
        u32x4 x = {va[j][eg][0].x, va[j][eg][0].y, va[j][eg][1].x, va[j][eg][1].y};
        bf16x8_t v = __builtin_bit_cast(bf16x8_t, x);
        if constexpr (Keys::kPaged) {
          if (t0 + kKT > keys.written) {  // 0 * a stale NaN would not be 0
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (t0 + 16 * j + 8 * (e >> 2) + 4 * half + (e & 3) >= keys.written) v[e] = (bf16)0.f;
          }
        }
        o[eg] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(v, pf[j], o[eg], 0, 0, 0);
      }
  }
  vm_wait<0>();  // loads issued for tiles past the last one
  const auto both = __builtin_amdgcn_permlane32_swap(__float_as_uint(ls), __float_as_uint(ls), false, false);
  ls = __uint_as_float(both[0]) + __uint_as_float(both[1]);
}

// This lane's normalised output row (d_head DH), inv = 1 / its row sum: the halves
// exchange 4-value pieces so that each stores 16 bytes.
template <int DH>
__device__ __forceinline__ void store_row(bf16* orow, bool valid, const f32x16_t (&o)[DH / 32],
                                          float inv) {
  const int half = (threadIdx.x & 63) >> 5;
#pragma unroll
  for (int eg = 0; eg < DH / 32; ++eg)
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      uint32_t lo[2], hi[2];  // this half's pieces of the 8-value groups 2p and 2p + 1
#pragma unroll
      for (int q = 0; q < 2; ++q) {
        const f32x2_t x = {o[eg][8 * p + 2 * q] * inv, o[eg][8 * p + 2 * q + 1] * inv};
        const f32x2_t y = {o[eg][8 * p + 4 + 2 * q] * inv, o[eg][8 * p + 5 + 2 * q] * inv};
        lo[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector(x, bf16x2_t));
        hi[q] = __builtin_bit_cast(uint32_t, __builtin_convertvector(y, bf16x2_t));
      }
      const auto s0 = __builtin_amdgcn_permlane32_swap(lo[0], hi[0], false, false);
      const auto s1 = __builtin_amdgcn_permlane32_swap(lo[1], hi[1], false, false);
      if (valid)
        *reinterpret_cast<uint4*>(orow + 32 * eg + 16 * p + 8 * half) =
            make_uint4(s0[0], s1[0], s0[1], s1[1]);
    }
}

template <int DH, int S, int NW>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(DH <= 64 ? 3 : 2)))
    training_attention_kernel(const bf16* __restrict__ Q, const bf16* __restrict__ K,
                              const bf16* __restrict__ V, bf16* __restrict__ O, int mask, int N,
                              int k, uint32_t km, int nq, int prow, int ldk, int H, int BH,
                              int o_inter, float c2) {
  using G = Geo<DH, S, NW>;
  constexpr int NC = DH / 16, QB = 32 * NW;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[S * G::STAGEB];

  // Work order.  Workgroups are dealt to the 8 XCDs round-robin, so XCD x runs
  // workgroups x, x + 8, ...  Each XCD is given a contiguous run of the item
  // list (whole heads, one after another), so that the query blocks of one
  // head share its keys and values through that XCD's L2.
  const int nqb = (prow + QB - 1) / QB * (prow < nq ? 2 : 1), total = BH * nqb;
  const int x8 = blockIdx.x & 7, j8 = blockIdx.x >> 3;
  const Item C = make_item(x8 * (total >> 3) + min(x8, total & 7) + j8, QB, nqb, mask, N, k, km, nq, prow);
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);

  // this lane's query row, its Q fragment (MFMA B operand: d_head 16c + 8 half ..
  // + 7) and intervals
  const int wrow = C.q0 + 32 * w, row = wrow + (lane & 31);
  const bool valid = row < C.qe;
  bf16x8_t qf[NC];
  {
    const bf16* qrow = Q + ((size_t)C.bh * nq + (valid ? row : 0)) * DH + 8 * (lane >> 5);
#pragma unroll
    for (int c = 0; c < NC; ++c)
      qf[c] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(qrow + 16 * c));
  }
  RowSets rs = {{0, 0, 0}, {0, 0, 0}, {1, 1, 1}, {0, 0, 0}, {0, 0, 0}, {0, 0, 0}, 0, 0};
  if (wrow < C.qe)
    row_bounds(mask, N, k, km, wrow, min(wrow + 32, C.qe), rs.wlo, rs.whi, rs.ilo, rs.ihi);
  const int wlast = min(wrow + 32, C.qe) - 1;
  if (mask == KF_MASK_DOUBLE && wrow < N * k && wlast >= N * k) {
    // Rows of both parts: the last groups' Future-1 rows and the first groups'
    // Future-2 rows, whose union in the Future-1 keys is nearly all of them.
    // Without the gap this wavefront multiplied N k / 64 tiles that none of its
    // rows sees (M_D at d_head 32, 256 heads, N = 400, k = 1: 39 -> 36 us).
    rs.glo = row_intervals(mask, N, k, km, wlast).hi[1];
    rs.ghi = row_intervals(mask, N, k, km, wrow).lo[1];
  }
  if (valid) {
    const Intervals iv = row_intervals(mask, N, k, km, row);
#pragma unroll
    for (int s = 0; s < 3; ++s) {
      rs.lo[s] = iv.lo[s];
      rs.hi[s] = iv.hi[s];
    }
  }
  f32x16_t o[DH / 32];
  float ls;
  const SeqKeys<DH> keys{K + (size_t)C.bh * ldk * DH, V + (size_t)C.bh * ldk * DH};
  attend<DH, S, NW>(smem, C, keys, rs, qf, c2, o, ls);  // ls >= 1 for a valid row: its maximum's term

  // O: [B][H][nq][DH], or [B][nq][H][DH] (rows of a residual stream) with o_inter
  const int ob = C.bh / H, oh = C.bh - ob * H;
  store_row<DH>(O + (o_inter ? (((size_t)ob * nq + row) * H + oh) * DH : ((size_t)C.bh * nq + row) * DH),
                valid, o, __builtin_amdgcn_rcpf(ls));
}

// Attention of a step with many rows per sequence (a prefill) over the paged KV
// cache: the rows of a step sit at cache slots C + i and see slots [0, C + i].
// The same walk as above with one key region, the tiles read from the pages.
// The decode kernel (16 query rows a workgroup, fragments straight from
// memory) reads each key of a prefill R / 16 times: per layer at d_head 64, 12
// heads, B = 16, R = 512 it took 100 us where this takes 18; B = 64, R = 128
// 37 -> 9.
template <int DH, int S, int NW>
__global__ void __launch_bounds__(64 * NW) __attribute__((amdgpu_waves_per_eu(DH <= 64 ? 3 : 2)))
    prefill_attention_kernel(const bf16* __restrict__ Q, const bf16* __restrict__ kv,
                             bf16* __restrict__ O, const KfDevState* st, KfStepGeom g, KfKvGeom kg,
                             int layer, float c2) {
  using G = Geo<DH, S, NW>;
  constexpr int NC = DH / 16, QB = 32 * NW;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[S * G::STAGEB];
  const int H = kg.H, nqb = (g.R + QB - 1) / QB, total = g.B * H * nqb;
  const int x8 = blockIdx.x & 7, j8 = blockIdx.x >> 3;
  const int t = x8 * (total >> 3) + min(x8, total & 7) + j8;
  const int bh = t / nqb, b = bh / H, h = bh - b * H;
  const int ctx = __builtin_amdgcn_readfirstlane(g.ctx(st, b));
  const int q0 = (nqb - 1 - (t - bh * nqb)) * QB;  // heaviest rows first
  const int keys_end = ctx + min(q0 + QB, g.R);
  const int ntiles = (keys_end + kKT - 1) / kKT;
  const Item C{bh, q0, 0, ntiles, ntiles, ntiles, 0, 0, 0, keys_end, 0, 0};
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wrow = q0 + 32 * w, row = wrow + (lane & 31);
  const bool valid = row < g.R;
  const size_t at = ((size_t)b * g.R + (valid ? row : 0)) * (H * DH) + h * DH;
  bf16x8_t qf[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c)
    qf[c] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(Q + at + 8 * (lane >> 5) + 16 * c));
  RowSets rs = {{0, 0, 0}, {0, 0, 0}, {1, 1, 1}, {0, 0, 0}, {0, 0, 0}, {0, 0, 0}, 0, 0};
  if (wrow < g.R) {
    rs.whi[0] = ctx + min(wrow + 32, g.R);
    rs.ilo[0] = 0;
    rs.ihi[0] = ctx + wrow + 1;
  }
  if (valid) rs.hi[0] = ctx + row + 1;
  f32x16_t o[DH / 32];
  float ls;
  const PagedKeys<DH> keys{kv, kg, __builtin_amdgcn_readfirstlane(g.slot(b)),
                           kg.head_off(layer, 0, h), kg.head_off(layer, 1, h), ctx + g.R};
  attend<DH, S, NW>(smem, C, keys, rs, qf, c2, o, ls);
  store_row<DH>(O + at, valid, o, 1.0f / ls);
}

// The same mask with 16 query rows per wavefront (64 per workgroup) on 16x16x32
// MFMA, one query per lane of a 16-lane group: twice the workgroups and half the
// serial work of each, which is what bounds a grid of a few workgroups per CU
// (d_head 64: B = 2, H = 8, N = 215, k = 8, M_D 39 -> 32 us; B = 22, H = 16, N =
// 495, k = 1, M_D 95 -> 86; d_head 32: B = 1, H = 12, N = 408, k = 2, M_D 22 -> 15).
//
// Its tiles' swizzle: 8 consecutive rows of two adjacent chunks (a transposing
// read of 16 lanes) and 16 consecutive rows of one chunk touch distinct banks.
template <int DH>
__device__ inline int swz16(int r) {
  constexpr int NCH = DH / 8, RP = 128 / DH;
  const int m = (r / RP) % NCH;
  return ((m & (NCH / 2 - 1)) << 1) | (m / (NCH / 2));
}
__device__ inline float max_xor16(float x) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return max2(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

template <int DH, int S>
__global__ void __launch_bounds__(256)
    training_attention16_kernel(const bf16* __restrict__ Q, const bf16* __restrict__ K,
                                const bf16* __restrict__ V, bf16* __restrict__ O, int mask, int N,
                                int k, uint32_t km, int nq, int ldk, int H, int BH, int o_inter,
                                float c2) {
  using G = Geo<DH, S, 4>;
  constexpr int QB = 64, NDC = DH / 32, NDB = DH / 16;
  __shared__ __attribute__((aligned(1024))) unsigned char smem[S * G::STAGEB];

  // Work order.  Workgroups are dealt to the 8 XCDs round-robin, so XCD x runs
  // workgroups x, x + 8, ...  Each XCD is given a contiguous run of the item
  // list (whole heads, one after another), so that the query blocks of one
  // head share its keys and values through that XCD's L2.
  const int nqb = (nq + QB - 1) / QB, total = BH * nqb;
  const int x8 = blockIdx.x & 7, j8 = blockIdx.x >> 3;
  const Item C = make_item(x8 * (total >> 3) + min(x8, total & 7) + j8, QB, nqb, mask, N, k, km, nq, nq);
  const int tid = threadIdx.x, lane = tid & 63, gq = lane >> 4, lq = lane & 15;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);

  // DMA: segment w + 4i of a tile is LDS bytes [1024 (w + 4i), +1024); lane L
  // fills 16 of them, the chunk that the swizzle puts there
  uint32_t voff[G::SEGW];
#pragma unroll
  for (int i = 0; i < G::SEGW; ++i) {
    const int byte = (w + 4 * i) * 1024 + 16 * lane;
    const int r = byte / G::ROWB, pc = (byte % G::ROWB) / 16;
    voff[i] = r * G::ROWB + ((pc ^ swz16<DH>(r)) * 16);
  }
  // LDS read offsets of this lane within a tile.  K (MFMA A of S^T): key row
  // 16g + lq, logical chunk 4c + gq.  V (transposing reads, MFMA A of O^T):
  // key row 32c + 4gq + lq/4 (+16 for the upper half of the k-slots), d_head
  // 16db + 4 (lq % 4), i.e. logical chunk 2db + (lq % 4) / 2, byte 8 (lq % 2).
  uint32_t kofs[NDC], vofs[NDB];
#pragma unroll
  for (int c = 0; c < NDC; ++c) kofs[c] = lq * G::ROWB + (((4 * c + gq) ^ swz16<DH>(lq)) * 16);
  {
    const int r = 4 * gq + (lq >> 2);
#pragma unroll
    for (int db = 0; db < NDB; ++db)
      vofs[db] = r * G::ROWB + (((2 * db + ((lq & 3) >> 1)) ^ swz16<DH>(r)) * 16) + (lq & 1) * 8;
  }
  const bf16x8_t ones = {1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f, 1.f};

  // Tiles past the last one load nothing, so every wavefront issues the same
  // number of loads per tile.
  auto issue = [&](int ti, int stage) {
    const bool live = ti < C.ntiles;
    const int t0 = live ? C.t0(ti) : 0;
    const int rows = live ? min(C.end(ti) - t0, kKT) : 0;
    const size_t off = ((size_t)C.bh * ldk + t0) * DH;
    const __amdgpu_buffer_rsrc_t rk = make_rsrc(K + off, rows * G::ROWB);
    const __amdgpu_buffer_rsrc_t rv = make_rsrc(V + off, rows * G::ROWB);
    unsigned char* st = smem + stage * G::STAGEB;
#pragma unroll
    for (int i = 0; i < G::SEGW; ++i) dma16(rk, voff[i], 0, st + (w + 4 * i) * 1024);
#pragma unroll
    for (int i = 0; i < G::SEGW; ++i) dma16(rv, voff[i], 0, st + G::TILEB + (w + 4 * i) * 1024);
  };
#pragma unroll
  for (int j = 0; j < S - 1; ++j) issue(j, j);

  // this lane's query row, its Q fragment (MFMA B operand: d_head 32c + 8gq..+7)
  // and intervals; the wavefront's union (wlo, whi) and intersection (ilo, ihi)
  // of its 16 rows' intervals per region
  const int row = C.q0 + 16 * w + lq;
  const bool valid = row < nq;
  bf16x8_t qf[NDC];
  {
    const bf16* qrow = Q + ((size_t)C.bh * nq + (valid ? row : 0)) * DH + 8 * gq;
#pragma unroll
    for (int c = 0; c < NDC; ++c)
      qf[c] = valid ? __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const uint4*>(qrow + 32 * c))
                    : bf16x8_t{};
  }
  int wlo[3] = {0, 0, 0}, whi[3] = {0, 0, 0}, ilo[3] = {1, 1, 1}, ihi[3] = {0, 0, 0};
  if (C.q0 + 16 * w < nq)
    row_bounds(mask, N, k, km, C.q0 + 16 * w, min(C.q0 + 16 * w + 16, nq), wlo, whi, ilo, ihi);
  const Intervals iv = valid ? row_intervals(mask, N, k, km, row) : no_intervals();
  // running max m (log2 units); o = the unnormalised O^T; ls = the row sums of
  // P, formed by the MFMA against a block of ones (each element of ls is the
  // sum of this lane's query row over the bf16 probabilities that o uses)
  float m_run = -INFINITY;
  f32x4_t o[NDB], ls = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int i = 0; i < NDB; ++i) o[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // per-region values of the current tile's region, updated where a region starts
  int cwlo = 0, cwhi = 0, cilo = 0, cihi = 0, rlo = 0, rhi = 0;
  for (int ti = 0; ti < C.ntiles; ++ti) {
    vm_wait<(S - 2) * G::PER>();  // this wavefront's part of tile ti has landed
    __builtin_amdgcn_s_barrier();  // ... and everyone's; stage (ti - 1) % S is free
    issue(ti + S - 1, (ti + S - 1) % S);
    if (ti == 0 || ti == C.b1 || ti == C.b2) {
      const int rs = (ti >= C.b1) + (ti >= C.b2);
      cwlo = pick(wlo, rs);
      cwhi = pick(whi, rs);
      cilo = pick(ilo, rs);
      cihi = pick(ihi, rs);
      rlo = pick(iv.lo, rs);
      rhi = pick(iv.hi, rs);
    }
    const int t0 = C.t0(ti);
    if (t0 < cwhi && t0 + kKT > cwlo) {  // some row of this wavefront sees the tile
      const uint32_t kb = lds_addr(smem + (ti % S) * G::STAGEB), vb = kb + G::TILEB;
      // S^T = K Q^T: lane holds query lq, keys 16g + 4gq + r
      u32x4 a[4][NDC];
      static_for<4>([&](auto gg) {
#pragma unroll
        for (int c = 0; c < NDC; ++c) a[gg][c] = ds_read16_off<gg * 16 * G::ROWB>(kb + kofs[c]);
      });
      lgkm_wait0();
      // value fragments of all 64 keys, in flight during the S MFMAs and the softmax
      u32x2 va[2][NDB], vc[2][NDB];
      static_for<2>([&](auto c) {
        static_for<NDB>([&](auto db) {
          va[c][db] = ds_read_tr16_off<c * 32 * G::ROWB>(vb + vofs[db]);
          vc[c][db] = ds_read_tr16_off<c * 32 * G::ROWB + 16 * G::ROWB>(vb + vofs[db]);
        });
      });
      f32x4_t sc[4];
#pragma unroll
      for (int gg = 0; gg < 4; ++gg) {
        sc[gg] = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < NDC; ++c) {
          pin(a[gg][c]);
          sc[gg] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a[gg][c]),
                                                           qf[c], sc[gg], 0, 0, 0);
        }
      }
      // mask: a tile serves its own region's interval only (its last keys may
      // spill into the next region, which has tiles of its own)
      if (!(t0 >= cilo && t0 + kKT <= cihi)) {
        const unsigned width = rhi > rlo ? (unsigned)(rhi - rlo) : 0u;
        const int base = t0 + 4 * gq - rlo;
#pragma unroll
        for (int gg = 0; gg < 4; ++gg)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if ((unsigned)(base + 16 * gg + r) >= width) sc[gg][r] = -INFINITY;
      }
      float mx = max3(max3(sc[0][0], sc[0][1], sc[0][2]), max3(sc[0][3], sc[1][0], sc[1][1]),
                      max3(sc[1][2], sc[1][3], sc[2][0]));
      mx = max3(mx, max3(sc[2][1], sc[2][2], sc[2][3]), max3(sc[3][0], sc[3][1], sc[3][2]));
      mx = max3(mx, sc[3][3], sc[3][3]);
      mx = max_xor32(max_xor16(mx)) * c2;
      // rescale only when the row maximum grows by more than 2^8: probabilities
      // stay below 256, and the same reference serves numerator and denominator
      const bool grow = mx > m_run + 8.f;
      if (__builtin_amdgcn_ballot_w64(grow)) {
        const float mn = grow ? mx : m_run;
        const float alpha = __builtin_amdgcn_exp2f(m_run - mn);
        ls *= alpha;
#pragma unroll
        for (int db = 0; db < NDB; ++db) o[db] *= alpha;
        m_run = mn;
      }
      const float mref = m_run == -INFINITY ? 0.f : m_run;
      bf16x8_t pf[2];
#pragma unroll
      for (int gg = 0; gg < 4; ++gg)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          pf[gg >> 1][4 * (gg & 1) + r] =
              (bf16)__builtin_amdgcn_exp2f(__builtin_fmaf(sc[gg][r], c2, -mref));
      ls = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[0], ls, 0, 0, 0);
      ls = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[1], ls, 0, 0, 0);
      // O^T += V^T P^T, keys 0..31 then 32..63
      lgkm_wait0();
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int db = 0; db < NDB; ++db) {
          pin(va[c][db]);
          pin(vc[c][db]);
          const u32x4 x = {va[c][db].x, va[c][db].y, vc[c][db].x, vc[c][db].y};
          o[db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, x), pf[c],
                                                          o[db], 0, 0, 0);
        }
    }
  }
  vm_wait<0>();  // loads issued for tiles past the last one

  // lane: query lq, d_head 16db + 4gq + r
  if (valid) {
    const float inv = __builtin_amdgcn_rcpf(ls[0]);  // ls >= 1: the row maximum's term
    // O: [B][H][nq][DH], or [B][nq][H][DH] (rows of a residual stream) with o_inter
    const int ob = C.bh / H, oh = C.bh - ob * H;
    bf16* orow = O + (o_inter ? (((size_t)ob * nq + row) * H + oh) * DH
                              : ((size_t)C.bh * nq + row) * DH) + 4 * gq;
#pragma unroll
    for (int db = 0; db < NDB; ++db) {
      const f32x2_t lo = {o[db][0] * inv, o[db][1] * inv}, hi = {o[db][2] * inv, o[db][3] * inv};
      *reinterpret_cast<uint2*>(orow + 16 * db) =
          make_uint2(__builtin_bit_cast(uint32_t, __builtin_convertvector(lo, bf16x2_t)),
                     __builtin_bit_cast(uint32_t, __builtin_convertvector(hi, bf16x2_t)));
    }
  }
}

}  // namespace

int training_attention_rows(int mask, int N, int k) {
  return mask == KF_MASK_SINGLE ? N + N * k : 2 * N * k;
}
int training_attention_keys(int mask, int N, int k) {
  return mask == KF_MASK_SINGLE ? N + N * k : N + 2 * N * k;
}

namespace {

// Four wavefronts per workgroup: 128 query rows share each tile's transfer; two
// (64 rows) measured slower or equal on large grids (OWT-shaped M_S, B = 16: 307
// us against 270).  16 rows per wavefront where training_route says so.
template <int DH, int S>
hipError_t launch_ta(int mask, int B, int H, int N, int k, const bf16* Q, const bf16* K,
                     const bf16* V, int ldk, bf16* O, int o_inter, float scale, hipStream_t s) {
  constexpr int NW = 4;
  const int nq = training_attention_rows(mask, N, k);
  const int BH = B * H;
  const float c2 = scale * 1.4426950408889634f;  // scale * log2(e)
  // q / k in the kernel by the rounded-up reciprocal: exact while q * k < 2^32
  if ((long long)nq * (k > 1 ? k : 1) >= (1LL << 32)) return hipErrorInvalidValue;
  const uint32_t km = k > 1 ? (uint32_t)(((1ULL << 32) + k - 1) / k) : 0u;
  const TrainingRoute r = training_route(DH, BH, mask == KF_MASK_DOUBLE, N, k, nq);
  if (!r.rows32) {
    launch(training_attention16_kernel<DH, S>, dim3((unsigned)((long long)BH * ((nq + 63) / 64))),
           dim3(256), 0, s, Q, K, V, O, mask, N, k, km, nq, ldk, H, BH, o_inter, c2);
    return hipGetLastError();
  }
  launch(training_attention_kernel<DH, S, NW>, dim3((unsigned)((long long)BH * r.blocks32)),
         dim3(64 * NW), 0, s, Q, K, V, O, mask, N, k, km, nq, r.prow, ldk, H, BH, o_inter, c2);
  return hipGetLastError();
}

template <int DH, int S, int NW>
hipError_t launch_pa(const bf16* Q, const bf16* kv, bf16* O, const KfDevState* st,
                     const KfStepGeom& g, const KfKvGeom& kg, int layer, float scale, hipStream_t s) {
  const dim3 grid((unsigned)(g.B * kg.H * ((g.R + 32 * NW - 1) / (32 * NW))));
  launch((prefill_attention_kernel<DH, S, NW>), grid, dim3(64 * NW), 0, s, Q, kv, O, st, g, kg,
         layer, scale * 1.4426950408889634f);
  return hipGetLastError();
}

hipError_t launch_ta_dh(int mask, int B, int H, int N, int k, int dh, const bf16* Q, const bf16* K,
                        const bf16* V, int ldk, bf16* O, int o_inter, float scale, hipStream_t s) {
  switch (dh) {
    case 32: return launch_ta<32, 3>(mask, B, H, N, k, Q, K, V, ldk, O, o_inter, scale, s);
    case 64: return launch_ta<64, 2>(mask, B, H, N, k, Q, K, V, ldk, O, o_inter, scale, s);
    case 128: return launch_ta<128, 2>(mask, B, H, N, k, Q, K, V, ldk, O, o_inter, scale, s);
    default: return hipErrorInvalidValue;
  }
}

}  // namespace

hipError_t launch_training_attention(int mask, int B, int H, int N, int k, int dh, const bf16* Q,
                                     const bf16* K, const bf16* V, bf16* O, float scale,
                                     hipStream_t s) {
  return launch_ta_dh(mask, B, H, N, k, dh, Q, K, V, training_attention_keys(mask, N, k), O, 0,
                      scale, s);
}

hipError_t launch_prefill_attention(const bf16* Q, const bf16* kv, bf16* O, const KfDevState* st,
                                    const KfStepGeom& g, const KfKvGeom& kg, int layer,
                                    float scale, hipStream_t s) {
  switch (kg.dh) {
    case 32: return launch_pa<32, 3, 4>(Q, kv, O, st, g, kg, layer, scale, s);
    case 64: return launch_pa<64, 2, 4>(Q, kv, O, st, g, kg, layer, scale, s);
    // two wavefronts: with four the d_head 128 kernel spills 12 registers (B =
    // 16, R = 512, 6 heads: 33 us a layer against 37; never slower)
    case 128: return launch_pa<128, 2, 2>(Q, kv, O, st, g, kg, layer, scale, s);
    default: return hipErrorInvalidValue;
  }
}

hipError_t launch_training_attention_seq(int mask, int B, int H, int N, int k, int dh, const bf16* Q,
                                         const bf16* K, const bf16* V, int ldk, bf16* O,
                                         float scale, hipStream_t s) {
  return launch_ta_dh(mask, B, H, N, k, dh, Q, K, V, ldk, O, 1, scale, s);
}

}  // namespace kf
