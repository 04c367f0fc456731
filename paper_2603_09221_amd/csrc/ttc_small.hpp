// The d = 16 shape of the solver: four problems per wavefront.
//
// At d = 16 a problem fills a quarter of a wavefront, and the dense solves (one pivot after the other,
// each a reduction and a broadcast) are most of the instructions.  This kernel gives a workgroup of one
// wavefront four problems at a time: the products are formed problem by problem on the matrix cores
// exactly as in the larger shapes (Z-land pair in LDS, constant row blocks in registers), and the dense
// solves of the four problems run side by side, lane 16q + r owning row r of problem q's augmented
// [M | RHS] in registers.  The method is that of solve_kernel: reverse symplectic steps (Thm 3.3,
// App. C "Kernel Fusion") in groups, a pivoted solve re-basing the pair after each group (Alg. 4's
// P = Y1^{-1} Y2), the last factor with Q_0 = 0, K_0 = -R^{-1} B^T A^{-T} P_0 (Thm A.4).
#pragma once
#include "ttc_common.hpp"

namespace ttc {

// max of an unsigned key over each row of 16 lanes; every lane of the row gets it (DPP only)
__device__ __forceinline__ uint32_t row16_max_u32(uint32_t x) {
  auto mx = [](uint32_t a, uint32_t b) { return a > b ? a : b; };
  x = mx(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0xB1, 0xF, 0xF, false));   // quad_perm [1,0,3,2]
  x = mx(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x4E, 0xF, 0xF, false));   // quad_perm [2,3,0,1]
  x = mx(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x141, 0xF, 0xF, false));  // row_half_mirror
  x = mx(x, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, 0x140, 0xF, 0xF, false));  // row_mirror
  return x;
}

#ifndef TTC_PIVOT_THRESHOLD
#define TTC_PIVOT_THRESHOLD 0.25f  // a diagonal entry this close to the column's largest is taken as the pivot
#endif
// Dense solves M X = RHS of the four 16 x 32 augmented arrays Wm[q] = [M | RHS] (row r at
// Wm[q] + r*PITCH), all at once: Gauss-Jordan with partial pivoting, a lane holding one row.  The pivot
// of a column is found by a 16-lane DPP max of a packed key (|value| with the row index in the low
// mantissa bits), the pivot row is broadcast with ds_bpermute, every other row of that problem is
// eliminated.  Rows never move; the row that was the pivot of column c ends up as row c of X, written
// to the right half.  The search is threshold pivoting: row c itself is preferred when it is still free and its
// entry is at least TTC_PIVOT_THRESHOLD times the column's largest (element growth stays bounded by 1 + 1/threshold
// per step instead of 2); when that holds for all four problems of the wavefront, the pivot row is known at compile
// time and is broadcast by DPP (row_newbcast) instead of going through the LDS crossbar, which is what bounds this
// function otherwise.  PIVOT = false always takes the diagonal (symmetric positive definite M).
// Returns, per lane, whether its problem broke down (zero / non-finite / non-positive pivot).
template <bool PIVOT>
__device__ __forceinline__ int solve_rows16(float* Wq, int lane) {
  using C = Cfg<16>;
  const int r = lane & 15;
  float a[32];
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    const floatx4 t = *reinterpret_cast<const floatx4*>(Wq + r * C::PITCH + 4 * k);
    a[4 * k + 0] = t[0]; a[4 * k + 1] = t[1]; a[4 * k + 2] = t[2]; a[4 * k + 3] = t[3];
  }
  __syncthreads();  // every row is in registers; the right half may be overwritten below
  bool act = true;
  int myj = 0;
  float mypiv = 1.f;
  int bad = 0;
  static_for<0, 16>([&](auto J) {
    constexpr int j = decltype(J)::value;
    int pr;
    bool diagonal = !PIVOT;  // the pivot row is lane j of every row of 16 lanes
    if constexpr (PIVOT) {
      uint32_t key = (__float_as_uint(a[j]) & 0x7FFFFF80u) | (uint32_t)(127 - r);
      key = act ? key : 0u;
      // Threshold pivoting: row j itself is taken when it is still free and its entry is within a factor of
      // TTC_PIVOT_THRESHOLD of the column's largest; when that holds for all of the wavefront's problems the
      // pivot row is known at compile time and travels by DPP instead of the LDS crossbar.
      const uint32_t own = (uint32_t)__builtin_amdgcn_mov_dpp((int)key, 0x150 + j, 0xF, 0xF, true);  // row j's key, 0 if used
      key = row16_max_u32(key);
      const float big = __uint_as_float(key & 0x7FFFFF80u), mine_abs = __uint_as_float(own & 0x7FFFFF80u);
      const bool fine = own != 0u && mine_abs >= TTC_PIVOT_THRESHOLD * big;
      diagonal = __ballot(!fine) == 0ull;
      pr = 127 - (int)(key & 0x7Fu);
      pr = pr < 16 ? pr : 15;  // never leave the problem's lanes, whatever the data
      pr = diagonal ? j : pr;
    } else {
      pr = j;
    }
    float prow[32];
    if (PIVOT && !diagonal) {
      const int src = ((lane & 48) | pr) << 2;  // byte address of the pivot row's lane
      static_for<j, 32>([&](auto K) {
        constexpr int k = decltype(K)::value;
        prow[k] = __builtin_bit_cast(float, __builtin_amdgcn_ds_bpermute(src, __builtin_bit_cast(int, a[k])));
      });
    } else {
      // the pivot row is lane j of every row of 16 lanes: a DPP broadcast within the row, no LDS crossbar
      static_for<j, 32>([&](auto K) {
        constexpr int k = decltype(K)::value;
        prow[k] = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, a[k]), 0x150 + j, 0xF, 0xF,
                                                                      true));  // row_newbcast:j
      });
    }
    const float pv = prow[j];
    const float apv = PIVOT ? fabsf(pv) : pv;
    if (!(apv > 0.f && apv < __builtin_inff())) bad = 1;
    const bool mine = (r == pr);
    const float nl = mine ? 0.f : -a[j] * __builtin_amdgcn_rcpf(pv);
    act = act && !mine;
    myj = mine ? j : myj;
    mypiv = mine ? pv : mypiv;
    static_for<j + 1, 32>([&](auto K) {
      constexpr int k = decltype(K)::value;
      a[k] = __builtin_fmaf(prow[k], nl, a[k]);  // nl = 0 for the pivot row itself
    });
  });
  const float s = __builtin_amdgcn_rcpf(mypiv);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    floatx4 t;
    t[0] = a[16 + 4 * k + 0] * s; t[1] = a[16 + 4 * k + 1] * s; t[2] = a[16 + 4 * k + 2] * s; t[3] = a[16 + 4 * k + 3] * s;
    *reinterpret_cast<floatx4*>(Wq + myj * C::PITCH + 16 + 4 * k) = t;
  }
  __syncthreads();
  return bad;
}

// Inverse of a symmetric positive definite 16 x 16 matrix, a row per lane (a[c] = M[r][c], r = lane & 15; the four rows
// of 16 lanes hold four matrices, or four copies of one): Gauss-Jordan without pivoting on [M | I], where the column of
// the right part that becomes non-trivial at step j takes the place of column j of M, which has just become a unit
// vector.  Rows are scaled by their pivots at the end (NEGATE leaves -M^{-1}, the sign riding on that scaling).
// The pivot row is broadcast within each row of 16 lanes as the DPP operand of the multiply-add itself.  What bounds a
// step is the chain multiplier -> column j + 1 -> its pivot's broadcast -> reciprocal -> next multiplier, some 65 cycles,
// beside the issue of 15 multiply-adds (4.4 cycles each): column j + 1 is updated first and its pivot's reciprocal is
// started under the other columns' updates, so that the larger of the two counts and not their sum.
// Returns, per lane, whether its row's pivot was not above piv_min and finite.
template <bool NEGATE = false>
__device__ __forceinline__ int invert_regs16(float (&a)[16], float piv_min = 0.f) {
  float mypiv = 1.f;
  float pv = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, a[0]), 0x150, 0xF, 0xF, true));
  float rc = __builtin_amdgcn_rcpf(pv);
  asm volatile("s_nop 1" : "+v"(rc));  // a transcendental's result may not be read by the very next vector instruction
  static_for<0, 16>([&](auto J) {
    constexpr int j = decltype(J)::value;
    float(&x)[16] = a;  // (named here, as an asm operand alone does not capture)
    float &kept = mypiv, &piv = pv, &rec = rc;
    constexpr unsigned mine = 0x00010001u << j;  // the lanes of the pivot row, either half of the mask (set up in vcc inside
                                                 // the block: as operands the masks are hoisted and spill scalar registers)
    // nl = the row's multiplier -a[j] / pivot (0 for the pivot row itself), then a[k] += nl * (a[k] of the pivot row, lane j
    // of this row of 16 lanes), k != j.  Written as one block so that the two wait states a DPP read needs after a vector
    // write of the same register are in our hands: the block starts with three instructions that write none of the
    // registers read by DPP, every multiply-add touches its own register, and the pivot of column j + 1 is read two
    // instructions after it was written.  %[p]: the pivot, kept by its row.
    float nl;
#define TTC_FMAC(n) "v_fmac_f32_dpp %" #n ", %" #n ", %[nl] row_newbcast:%[j] row_mask:0xf bank_mask:0xf\n\t"
    if constexpr (j < 15) {
#define TTC_AK(n) x[(n) == 0 ? j + 1 : ((n) <= j ? (n) - 1 : (n) + 1)]  // a[j + 1], then the other 14, in ascending order
      asm volatile(
          "s_mov_b32 vcc_lo, %[m]\n\ts_mov_b32 vcc_hi, %[m]\n\tv_mul_f32 %[nl], %[rc], -%[aj]\n\tv_cndmask_b32 %[p], %[p], %[pv], vcc\n\tv_cndmask_b32 %[nl], %[nl], 0, vcc\n\t"
          TTC_FMAC(0) TTC_FMAC(1) TTC_FMAC(2)
          "v_mov_b32_dpp %[pv], %0 row_newbcast:%[jn] row_mask:0xf bank_mask:0xf\n\t" TTC_FMAC(3) TTC_FMAC(4)
          "v_rcp_f32 %[rc], %[pv]\n\t" TTC_FMAC(5) TTC_FMAC(6) TTC_FMAC(7) TTC_FMAC(8) TTC_FMAC(9) TTC_FMAC(10) TTC_FMAC(11)
              TTC_FMAC(12) TTC_FMAC(13) TTC_FMAC(14) "v_cndmask_b32 %[aj], %[nl], 1.0, vcc"
          : "+v"(TTC_AK(0)), "+v"(TTC_AK(1)), "+v"(TTC_AK(2)), "+v"(TTC_AK(3)), "+v"(TTC_AK(4)), "+v"(TTC_AK(5)),
            "+v"(TTC_AK(6)), "+v"(TTC_AK(7)), "+v"(TTC_AK(8)), "+v"(TTC_AK(9)), "+v"(TTC_AK(10)), "+v"(TTC_AK(11)),
            "+v"(TTC_AK(12)), "+v"(TTC_AK(13)), "+v"(TTC_AK(14)), [aj] "+v"(x[j]), [p] "+v"(kept), [pv] "+v"(piv),
            [rc] "+v"(rec), [nl] "=&v"(nl)
          : [m] "n"(mine), [j] "n"(j), [jn] "n"(j + 1)
          : "vcc");
#undef TTC_AK
    } else {
      asm volatile(
          "s_mov_b32 vcc_lo, %[m]\n\ts_mov_b32 vcc_hi, %[m]\n\tv_mul_f32 %[nl], %[rc], -%[aj]\n\tv_cndmask_b32 %[p], %[p], %[pv], vcc\n\tv_cndmask_b32 %[nl], %[nl], 0, vcc\n\t"
          TTC_FMAC(0) TTC_FMAC(1) TTC_FMAC(2) TTC_FMAC(3) TTC_FMAC(4) TTC_FMAC(5) TTC_FMAC(6) TTC_FMAC(7) TTC_FMAC(8)
              TTC_FMAC(9) TTC_FMAC(10) TTC_FMAC(11) TTC_FMAC(12) TTC_FMAC(13) TTC_FMAC(14)
          "v_cndmask_b32 %[aj], %[nl], 1.0, vcc\n\ts_nop 1"
          : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(x[4]), "+v"(x[5]), "+v"(x[6]), "+v"(x[7]), "+v"(x[8]),
            "+v"(x[9]), "+v"(x[10]), "+v"(x[11]), "+v"(x[12]), "+v"(x[13]), "+v"(x[14]), [aj] "+v"(x[15]), [p] "+v"(kept),
            [pv] "+v"(piv), [rc] "+v"(rec), [nl] "=&v"(nl)
          : [m] "n"(mine), [j] "n"(15)
          : "vcc");
    }
#undef TTC_FMAC
  });
  const float s = NEGATE ? -__builtin_amdgcn_rcpf(mypiv) : __builtin_amdgcn_rcpf(mypiv);
#pragma unroll
  for (int k = 0; k < 16; ++k) a[k] *= s;
  return !(mypiv > piv_min && mypiv < __builtin_inff());
}

// x of the sixteen lanes of group J (lane / 16), in every group
template <int J>
__device__ __forceinline__ float broadcast_group(float x) {
  const unsigned u = __float_as_uint(x);
  const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);  // both halves: groups (0, 1), or (2, 3)
  const unsigned y = J >= 2 ? h[1] : h[0];
  const auto q = __builtin_amdgcn_permlane16_swap(y, y, false, false);
  return __uint_as_float((J & 1) ? q[1] : q[0]);
}

// The same inverse of one matrix by the whole wavefront, for results that must not depend on how many problems a wavefront has (invert_blocks16,
// below, is the faster): lane (i, g) holds M[i][4g .. 4g+3] (for a symmetric M its
// accumulator layout) and ends with the same entries of the inverse, which is its A operand, so that nothing passes
// through LDS.  Columns are taken four at a time: the four columns of a group are copied to every group first, where they
// are kept up to date beside the lane's own four; a column then costs seven multiply-adds instead of fifteen.  Every entry
// sees the operations of invert_regs16 in the same order.
__device__ __forceinline__ int invert_columns16(floatx4& m, int lane, float piv_min = 0.f) {
  const int g = lane >> 4;
  float a[4] = {m[0], m[1], m[2], m[3]};
  float mypiv = 1.f;
  static_for<0, 4>([&](auto JB) {
    constexpr int J = decltype(JB)::value;
    float c[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) c[k] = broadcast_group<J>(a[k]);
    float pv = __builtin_bit_cast(float, __builtin_amdgcn_mov_dpp(__builtin_bit_cast(int, c[0]), 0x150 + 4 * J, 0xF, 0xF,
                                                                  true));  // row_newbcast:4J
    float rc = __builtin_amdgcn_rcpf(pv);
    asm volatile("s_nop 1" : "+v"(rc));
    static_for<0, 4>([&](auto JJ) {
      constexpr int jj = decltype(JJ)::value, j = 4 * J + jj;
      constexpr unsigned mine = 0x00010001u << j;
      float(&x)[4] = a, (&y)[4] = c;
      float &kept = mypiv, &piv = pv, &rec = rc;
      // as in invert_regs16: the next column and its pivot's reciprocal first, the other columns under them
      float nl;
#define TTC_FMAC(n) "v_fmac_f32_dpp %" #n ", %" #n ", %[nl] row_newbcast:%[j] row_mask:0xf bank_mask:0xf\n\t"
      if constexpr (jj < 3) {
        asm volatile(
            "s_mov_b32 vcc_lo, %[m]\n\ts_mov_b32 vcc_hi, %[m]\n\tv_mul_f32 %[nl], %[rc], -%[cj]\n\tv_cndmask_b32 %[p], %[p], %[pv], vcc\n\tv_cndmask_b32 %[nl], %[nl], 0, vcc\n\t"
            TTC_FMAC(0) TTC_FMAC(3) TTC_FMAC(4)
            "v_mov_b32_dpp %[pv], %0 row_newbcast:%[jn] row_mask:0xf bank_mask:0xf\n\t" TTC_FMAC(5) TTC_FMAC(6)
            "v_rcp_f32 %[rc], %[pv]\n\t" TTC_FMAC(1) TTC_FMAC(2) "v_cndmask_b32 %[cj], %[nl], 1.0, vcc"
            : "+v"(y[jj + 1]), "+v"(y[(jj + 2) & 3]), "+v"(y[(jj + 3) & 3]), "+v"(x[0]), "+v"(x[1]), "+v"(x[2]),
              "+v"(x[3]), [cj] "+v"(y[jj]), [p] "+v"(kept), [pv] "+v"(piv), [rc] "+v"(rec), [nl] "=&v"(nl)
            : [m] "n"(mine), [j] "n"(j), [jn] "n"(j + 1)
          : "vcc");
      } else {
        asm volatile(
            "s_mov_b32 vcc_lo, %[m]\n\ts_mov_b32 vcc_hi, %[m]\n\tv_mul_f32 %[nl], %[rc], -%[cj]\n\tv_cndmask_b32 %[p], %[p], %[pv], vcc\n\tv_cndmask_b32 %[nl], %[nl], 0, vcc\n\t"
            TTC_FMAC(0) TTC_FMAC(1) TTC_FMAC(2) TTC_FMAC(3) TTC_FMAC(4) TTC_FMAC(5) TTC_FMAC(6)
            "v_cndmask_b32 %[cj], %[nl], 1.0, vcc\n\ts_nop 1"
            : "+v"(x[0]), "+v"(x[1]), "+v"(x[2]), "+v"(x[3]), "+v"(y[0]), "+v"(y[1]), "+v"(y[2]), [cj] "+v"(y[3]),
              [p] "+v"(kept), [pv] "+v"(piv), [rc] "+v"(rec), [nl] "=&v"(nl)
            : [m] "n"(mine), [j] "n"(j)
            : "vcc");
      }
#undef TTC_FMAC
    });
    const bool own = (g == J);
#pragma unroll
    for (int k = 0; k < 4; ++k) a[k] = own ? c[k] : a[k];
  });
  const float s = __builtin_amdgcn_rcpf(mypiv);
  m = floatx4{a[0] * s, a[1] * s, a[2] * s, a[3] * s};
  return !(mypiv > piv_min && mypiv < __builtin_inff());
}

// x of the sixteen lanes of group r (lane / 16) in every group, r = 0..3
__device__ __forceinline__ void groups_of(float x, float (&e)[4]) {
  const unsigned u = __float_as_uint(x);
  const auto h = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const auto lo = __builtin_amdgcn_permlane16_swap(h[0], h[0], false, false);
  const auto hi = __builtin_amdgcn_permlane16_swap(h[1], h[1], false, false);
  e[0] = __uint_as_float(lo[0]);
  e[1] = __uint_as_float(lo[1]);
  e[2] = __uint_as_float(hi[0]);
  e[3] = __uint_as_float(hi[1]);
}
// a where the mask is set, b elsewhere
__device__ __forceinline__ float bits_select(unsigned mask, float a, float b) {
  return __uint_as_float((mask & __float_as_uint(a)) | (~mask & __float_as_uint(b)));
}
__device__ __forceinline__ float bits_negate(float x) { return __uint_as_float(__float_as_uint(x) ^ 0x80000000u); }

// The inverse of one 16 x 16 matrix by the whole wavefront, in order, in place: m in the accumulator layout (lane (i, g) holds
// M[4g + v][i]) ends as the inverse in the same layout (for a symmetric M its A operand as well).  Block Gauss-Jordan with four pivot rows
// at a time, rows 4 k + b, k = 0..3: register m[b], which is the panel of these rows as an operand from the right.  The panel is copied to
// all four lane groups; there row r of it is e[r], of which only the block's own columns count, and y[r], which starts as the rows with the
// identity in those columns and ends as the rows times the inverse of the block: elimination in order and back substitution, the pivot
// row's entries broadcast within 16 lanes as the DPP operand of the multiply-add.  The other rows take their update, rank 4, as one matrix
// instruction, whose operand from the left is minus the block's columns: z = -M^T, kept beside m in the same layout for one more matrix
// instruction a block.  (Of a symmetric M they are the panel itself, signs turned where a column has been a pivot; taken from there, 60
// cycles less, solves at d = 64 with R of condition 1e6 came out twice as far off.)
//
// What bounds it is the number of instructions a lone wavefront issues (one in five cycles or so) and the chain of sixteen pivots; a
// column at a time, every lane group updating its four columns and a copy of the pivots' (390 instructions), took 2018 cycles, this
// (260) 1600; three wavefronts a SIMD slow each other by 6 % only.  Error against float64,
// well-conditioned matrices: 1.2e-7 (1.3e-7 before).
// Returns, uniformly, whether a pivot was not above piv_min and finite.
__device__ __forceinline__ int invert_blocks16(floatx4& m, floatx4 z, int lane, float piv_min) {
  const int i = lane & 15, g = lane >> 4;
  unsigned mask = (i & 3) == 0 ? ~0u : 0u;  // the columns of the pivot block, lanes 4 k + b
  float unit[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) unit[r] = (i >> 2) == r ? 1.f : 0.f;
  const float own = (i >> 2) == g ? -1.f : 0.f;
  float kept = 1.f;  // the sixteen pivots: pivot 4 k + b in the lanes 4 b .. 4 b + 3 of group k
  static_for<0, 4>([&](auto BB) {
    constexpr int b = decltype(BB)::value;
    float e[4], y[4], rc;
    const float a = z[b];  // minus the block's columns
    groups_of(m[b], e);
#pragma unroll
    for (int r = 0; r < 4; ++r) y[r] = bits_select(mask, unit[r], e[r]);
    float(&E)[4] = e, (&Y)[4] = y;  // (named here, as an asm operand alone does not capture)
    float& K = kept;
    // One block, so that the wait states are in our hands: two instructions between a vector write of a register and its DPP read, one
    // between a reciprocal and its use.  -e[r] as a DPP operand: minus the entry of row r in the pivot's column.
#define TTC_ALL " row_mask:0xf bank_mask:0xf\n\t"
#define TTC_RCP(p) "v_rcp_f32_dpp %[rc], %[e" #p "] row_newbcast:%[c" #p "]" TTC_ALL \
                   "v_mov_b32_dpp %[k], %[e" #p "] row_newbcast:%[c" #p "] row_mask:%[r" #p "] bank_mask:%[bm]\n\t"
#define TTC_MUL(v, p) "v_mul_f32 %[" #v #p "], %[" #v #p "], %[rc]\n\t"
#define TTC_SUB(v, r, p) "v_fmac_f32_dpp %[" #v #r "], -%[e" #r "], %[" #v #p "] row_newbcast:%[c" #p "]" TTC_ALL
#define TTC_ROW(r, m) "v_mov_b32_dpp %[y0], %[y" #r "] quad_perm:[0,1,2,3] row_mask:" #m " bank_mask:0xf\n\t"
    asm volatile(
        "s_nop 1\n\t" TTC_RCP(0) TTC_MUL(e, 0) TTC_MUL(y, 0)
        TTC_SUB(y, 1, 0) TTC_SUB(e, 1, 0) TTC_SUB(y, 2, 0) TTC_SUB(e, 2, 0) TTC_RCP(1) TTC_SUB(y, 3, 0) TTC_SUB(e, 3, 0)
        TTC_MUL(e, 1) TTC_MUL(y, 1) TTC_SUB(y, 2, 1) TTC_SUB(e, 2, 1) TTC_SUB(y, 3, 1) TTC_SUB(e, 3, 1) TTC_RCP(2)
        TTC_MUL(e, 2) TTC_MUL(y, 2) TTC_SUB(y, 3, 2) TTC_SUB(e, 3, 2) "s_nop 1\n\t" TTC_RCP(3)
        TTC_MUL(y, 3) TTC_SUB(y, 2, 3) TTC_SUB(y, 1, 3) TTC_SUB(y, 0, 3) TTC_SUB(y, 1, 2) TTC_SUB(y, 0, 2) TTC_SUB(y, 0, 1)
        TTC_ROW(1, 0x2) TTC_ROW(2, 0x4) TTC_ROW(3, 0x8) "s_nop 1"
        : [e0] "+v"(E[0]), [e1] "+v"(E[1]), [e2] "+v"(E[2]), [e3] "+v"(E[3]), [y0] "+v"(Y[0]), [y1] "+v"(Y[1]), [y2] "+v"(Y[2]),
          [y3] "+v"(Y[3]), [k] "+v"(K), [rc] "=&v"(rc)
        : [c0] "n"(b), [c1] "n"(4 + b), [c2] "n"(8 + b), [c3] "n"(12 + b), [r0] "n"(1), [r1] "n"(2), [r2] "n"(4), [r3] "n"(8),
          [bm] "n"(1 << b));
#undef TTC_ALL
#undef TTC_RCP
#undef TTC_MUL
#undef TTC_SUB
#undef TTC_ROW
    const float t = y[0];  // the panel times the inverse of the block, that inverse in the block's columns: row k in group k
    floatx4 rest;
#pragma unroll
    for (int v = 0; v < 4; ++v) rest[v] = bits_select(mask, 0.f, m[v]);
    m = __builtin_amdgcn_mfma_f32_16x16x4f32(a, t, rest, 0, 0, 0);
    m[b] = t;
    if constexpr (b < 3) {
      const float c = bits_select(mask, own, bits_negate(a));
#pragma unroll
      for (int v = 0; v < 4; ++v) rest[v] = v > b ? bits_select(mask, 0.f, z[v]) : z[v];
      z = __builtin_amdgcn_mfma_f32_16x16x4f32(t, c, rest, 0, 0, 0);
    }
    mask = (unsigned)__builtin_amdgcn_update_dpp(0, (int)mask, 0x93, 0xF, 0xF, false);  // quad_perm [3,0,1,2]
  });
  return __any(!(kept > piv_min && kept < __builtin_inff())) ? 1 : 0;
}
// of a symmetric matrix (symmetric up to rounding; where what follows is refined, as an R of condition 1e6 at d = 64 is 1.6 times as far
// off as with its own transpose)
__device__ __forceinline__ int invert_spread16(floatx4& m, int lane, float piv_min = 0.f) {
  return invert_blocks16(m, -m, lane, piv_min);
}
// of any matrix whose elimination in order is safe; T: 16 rows of `pitch` floats (a multiple of four) of LDS that are this wavefront's own,
// the last read of which it waits for
__device__ __forceinline__ int invert_spread16(floatx4& m, float* T, int pitch, int lane, float piv_min) {
  const int i = lane & 15, g = lane >> 4;
#pragma unroll
  for (int v = 0; v < 4; ++v) T[(4 * g + v) * pitch + i] = -m[v];
  wave_lds_sync();
  const floatx4 z = *reinterpret_cast<const floatx4*>(T + i * pitch + 4 * g);
  const int bad = invert_blocks16(m, z, lane, piv_min);
  wave_lds_sync();
  return bad;
}

// The same in place in LDS: the left halves of Wm[q] (row r at Wq + r*PITCH), by a workgroup of one wavefront.  The
// caller has ordered its writes of M; the function ends with an ordering of the wavefront's LDS traffic, which does not
// wait for global accesses.
template <bool NEGATE = false>
__device__ __forceinline__ int invert_rows16(float* Wq, int lane) {
  using C = Cfg<16>;
  const int r = lane & 15;
  float a[16];
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const floatx4 t = *reinterpret_cast<const floatx4*>(Wq + r * C::PITCH + 4 * k);
    a[4 * k + 0] = t[0]; a[4 * k + 1] = t[1]; a[4 * k + 2] = t[2]; a[4 * k + 3] = t[3];
  }
  const int bad = invert_regs16<NEGATE>(a);
#pragma unroll
  for (int k = 0; k < 4; ++k)
    *reinterpret_cast<floatx4*>(Wq + r * C::PITCH + 4 * k) = floatx4{a[4 * k], a[4 * k + 1], a[4 * k + 2], a[4 * k + 3]};
  wave_lds_sync();
  return bad;
}

// acc[q] += C_q Z_q for the wavefront's PPW problems at once, Z_q = the half of Wm[q] starting at column `half`.
// At d = 16 a product is four dependent matrix-core instructions; taking the k-steps of the four
// problems in turn keeps the pipe busy, and all sixteen B-operand reads are in flight together.
template <int PPW = 4>
__device__ __forceinline__ void gemm_acc_quad(floatx4 (&acc)[PPW][1][1], const float (&a)[PPW][1][4],
                                              float (*Wm)[16 * Cfg<16>::PITCH], int half, int i, int g) {
  using C = Cfg<16>;
  float b[PPW][4];
#pragma unroll
  for (int q = 0; q < PPW; ++q)
#pragma unroll
    for (int t = 0; t < 4; ++t) b[q][t] = Wm[q][half + (4 * g + t) * C::PITCH + i];
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int q = 0; q < PPW; ++q)
      acc[q][0][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[q][0][t], b[q][t], acc[q][0][0], 0, 0, 0);
}

}  // namespace ttc
