// List form of the shared-union search: wide tiles, narrow slices, and
// per-wave lists of (row, document) entries.
//
// A workgroup of S = 8 waves takes D = S * DW consecutive documents of the
// tiled order and one slice of 64 * NPL neurons whose rows are 512 bytes
// (128 fp32 or 256 fp16 neurons).  The tile's feature union is swept once, in
// stages of R = 64 rows held in a two-slot LDS ring (64 KB, two workgroups per
// CU), each wave moving its eight rows of a stage with four direct
// global-to-LDS loads.  Wave w owns documents w*DW .. w*DW+DW-1; a lane keeps
// NPL neurons of each in registers.  The plan stores, per stage and wave, the
// stage's (row, document) memberships as 16-bit entries (row offset in the
// slot | document), per document in ascending row order, padded to whole units
// of four with entries that add row 0 into a spare register.  A wave walks its
// list from scalar registers: per entry one vector instruction forms the LDS
// address, one LDS read fetches the lane's NPL weights, and NPL adds, whose
// accumulator is named through the VGPR index register, fold them in.  A
// unit's reads are issued before the previous unit's adds.
//
// What bounds it: no one unit.  An entry takes three vector instructions, two or
// three scalar ones and 512 bytes of LDS reads; on a 1,048,576-document batch of
// the 512^2 map (2.28 s) vector instructions fill 41% of the CUs' vector issue and
// scalar ones 37%, the LDS is busy for 21% of the cycles and a SIMD's matrix cores
// for 5%, and the waves, 16 per CU, wait 55% of their cycles: at the stage barrier,
// for their LDS reads and for the row loads, which come from the L2 for 78%
// (fp16: 55, 31, 19, 0 and 54%; topics: 36, 35, 20, 1 and 57%, 68% from the L2).
// A 262,144-document batch takes 504 ms (523 with every row in the lists; its row
// loads alone 300, beside the rest).  Kernel 3 took 545 ms there: its 64-document
// tiles of 256-neuron slices need 484 ms of row loads (33.6 rows per document at a
// working set of 20 MB per slice against 21.7 rows at 10 MB) and a scalar test per
// document and 16-row stage.  On the 512^2 topic batch 131,072 documents took
// 449-455 ms (kernel 3: 648); the 128^2 map's 65,536-document pass 8.4 ms (12.0).
// Measured and not kept: rows held by one document loaded straight into
// registers by the document's wave (575 ms: the loads wait for each other, where
// the staged ones are in flight together), and scalar copies of the next list's
// first entries instead of loading them inside the list's own statement.
//
// Sweep order, fixed by the plan's form (common.h) and the launch: ascending; as
// kernel 3's rotated sweep (see search_st.h) from a phase of the tile's own, taken
// in work (list entries and rows); or kernel 3's very order, super-tile by
// super-tile.  Each way a document's dot product is summed in the sweep's order,
// one fp32 add per feature, so the ascending sweep gives every kernel's bits and
// the last one kernel 3's.
#pragma once

#include <type_traits>

#include "search_st.h"

namespace som {
namespace {

typedef float f32x16v __attribute__((ext_vector_type(16)));
typedef float f32x32v __attribute__((ext_vector_type(32)));
typedef uint32_t u32x8v __attribute__((ext_vector_type(8)));
typedef int32_t i32x4v __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// A wave's list of one stage, as one inline-assembly statement.
//
// Registers: s[32:39] (s[40:47] in odd steps) and s[48:55] hold 16 entries (four
// units) each, reloaded alternately; s56-s59 hold the odd entries of the unit
// being added and of the next one, shifted down.  Rows land in v[24:31] (even
// units) and v[32:39] (odd units).  The statement also loads the next stage's
// first set into the other parity's registers.  The accumulators start at v40,
// one plane of DW registers per neuron of the lane, planes DW + 2 registers
// apart; register DW of a plane takes the padding.  Scalar loads and LDS reads
// share one counter and return out of order with each other, so every wait for
// them is for zero; a unit's wait falls after the whole adds of the unit before.
// Every load is waited for before the statement ends.
// ---------------------------------------------------------------------------
#define SOM_L_RD(S, R, R1) \
  "v_and_or_b32 v" #R ", s" #S ", %[vm], %[vl]\n\tds_read_b64 v[" #R ":" #R1 "], v" #R "\n\t"
#define SOM_L_ISSUE0(A, B)                                                               \
  SOM_L_RD(A, 24, 25) "s_lshr_b32 s56, s" #A ", 16\n\t" SOM_L_RD(56, 26, 27)             \
  SOM_L_RD(B, 28, 29) "s_lshr_b32 s57, s" #B ", 16\n\t" SOM_L_RD(57, 30, 31)
#define SOM_L_ISSUE1(A, B)                                                               \
  SOM_L_RD(A, 32, 33) "s_lshr_b32 s58, s" #A ", 16\n\t" SOM_L_RD(58, 34, 35)             \
  SOM_L_RD(B, 36, 37) "s_lshr_b32 s59, s" #B ", 16\n\t" SOM_L_RD(59, 38, 39)
#define SOM_L_IDX(S) "s_set_gpr_idx_idx s" #S "\n\t"
// four adds: entries (or singles) S0..S3, rows from v R, R + 2, ..
#define SOM_L_ADD4(S0, S1, S2, S3, R0, R1, R2, R3, R4, R5, R6, R7)                          \
  "s_set_gpr_idx_on s" #S0 ", " SOM_L_MODE "\n\t" SOM_L_ADD(R0, R1) SOM_L_IDX(S1)           \
      SOM_L_ADD(R2, R3) SOM_L_IDX(S2) SOM_L_ADD(R4, R5) SOM_L_IDX(S3) SOM_L_ADD(R6, R7) "s_set_gpr_idx_off\n\t"
#define SOM_L_ADDS0(A, B) SOM_L_ADD4(A, 56, B, 57, 24, 25, 26, 27, 28, 29, 30, 31)
#define SOM_L_ADDS1(A, B) SOM_L_ADD4(A, 58, B, 59, 32, 33, 34, 35, 36, 37, 38, 39)
// unit in dwords A, B, next unit's dwords NA, NB; n counts the units after
// this one (its borrow ends the list)
#define SOM_L_UNIT0(LBL, LOAD, A, B, NA, NB)                                            \
  "s_waitcnt lgkmcnt(0)\n\t" LOAD "s_sub_u32 %[n], %[n], 1\n\ts_cbranch_scc1 " LBL "\n\t" \
      SOM_L_ISSUE1(NA, NB) SOM_L_ADDS0(A, B)
#define SOM_L_UNIT1(LBL, LOAD, A, B, NA, NB)                                            \
  "s_waitcnt lgkmcnt(0)\n\t" LOAD "s_sub_u32 %[n], %[n], 1\n\ts_cbranch_scc1 " LBL "\n\t" \
      SOM_L_ISSUE0(NA, NB) SOM_L_ADDS1(A, B)
#define SOM_L_LAST0(LBL, A, B) LBL ":\n\t" SOM_L_ADDS0(A, B) "s_branch .Lsom_end%=\n"
#define SOM_L_LAST1(LBL, A, B) LBL ":\n\t" SOM_L_ADDS1(A, B) "s_branch .Lsom_end%=\n"
#define SOM_L_LB(K) ".Lsom_u" #K "_%="
// reload of an entry set when four or more units follow (n as above)
#define SOM_L_RELOAD(K, SET, OFF)                                                          \
  "s_cmp_lt_u32 %[n], 4\n\ts_cbranch_scc1 .Lsom_l" #K "_%=\n\ts_load_dwordx8 " SET ", %[lb], %[eo] offset:" OFF "\n.Lsom_l" #K "_%=:\n\t"
// SET, A0..A7: the first entry set; NSET: the next stage's
#define SOM_L_BODY(SET, NSET, A0, A1, A2, A3, A4, A5, A6, A7)                              \
  "s_load_dwordx8 " NSET ", %[lb], %[neo]\n\t"                                             \
  "s_cmp_eq_u32 %[n], -1\n\ts_cbranch_scc1 .Lsom_end%=\n\t"                                \
  SOM_L_ISSUE0(A0, A1)                                                                     \
  ".Lsom_top%=:\n\t"                                                                       \
  SOM_L_UNIT0(SOM_L_LB(0), SOM_L_RELOAD(0, "s[48:55]", "0x20"), A0, A1, A2, A3)            \
  SOM_L_UNIT1(SOM_L_LB(1), "", A2, A3, A4, A5)                                             \
  SOM_L_UNIT0(SOM_L_LB(2), "", A4, A5, A6, A7)                                             \
  SOM_L_UNIT1(SOM_L_LB(3), "", A6, A7, 48, 49)                                             \
  SOM_L_UNIT0(SOM_L_LB(4), SOM_L_RELOAD(4, SET, "0x40"), 48, 49, 50, 51)                   \
  SOM_L_UNIT1(SOM_L_LB(5), "", 50, 51, 52, 53)                                             \
  SOM_L_UNIT0(SOM_L_LB(6), "", 52, 53, 54, 55)                                             \
  SOM_L_UNIT1(SOM_L_LB(7), "", 54, 55, A0, A1)                                             \
  "s_add_u32 %[eo], %[eo], 0x40\n\ts_branch .Lsom_top%=\n"                                 \
  SOM_L_LAST0(SOM_L_LB(0), A0, A1) SOM_L_LAST1(SOM_L_LB(1), A2, A3)                        \
  SOM_L_LAST0(SOM_L_LB(2), A4, A5) SOM_L_LAST1(SOM_L_LB(3), A6, A7)                        \
  SOM_L_LAST0(SOM_L_LB(4), 48, 49) SOM_L_LAST1(SOM_L_LB(5), 50, 51)                        \
  SOM_L_LAST0(SOM_L_LB(6), 52, 53) SOM_L_LAST1(SOM_L_LB(7), 54, 55)                        \
  ".Lsom_end%=:\n\ts_waitcnt lgkmcnt(0)\n\t"
#define SOM_L_EVEN SOM_L_BODY("s[32:39]", "s[40:47]", 32, 33, 34, 35, 36, 37, 38, 39)
#define SOM_L_ODD SOM_L_BODY("s[40:47]", "s[32:39]", 40, 41, 42, 43, 44, 45, 46, 47)
#define SOM_L_CLOBBERS                                                                                             \
  "v24", "v25", "v26", "v27", "v28", "v29", "v30", "v31", "v32", "v33", "v34", "v35", "v36", "v37", "v38", "v39",  \
      "s48", "s49", "s50", "s51", "s52", "s53", "s54", "s55", "s56", "s57", "s58", "s59", "scc", "memory"

// Accumulators of a wave: plane q holds neuron q of the lane for each document.
template <int DW, int NPL>
struct ListAcc;
template <int NPL>
struct ListAcc<32, NPL> {
  f32x32v p[NPL];
};
template <int NPL>
struct ListAcc<16, NPL> {
  f32x16v p[NPL];
};

// Adds a stage's list and loads the next one's first set.  lb: the tile's
// lists; eo, neo: byte offsets of this stage's list and the next one's; n: units
// of four entries, less one; vl: the slot's base | the lane's byte offset in a
// row; vm: the mask of an entry's row offset.
#define SOM_L_OPERANDS(SET, NSET) "={m0}"(m0), SET(set), NSET(nset), [eo] "+s"(eo), [n] "+s"(n), SOM_L_ACC
#define SOM_L_INPUTS [lb] "s"(lb), [neo] "s"(neo), [vl] "v"(vl), [vm] "v"(vm)
// (the index register is M0)
#define SOM_L_DEFINE(DW, NPL)                                                                                       \
  template <bool ODD>                                                                                               \
  __device__ __forceinline__ u32x8v add_list(ListAcc<DW, NPL>& acc, u32x8v set, uint64_t lb, uint32_t eo,           \
                                             uint32_t neo, uint32_t n, uint32_t vl, uint32_t vm) {                  \
    u32x8v nset;                                                                                                    \
    uint32_t m0;                                                                                                    \
    if constexpr (ODD)                                                                                              \
      asm volatile(SOM_L_ODD                                                                                        \
                   : SOM_L_OPERANDS("+{s[40:47]}", "=&{s[32:39]}") : SOM_L_INPUTS : SOM_L_CLOBBERS, SOM_L_SPARE);   \
    else                                                                                                            \
      asm volatile(SOM_L_EVEN                                                                                       \
                   : SOM_L_OPERANDS("+{s[32:39]}", "=&{s[40:47]}") : SOM_L_INPUTS : SOM_L_CLOBBERS, SOM_L_SPARE);   \
    return nset;                                                                                                    \
  }
// The dense rows.  A row's products with a wave's 32 documents, into the plane of
// accumulators from register BASE on; v W: its weights, v H: 1 where lane s's
// document holds it, else 0.
#define SOM_L_MFMA(BASE, I, W, H)                                                                                  \
  "v_mfma_f32_4x4x1_16b_f32 v[" #BASE "+4*" #I ":" #BASE "+4*" #I "+3], v" #H ", v" #W ", v[" #BASE "+4*" #I       \
  ":" #BASE "+4*" #I "+3] cbsz:4 abid:" #I "\n\t"
#define SOM_L_MFMA32(BASE, W, H)                                                                               \
  SOM_L_MFMA(BASE, 0, W, H) SOM_L_MFMA(BASE, 1, W, H) SOM_L_MFMA(BASE, 2, W, H) SOM_L_MFMA(BASE, 3, W, H)      \
  SOM_L_MFMA(BASE, 4, W, H) SOM_L_MFMA(BASE, 5, W, H) SOM_L_MFMA(BASE, 6, W, H) SOM_L_MFMA(BASE, 7, W, H)
#define SOM_L_HELD(K, H) "v_bfe_u32 v" #H ", %[lo], " #K ", 1\n\tv_cvt_f32_u32_e32 v" #H ", v" #H "\n\t"
// Four rows per step, two vector instructions and a wait state before the first
// product; after the last, the wait states until other instructions may read
// the sums.  special: row by row, each holder by the lists' indexed add.
#define SOM_L_DENSE                                                                                               \
  "s_cmp_lg_u32 %[special], 0\n\ts_cbranch_scc1 .Lsom_special%=\n"                                                \
  ".Lsom_four%=:\n\t"                                                                                             \
  "ds_read_b64 v[24:25], %[row]\n\tds_read_b64 v[26:27], %[row] offset:512\n\t"                                   \
  "ds_read_b64 v[28:29], %[row] offset:1024\n\tds_read_b64 v[30:31], %[row] offset:1536\n\t"                      \
  SOM_L_HELD(0, 32) SOM_L_HELD(1, 33) SOM_L_HELD(2, 34) SOM_L_HELD(3, 35)                                         \
  "v_alignbit_b32 %[lo], %[hi], %[lo], 4\n\tv_lshrrev_b32_e32 %[hi], 4, %[hi]\n\tv_add_u32_e32 %[row], 0x800, %[row]\n\t"                                  \
  "s_waitcnt lgkmcnt(0)\n\ts_nop 1\n\t"                                                                           \
  SOM_L_PRODUCTS(24, 25, 32) SOM_L_PRODUCTS(26, 27, 33) SOM_L_PRODUCTS(28, 29, 34) SOM_L_PRODUCTS(30, 31, 35)     \
  "s_sub_u32 %[n], %[n], 4\n\ts_cmp_lg_u32 %[n], 0\n\ts_cbranch_scc1 .Lsom_four%=\n\t"                            \
  "s_nop 7\n\ts_nop 7\n\ts_branch .Lsom_done%=\n"                                                                 \
  ".Lsom_special%=:\n\t"                                                                                          \
  "ds_read_b64 v[24:25], %[row]\n\t"                                                                              \
  "v_and_b32_e32 v32, 1, %[lo]\n\tv_cmp_ne_u32_e32 vcc, 0, v32\n\ts_nop 4\n\t"                                 \
  "s_mov_b32 s48, vcc_lo\n\ts_waitcnt lgkmcnt(0)\n"                                                                 \
  ".Lsom_holder%=:\n\t"                                                                                           \
  "s_cmp_eq_u32 s48, 0\n\ts_cbranch_scc1 .Lsom_next%=\n\t"                                                        \
  "s_ff1_i32_b32 s49, s48\n\ts_bitset0_b32 s48, s49\n\t"                                                          \
  "s_set_gpr_idx_on s49, " SOM_L_MODE "\n\t" SOM_L_ADD(24, 25) "s_set_gpr_idx_off\n\t"                            \
  "s_branch .Lsom_holder%=\n"                                                                                     \
  ".Lsom_next%=:\n\t"                                                                                             \
  "v_alignbit_b32 %[lo], %[hi], %[lo], 1\n\tv_lshrrev_b32_e32 %[hi], 1, %[hi]\n\tv_add_u32_e32 %[row], 0x200, %[row]\n\t"                                  \
  "s_sub_u32 %[n], %[n], 1\n\ts_cmp_lg_u32 %[n], 0\n\ts_cbranch_scc1 .Lsom_special%=\n"                           \
  ".Lsom_done%=:\n\t"
#define SOM_L_DEFINE_DENSE(NPL)                                                                                     \
  __device__ __forceinline__ void add_dense_rows(ListAcc<32, NPL>& acc, uint32_t row, uint32_t n, uint32_t lo,       \
                                                 uint32_t hi, uint32_t special) {                                   \
    uint32_t m0;                                                                                                    \
    asm volatile(SOM_L_DENSE                                                                                        \
                 : "={m0}"(m0), [row] "+v"(row), [n] "+s"(n), [lo] "+v"(lo), [hi] "+v"(hi), SOM_L_ACC               \
                 : [special] "s"(special) : SOM_L_CLOBBERS, "vcc", SOM_L_SPARE);                                    \
  }
// fp32 rows: two neurons per lane
#define SOM_L_MODE "gpr_idx(SRC0,DST)"
#define SOM_L_ADD(R, R1) "v_add_f32_e32 v40, v40, v" #R "\n\tv_add_f32_e32 v74, v74, v" #R1 "\n\t"
#define SOM_L_ACC "+{v[40:71]}"(acc.p[0]), "+{v[74:105]}"(acc.p[1])
#define SOM_L_SPARE "v72", "v106"
#define SOM_L_PRODUCTS(R, R1, H) \
  SOM_L_MFMA32(40, R, H) SOM_L_MFMA32(74, R1, H)
SOM_L_DEFINE(32, 2)
SOM_L_DEFINE_DENSE(2)
#undef SOM_L_PRODUCTS
#undef SOM_L_ADD
#undef SOM_L_ACC
#undef SOM_L_SPARE
#define SOM_L_ADD(R, R1) "v_add_f32_e32 v40, v40, v" #R "\n\tv_add_f32_e32 v58, v58, v" #R1 "\n\t"
#define SOM_L_ACC "+{v[40:55]}"(acc.p[0]), "+{v[58:73]}"(acc.p[1])
#define SOM_L_SPARE "v56", "v74"
SOM_L_DEFINE(16, 2)
#undef SOM_L_ADD
#undef SOM_L_ACC
#undef SOM_L_SPARE
#undef SOM_L_MODE
#define SOM_L_WIDEN(R, R1) \
  "v_cvt_f32_f16_e32 v36, v" #R "\n\tv_cvt_f32_f16_sdwa v37, v" #R " dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1\n\t" \
  "v_cvt_f32_f16_e32 v38, v" #R1 "\n\tv_cvt_f32_f16_sdwa v39, v" #R1 " dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1\n\ts_nop 1\n\t"
// fp16 rows: four neurons per lane, each half widened and added by one fused
// multiply-add with 1.0 (exact product, one rounding: the widened add)
#define SOM_L_MODE "gpr_idx(SRC2,DST)"
#define SOM_L_MIX(P, R, HI) \
  "v_fma_mix_f32 v" #P ", v" #R ", 1.0, v" #P " op_sel:[" #HI ",0,0] op_sel_hi:[1,0,0]\n\t"
#define SOM_L_ADD(R, R1) SOM_L_MIX(40, R, 0) SOM_L_MIX(58, R, 1) SOM_L_MIX(76, R1, 0) SOM_L_MIX(94, R1, 1)
#define SOM_L_ACC "+{v[40:55]}"(acc.p[0]), "+{v[58:73]}"(acc.p[1]), "+{v[76:91]}"(acc.p[2]), "+{v[94:109]}"(acc.p[3])
#define SOM_L_SPARE "v56", "v74", "v92", "v110"
SOM_L_DEFINE(16, 4)
#undef SOM_L_ADD
#undef SOM_L_ACC
#undef SOM_L_SPARE
#define SOM_L_ADD(R, R1) SOM_L_MIX(40, R, 0) SOM_L_MIX(74, R, 1) SOM_L_MIX(108, R1, 0) SOM_L_MIX(142, R1, 1)
#define SOM_L_ACC "+{v[40:71]}"(acc.p[0]), "+{v[74:105]}"(acc.p[1]), "+{v[108:139]}"(acc.p[2]), "+{v[142:173]}"(acc.p[3])
#define SOM_L_SPARE "v72", "v106", "v140", "v174"
#define SOM_L_PRODUCTS(R, R1, H) \
  SOM_L_WIDEN(R, R1) SOM_L_MFMA32(40, 36, H) SOM_L_MFMA32(74, 37, H) SOM_L_MFMA32(108, 38, H) SOM_L_MFMA32(142, 39, H)
SOM_L_DEFINE(32, 4)
SOM_L_DEFINE_DENSE(4)
#undef SOM_L_PRODUCTS
#undef SOM_L_ADD
#undef SOM_L_ACC
#undef SOM_L_SPARE
#undef SOM_L_MODE

typedef uint32_t u32x2w __attribute__((ext_vector_type(2)));

// A lane's 8 bytes of a row as its neurons' weights.
template <typename WT, int NPL>
__device__ __forceinline__ void widen(u32x2w raw, float (&w)[NPL]) {
  if constexpr (sizeof(WT) == 4) {
    w[0] = __uint_as_float(raw.x);
    w[1] = __uint_as_float(raw.y);
  } else {
    typedef _Float16 half4 __attribute__((ext_vector_type(4)));
    const half4 v = __builtin_bit_cast(half4, raw);
#pragma unroll
    for (int q = 0; q < NPL; ++q) w[q] = static_cast<float>(v[q]);
  }
}

// Adds the dense rows (nd of them, in the first rows of the slot; ring + row: the
// lane's 8 bytes of slot row 0) on the matrix cores: v_mfma_f32_4x4x1 multiplies
// four documents' 0 or 1 (one block of A, named by the instruction and broadcast
// to all sixteen) with the lane's neuron of one row, and adds into the four
// documents' accumulators, which lie as the lists' adds have them (lane =
// neuron, register = document).  8 * NPL of them add a row into the wave's 32
// documents; the products are exact and each sum is rounded once, as an add is.
// The 16 instructions of a row of fp32 weights take 128 cycles whatever it holds;
// the lists' three per holder take about twelve, so the plan takes a row from
// 3/8 of the documents on.  Measured, before -> after (fp32): 512^2 and 256^2 maps with 256k documents, and 1M documents on 32 x 32 -3.6%, -3.7%, -4.7% (523.2 -> 504.5, 133.5 ->
// 128.5, 10.5 -> 10.0 ms); with 1/4 of the documents 510, 1/2 507, 3/4 536.  fp16
// tiles (16 documents a wave) gained nothing (354 -> 355) and have lists only.
template <typename WT, int NPL>
__device__ __forceinline__ void add_dense(ListAcc<32, NPL>& acc, const unsigned char* ring, uint32_t row, int nd,
                                          const unsigned char* masks, int lane) {
  // lane s < 32: the dense rows that document s of the wave holds, by slot row
  // (read here: kept in flight over the wait above, it delayed the stage by 2%)
  const uint64_t held = reinterpret_cast<const uint64_t*>(masks)[lane & 31];
  bool special = false;
  const int n = (nd + 7) & ~7;   // (rows past the last have no holder)
#pragma clang loop unroll(disable)
  for (int u = 0; u < n; u += 8)
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      float w[NPL];
      widen<WT, NPL>(*reinterpret_cast<const u32x2w*>(ring + row + (u + k) * kListRowBytes), w);
#pragma unroll
      for (int q = 0; q < NPL; ++q) special |= __builtin_amdgcn_classf(w[q], 0x207);   // an infinity or a NaN
    }
  // 0 times such a value is no 0: these rows are added to their holders only
  add_dense_rows(acc, lds_offset(ring) + row, n, static_cast<uint32_t>(held), static_cast<uint32_t>(held >> 32),
                 __builtin_amdgcn_readfirstlane(__ballot(special) != 0));
}

// Minimum of x over the wave, uniform (data-parallel-primitive row shifts, then
// the two row broadcasts: lane 63 ends with the whole wave's).
__device__ __forceinline__ uint32_t wave_min_u32(uint32_t x) {
#define SOM_DPP_MIN(CTRL, ROWS)                                                                   \
  {                                                                                               \
    const uint32_t y_ = static_cast<uint32_t>(                                                    \
        __builtin_amdgcn_update_dpp(-1, static_cast<int>(x), CTRL, ROWS, 0xf, false));            \
    x = y_ < x ? y_ : x;                                                                          \
  }
  SOM_DPP_MIN(0x111, 0xf)
  SOM_DPP_MIN(0x112, 0xf)
  SOM_DPP_MIN(0x114, 0xf)
  SOM_DPP_MIN(0x118, 0xf)
  SOM_DPP_MIN(0x142, 0xa)
  SOM_DPP_MIN(0x143, 0xc)
#undef SOM_DPP_MIN
  return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(x), 63));
}

// Distances, argmin (or the two smallest) and key merge of a wave's DW
// documents over its slice.  Per document the lane's best neuron is reduced
// over the wave as ordered distance bits; the lowest lane that holds the
// minimum gives the lowest index (a lane's neurons ascend, and lanes do).  Columns
// past the last neuron are left out by their index, as their accumulators hold
// whatever lies between the rows: inside a lane they follow its neurons with an
// infinite or NaN distance, which is never less than another; lanes without a
// neuron, or (second best) without a second one, take no part.  Lane s then holds
// document s's key, and one vector compare filters the atomics: a stale read of
// the stored key only lets a useless update through, as keys only fall.
template <int DW, int NPL, bool TOP2>
__device__ __forceinline__ void list_epilogue(const SearchArgs& a, const ListAcc<DW, NPL>& acc, int64_t p0, int64_t n0,
                                              int lane) {
  if (p0 >= a.B) return;   // (documents past the last are reduced with the others, and not stored)
  float nrm[NPL];
#pragma unroll
  for (int q = 0; q < NPL; ++q) {
    const int64_t j = n0 + lane * NPL + q;
    nrm[q] = j < a.N ? a.norms[j] : __builtin_inff();
  }
  const bool one = n0 + lane * NPL < a.N, two = n0 + lane * NPL + 1 < a.N;   // neurons of this lane
  const uint64_t ones = __ballot(one), twos = __ballot(two);
  const int64_t p = p0 + lane;
  const bool mine = lane < DW && p < a.B;
  float nnz = 0.f;
  if (mine) {
    const int64_t d = a.perm ? static_cast<int64_t>(a.perm[p]) : p;
    nnz = static_cast<float>(a.indptr[d + 1] - a.indptr[d]);
  }
  int m1 = -1, j1 = 0, m2 = -1, j2 = 0;
#pragma unroll
  for (int s = 0; s < DW; ++s) {
    const float nn = __uint_as_float(
        static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(__float_as_uint(nnz)), s)));
    float d1 = 0.f, d2 = __builtin_inff();   // the lane's best, and second best
    uint32_t q1 = 0, q2 = 0;
#pragma unroll
    for (int q = 0; q < NPL; ++q) {
      const float d = fmaf(-2.f, acc.p[q][s], nn + nrm[q]);
      const bool lt1 = q == 0 || d < d1;     // ascending neurons: strict < keeps the lowest
      if (TOP2) {
        const bool lt2 = q == 1 || d < d2;
        if (q > 0) {
          d2 = lt1 ? d1 : (lt2 ? d : d2);
          q2 = lt1 ? q1 : (lt2 ? static_cast<uint32_t>(q) : q2);
        }
      }
      q1 = lt1 ? static_cast<uint32_t>(q) : q1;
      d1 = lt1 ? d : d1;
    }
    const uint32_t b1 = one ? ordered_bits(d1) : ~0u;
    const uint32_t m = wave_min_u32(b1);
    const int l = __builtin_ctzll(__ballot(b1 == m));   // some lane holds the minimum; lane 0 has a neuron
    const int j = static_cast<int>(n0) + l * NPL + __builtin_amdgcn_readlane(static_cast<int>(q1), l);
    m1 = lane == s ? static_cast<int>(m) : m1;
    j1 = lane == s ? j : j1;
    if (TOP2) {
      const uint32_t c = lane == l ? (two ? ordered_bits(d2) : ~0u) : b1;
      const uint32_t cq = lane == l ? q2 : q1;
      const uint32_t mm = wave_min_u32(c);
      const uint64_t others = (ones & ~(1ull << l)) | (twos & (1ull << l));
      int jj = -1;   // a slice of one neuron has no second best: m2 = j2 = -1, kNoKey
      if (others) {
        const int l2 = __builtin_ctzll(__ballot(c == mm) & others);
        jj = static_cast<int>(n0) + l2 * NPL + __builtin_amdgcn_readlane(static_cast<int>(cq), l2);
      }
      m2 = lane == s ? static_cast<int>(mm) : m2;
      j2 = lane == s ? jj : j2;
    }
  }
  if (!mine) return;
  const uint64_t k1 = (static_cast<uint64_t>(static_cast<uint32_t>(m1)) << 32) | static_cast<uint32_t>(j1);
  uint64_t* kb = a.keys + p;
  if (!TOP2) {
    if (k1 < *kb) atomicMin(reinterpret_cast<unsigned long long*>(kb), static_cast<unsigned long long>(k1));
    return;
  }
  const uint64_t k2 = (static_cast<uint64_t>(static_cast<uint32_t>(m2)) << 32) | static_cast<uint32_t>(j2);
  const uint64_t displaced = k1 < *kb ? top2_displaced(kb, k1) : k1;
  const uint64_t cand = displaced < k2 ? displaced : k2;
  uint64_t* ks = a.keys2 + p;
  if (cand < *ks) atomicMin(reinterpret_cast<unsigned long long*>(ks), static_cast<unsigned long long>(cand));
}

// Waves per SIMD the registers must allow: the four that two workgroups per CU
// make, except where an fp16 codebook is searched with a plan made for fp32 (128
// accumulators per lane).
template <typename WT, int DW>
constexpr int list_min_waves() {
  return sizeof(WT) == 2 && DW == 32 ? 2 : 4;
}

// WIDE: codebook rows of 4 GB and more.  SUPER: a kListSuperOrder plan (a second
// place in the lists, beside the stages', cost the other forms 0.6% at 512^2: 507.5
// against 504.3 ms per 262,144 documents).
template <typename WT, int DW, bool TOP2, bool WIDE, bool SUPER>
__global__ void __launch_bounds__(kListWaves * 64) __attribute__((amdgpu_waves_per_eu(list_min_waves<WT, DW>())))
k_search_list(SearchArgs a) {
  constexpr int E = Storage<WT>::kE;                               // elements per 128-bit load
  constexpr int NPL = kListRowBytes / 64 / static_cast<int>(sizeof(WT));  // neurons per lane
  constexpr int64_t WN = 64 * NPL;                                 // neurons per slice
  constexpr int S = kListWaves, R = kListRows;
  constexpr uint32_t kSlot = R * kListRowBytes;
  static_assert(R == 8 * S && kListRowBytes == 512 && kSlot == 0x8000, "four two-row loads per wave and stage");
  // the kernel's only LDS object, at LDS address 0: entry addresses are formed
  // by or-ing a row's offset into the slot's base
  __shared__ __attribute__((aligned(1024))) unsigned char ring[2 * R * kListRowBytes];

  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // XCD-contiguous tile ranges, slice-major (see k_search).  SUPER: the tiles are
  // few, and whole ranges of them per XCD would leave some XCDs with less, or
  // nothing; dealt out tile by tile over all slices, each XCD gets its share (2,560
  // documents on 256^2: ranges 0.77 of kernel 3's speed, dealt out 1.16)
  const uint32_t per_xcd = gridDim.x / kXcds;
  const int64_t t = SUPER ? static_cast<int64_t>(blockIdx.x)
                          : static_cast<int64_t>(blockIdx.x % kXcds) * per_xcd + blockIdx.x / kXcds;
  if (t >= a.ntiles) return;  // whole workgroup: no barrier is skipped by part of it
  if (a.either && !(static_cast<uint32_t>(a.tile_offset[0]) & kListTag)) return;  // a tile plan
  const int64_t n0 = (a.slice_base + blockIdx.y) * WN;

  ListAcc<DW, NPL> acc;
#pragma unroll
  for (int q = 0; q < NPL; ++q)
#pragma unroll
    for (int s = 0; s < DW; ++s) acc.p[q][s] = 0.f;

  // lane's 16 bytes of a row: piece lane % 32; lanes past the last neuron
  // re-read the last 128-bit group holding one, so no load leaves
  // [0, round_up(N, E)) of its row
  const int64_t o = E * (lane & 31);
  const int64_t nv = (a.N + E - 1) / E * E;
  const char* __restrict__ Wl = reinterpret_cast<const char*>(static_cast<const WT*>(a.W) + n0 +
                                                              (n0 + o < nv ? o : nv - E - n0));
  const uint64_t ldw_b = static_cast<uint64_t>(a.ldw) * sizeof(WT);
  typedef const __attribute__((address_space(4))) uint32_t* const_u32;
  typedef const __attribute__((address_space(4))) int32_t* const_i32;
  typedef const __attribute__((address_space(4))) char* const_char;
  auto offset = [&](int64_t i) {
    return static_cast<uint64_t>(static_cast<uint32_t>(((const_i32)a.tile_offset)[i]) & ~kListTag);
  };
  const int64_t cap0 = static_cast<int64_t>(offset(t));
  const uint32_t tc = static_cast<uint32_t>(((const_i32)a.tile_count)[t]);
  const int32_t nst = static_cast<int32_t>(tc & 0x7ffu);                      // stages
  const int32_t nd = SUPER ? 0 : static_cast<int32_t>(tc >> 16);              // dense rows
  // visits of stages: one each, and (kListSuperOrder) some again
  const int32_t visits = nst + (SUPER ? static_cast<int32_t>(tc >> 21) : 0);
  // unit offsets of the tile's lists, visit by visit: list (v, w) holds units
  // pt[v * S + w] .. pt[v * S + w + 1]
  const const_u32 pt = (const_u32)(a.list_start + cap0 * list_cap_lists(SUPER) + t);
  const unsigned char* masks = a.list_data + cap0 * list_cap_bytes(SUPER);
  const unsigned char* data = masks + (nd ? S * DW * 8 : 0);
  const const_char lists = (const_char)(data + nst * (R * 4));

  if (nst > 0) {
    // Rotated sweep: the plan's first stage, or the tile's phase, as in kernel 3 (the nonzeros of
    // the XCD's earlier tiles over a.phase_wgs tiles' mean, mod 1), then the
    // stage that holds this fraction of the tile's own work, a stage counting
    // as kListStageWork entries beside those it holds.
    int32_t q = SUPER ? static_cast<int32_t>(tc >> 11 & 0x3ffu) : 0;
    if (!SUPER && a.rotate && nst > 1) {
      const int64_t first = static_cast<int64_t>(blockIdx.x % kXcds) * per_xcd;
      const int64_t end = first + per_xcd < a.ntiles ? first + per_xcd : a.ntiles;
      const uint64_t o_first = offset(first);
      const uint64_t work = offset(end) - o_first;                 // > 0
      const uint64_t den = static_cast<uint64_t>(a.phase_wgs) * work;
      const uint64_t num = (static_cast<uint64_t>(cap0) - o_first) * static_cast<uint64_t>(end - first) % den;
      const uint64_t ph = (num << 20) / den;                       // phase in 2^-20
      const uint64_t total = 4ull * pt[nst * S] + static_cast<uint64_t>(kListStageWork) * nst;
      const uint64_t target = (ph * total) >> 20;
      int32_t hi = nst;                                            // largest q whose work is at most the target
      while (hi - q > 1) {
        const int32_t mid = (q + hi) >> 1;
        if (4ull * pt[mid * S] + static_cast<uint64_t>(kListStageWork) * mid <= target)
          q = mid;
        else
          hi = mid;
      }
      q = __builtin_amdgcn_readfirstlane(q);
    }
    const uint32_t ring0 = lds_offset(ring);
    const uint32_t wbase = ring0 + static_cast<uint32_t>(wave * 4096);
    // this lane's half loads rows wave*8 + 4*half + i of a stage, i = 0..3,
    // into slot rows (wave*4 + i)*2 + half (the plan's entries hold slot rows)
    const char* __restrict__ ids = reinterpret_cast<const char*>(data);
    const uint32_t idl = static_cast<uint32_t>(wave * 32 + (lane >> 5) * 16);
    constexpr uint32_t kStarts = S * 4;   // bytes of list starts per stage
    auto load_ids = [&](uint32_t sb) { return *reinterpret_cast<const i32x4v*>(ids + (sb * (R * 4 / kStarts) + idl)); };
    const uint32_t ldw_lo = static_cast<uint32_t>(ldw_b);
    auto issue = [&](const i32x4v& id, uint32_t slot) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        dma_b128(Wl + static_cast<uint64_t>(static_cast<uint32_t>(id[i])) * (WIDE ? ldw_b : static_cast<uint64_t>(ldw_lo)),
                 wbase + slot + static_cast<uint32_t>(i * 1024));
    };
    typedef uint32_t u32x2v __attribute__((ext_vector_type(2)));
    const const_char starts = (const_char)(pt + wave);
    auto load_range = [&](uint32_t sb) { return *(const __attribute__((address_space(4))) u32x2v*)(starts + sb); };
    const uint32_t end = static_cast<uint32_t>(nst) * kStarts;
    const uint32_t vend = static_cast<uint32_t>(visits) * kStarts;
    auto after = [&](uint32_t sb) { return sb + kStarts == end ? 0u : sb + kStarts; };
    auto after_visit = [&](uint32_t vb) { return vb + kStarts == vend ? 0u : vb + kStarts; };   // (SUPER)

    // offsets in the list starts, of a stage (for its ids) and of a visit: the
    // next one's, and the one after (past the last visit: loaded, not used)
    uint32_t sb = static_cast<uint32_t>(q) * kStarts;
    uint32_t vb = SUPER ? 0u : sb;
    i32x4v id = load_ids(sb);
    issue(id, 0);
    u32x2v cur = load_range(vb);
    u32x8v set = *(const __attribute__((address_space(4))) u32x8v*)(lists + cur.x * 8u);
    sb = after(sb);
    vb = SUPER ? after_visit(vb) : sb;
    id = load_ids(sb);
    u32x2v next = load_range(vb);
    const uint32_t vl0 = ring0 | static_cast<uint32_t>(lane * 8);
    const uint32_t vm = 0xfe00u;
    const uint64_t lb = reinterpret_cast<uint64_t>((const char*)lists);
    uint32_t sbc = static_cast<uint32_t>(q) * kStarts;   // the current stage
    // `more`: a stage follows (its loads are issued); `none`: no stage at all,
    // the filler of an odd count
    auto step = [&](auto odd, bool more, bool none) {
      constexpr bool ODD = decltype(odd)::value;
      constexpr uint32_t slot = ODD ? kSlot : 0;
      // this wave's rows of the stage (and its ids of the next) have landed;
      // the builtin (vmcnt(0), the other counters untouched) tells the compiler
      // so about the ids, whose own wait would otherwise fall after the issue
      // below and drain it
      __builtin_amdgcn_s_waitcnt(0x0f70);
      lds_barrier();  // the stage is visible to all waves; every wave is done with the stage before
      if (more) issue(id, kSlot - slot);
      sb = after(sb);
      vb = SUPER ? after_visit(vb) : sb;
      id = load_ids(sb);
      const u32x2v next2 = load_range(vb);
      if constexpr (DW == 32 && !SUPER)
        if (nd && sbc == 0 && !none)
          add_dense<WT, NPL>(acc, ring, slot + lane * 8, nd, masks + wave * DW * 8, lane);
      sbc = after(sbc);
      const uint32_t n = none ? ~0u : cur.y - cur.x - 1u;
      set = add_list<ODD>(acc, set, lb, cur.x * 8u, next.x * 8u, n, vl0 | slot, vm);
      cur = next;
      next = next2;
    };
    for (int32_t left = visits; left > 0; left -= 2) {   // visits from this one on
      step(std::false_type{}, left > 1, false);
      step(std::true_type{}, left > 2, left == 1);
    }
  }
  list_epilogue<DW, NPL, TOP2>(a, acc, t * (S * DW) + wave * DW, n0, lane);
}

template <typename WT, int DW, bool TOP2, bool WIDE>
void launch_list_grid(const SearchArgs& a, dim3 grid, hipStream_t stream) {
  if constexpr (DW == 32) {
    if (a.rotate == 2) {
      grid.x = static_cast<uint32_t>(a.ntiles);
      hipLaunchKernelGGL((k_search_list<WT, DW, TOP2, WIDE, true>), grid, dim3(kListWaves * 64), 0, stream, a);
      return;
    }
  }
  hipLaunchKernelGGL((k_search_list<WT, DW, TOP2, WIDE, false>), grid, dim3(kListWaves * 64), 0, stream, a);
}

template <typename WT, int DW>
hipError_t launch_list(const SearchArgs& a, hipStream_t stream) {
  // grid.y holds at most 65,535 slices: wider maps take several launches
  constexpr int64_t WN = 64 * kListRowBytes / 64 / static_cast<int64_t>(sizeof(WT));
  const int64_t slices = (a.N + WN - 1) / WN;
  const bool wide = static_cast<uint64_t>(a.ldw) * sizeof(WT) >> 32;
  SearchArgs b = a;
  b.phase_wgs = kListPhaseWgs;
  for (int64_t c = 0; c < slices; c += 65535) {
    b.slice_base = c;
    const dim3 grid(static_cast<uint32_t>((a.ntiles + kXcds - 1) / kXcds * kXcds),
                    static_cast<uint32_t>(slices - c < 65535 ? slices - c : 65535));
    if (wide && a.keys2)
      launch_list_grid<WT, DW, true, true>(b, grid, stream);
    else if (wide)
      launch_list_grid<WT, DW, false, true>(b, grid, stream);
    else if (a.keys2)
      launch_list_grid<WT, DW, true, false>(b, grid, stream);
    else
      launch_list_grid<WT, DW, false, false>(b, grid, stream);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

}  // namespace
}  // namespace som
