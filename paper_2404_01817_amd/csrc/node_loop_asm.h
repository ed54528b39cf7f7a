// node_loop_asm.h -- GENERATED by gen_node_loop.py; edit that script.
//
// One tile of the calculation stage (Section 3.3) in gfx950 assembly, for
// one wave with one or two samples per lane: for every computed node in
// topological order, v[dst] = act(bias + response * agg(w * v[src])).
//
// A tile block (NEAT_TILE_<variant>) does, in order:
//   1. v[i] = input i of the lane's sample(s), i < %[ni], from the LDS
//      staging area at byte address %[dm0] (sample s's inputs at + 4 s ni;
//      lane l holds samples l, 64 + l, ...: one per sample of the lane); then the
//      constants 0 and 1 at slots %[zs], %[zs] + 1;
//   2. the DMA of the next tile's inputs into the staging area: %[dn]
//      pieces of 16 bytes (%[dvec] = 1) or 4 bytes (%[dvec] = 0) from the
//      global address %[dsrc] onward, lane l taking piece l of each round
//      of 64; %[lane] is the lane id (the only VGPR operand);
//   3. the node loop over the records from %[rec] up to the sentinel record
//      that follows the last node, overflow edges from %[edg];
//   4. output j of each sample s = v[slot j] (slots at %[outs], j < %[no])
//      to the LDS output area at %[om0] + 4 (s O + j).
// The value vectors (slot s of sample h in v[base_h + s]; every slot the
// program names is below the variant's slot count) live only inside the
// block and are listed as clobbers with the scratch VGPRs after them.
//
// Scalar registers: s40..s55 record buffer A, s56..s71 record buffer B
// (16-word records with the node's first three edge pairs; the next record
// is prefetched while the current one runs), s72..s79 two overflow pairs
// (the first two requested at the start of the node), s80:81 record array,
// s82:83 overflow read pointer, s84:85 overflow edges of the current node,
// s86 record byte offset, s87 pairs left, s88:89 jump target and scratch,
// s90 saved M0, s92:93 and s94:95 the two copies' activation blocks; steps
// 1, 2 and 4 use s40..s55 before and after the node loop.
// Reads of v[slot] and the write of v[dst] use GPR-index mode with the
// program's uniform slots; an indexed read of a pair keeps the mode on and
// only moves the index, and every sample of the lane shares it.
//
// Aggregation classes (program.h): sum (mean folds 1/degree into the
// response), product, max (min is max over negated weights with negated
// response), the first pair initialising the accumulator and an empty sum
// giving 0.  Max uses the NaN-propagating maximum.  Activations: one block
// per code, entered by a computed jump (blocks aligned to a fixed stride):
// identity; relu maximum(z, 0) and abs maximum(z, -z); sigmoid, tanh and
// gaussian on the hardware base-2 exponential and reciprocal; sin by
// Cody-Waite reduction and Taylor polynomials.  Each block ends with the
// write of v[dst] and the jump to the next node.  The C++ node loop of the
// LDS store performs the same operations in the same order.
//
// The recurrent blocks (NEAT_TILE_S1_64R here, _S2_32R and _S1_52R in
// node_loop_wide.h) zero the read vectors (v0..v63 here), place the inputs and
// constants in them and in the write vectors (v64..v127), then run the node
// loop %[nsw] times: every sweep reads the first and writes the second, and all
// but the last copy the %[n] + %[ni] nodes' slots back (s91 counts the sweeps);
// the outputs are read from the write vectors.
//
// Hazards: a transcendental's result is read no sooner than one instruction
// later (with two samples the other sample's instruction sits between); a
// write of M0 is followed by one wait state before the LDS DMA reads it.
#pragma once

// S1_64: 1 sample(s) per lane, value vectors at v0, scratch v64..v75

#define NEAT_TILE_S1_64 \
    "  s_mov_b32 s90, m0\n" \
    "  s_lshl_b32 s41, %[ni], 2\n" \
    "  v_mul_u32_u24_e32 v72, s41, %[lane]\n" \
    "  v_add_u32_e32 v72, %[dm0], v72\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_cmp_eq_u32 %[ni], 0\n" \
    "  s_cbranch_scc1 Lpl_done%=\n" \
    "Lpl%=:\n" \
    "  ds_read2_b32 v[64:65], v72 offset0:0 offset1:1\n" \
    "  ds_read2_b32 v[66:67], v72 offset0:2 offset1:3\n" \
    "  ds_read2_b32 v[68:69], v72 offset0:4 offset1:5\n" \
    "  ds_read2_b32 v[70:71], v72 offset0:6 offset1:7\n" \
    "  v_add_u32_e32 v72, 32, v72\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v64\n" \
    "  v_mov_b32_e32 v1, v65\n" \
    "  v_mov_b32_e32 v2, v66\n" \
    "  v_mov_b32_e32 v3, v67\n" \
    "  v_mov_b32_e32 v4, v68\n" \
    "  v_mov_b32_e32 v5, v69\n" \
    "  v_mov_b32_e32 v6, v70\n" \
    "  v_mov_b32_e32 v7, v71\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_add_u32 s40, s40, 8\n" \
    "  s_cmp_lt_u32 s40, %[ni]\n" \
    "  s_cbranch_scc1 Lpl%=\n" \
    "Lpl_done%=:\n" \
    "  s_set_gpr_idx_on %[zs], gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, 0\n" \
    "  v_mov_b32_e32 v1, 1.0\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 %[dn], 0\n" \
    "  s_cbranch_scc1 Ldma_done%=\n" \
    "  s_mov_b64 s[42:43], exec\n" \
    "  s_cmp_eq_u32 %[dvec], 0\n" \
    "  s_cselect_b32 s41, 2, 4\n" \
    "  v_lshlrev_b32_e32 v74, s41, %[lane]\n" \
    "  v_mov_b32_e32 v75, 0\n" \
    "  v_lshl_add_u64 v[74:75], v[74:75], 0, %[dsrc]\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_mov_b32 m0, %[dm0]\n" \
    "  s_cmp_eq_u32 %[dvec], 0\n" \
    "  s_cbranch_scc1 Ldma1%=\n" \
    "  s_mov_b64 s[46:47], 1024\n" \
    "Ldl4%=:\n" \
    "  s_sub_u32 s41, %[dn], s40\n" \
    "  v_cmp_gt_u32_e64 s[44:45], s41, %[lane]\n" \
    "  s_and_b64 exec, s[42:43], s[44:45]\n" \
    "  s_nop 0\n" \
    "  global_load_lds_dwordx4 v[74:75], off nt\n" \
    "  s_mov_b64 exec, s[42:43]\n" \
    "  v_lshl_add_u64 v[74:75], v[74:75], 0, s[46:47]\n" \
    "  s_add_u32 m0, m0, 1024\n" \
    "  s_add_u32 s40, s40, 64\n" \
    "  s_cmp_lt_u32 s40, %[dn]\n" \
    "  s_cbranch_scc1 Ldl4%=\n" \
    "  s_branch Ldma_done%=\n" \
    "Ldma1%=:\n" \
    "  s_mov_b64 s[46:47], 256\n" \
    "Ldl1%=:\n" \
    "  s_sub_u32 s41, %[dn], s40\n" \
    "  v_cmp_gt_u32_e64 s[44:45], s41, %[lane]\n" \
    "  s_and_b64 exec, s[42:43], s[44:45]\n" \
    "  s_nop 0\n" \
    "  global_load_lds_dword v[74:75], off nt\n" \
    "  s_mov_b64 exec, s[42:43]\n" \
    "  v_lshl_add_u64 v[74:75], v[74:75], 0, s[46:47]\n" \
    "  s_add_u32 m0, m0, 256\n" \
    "  s_add_u32 s40, s40, 64\n" \
    "  s_cmp_lt_u32 s40, %[dn]\n" \
    "  s_cbranch_scc1 Ldl1%=\n" \
    "  s_branch Ldma_done%=\n" \
    "Ldma_done%=:\n" \
    "  s_mov_b64 s[80:81], %[rec]\n" \
    "  s_mov_b64 s[84:85], %[edg]\n" \
    "  s_mov_b32 s86, 0\n" \
    "  v_mov_b32_e32 v68, 0x2f309231\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], 0x0\n" \
    "  s_getpc_b64 s[92:93]\n" \
    "Lpc%=:\n" \
    "  s_add_u32 s94, s92, Ltab_B%= - Lpc%=\n" \
    "  s_addc_u32 s95, s93, 0\n" \
    "  s_add_u32 s92, s92, Ltab_A%= - Lpc%=\n" \
    "  s_addc_u32 s93, s93, 0\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "Ltab_A%=:\n" \
    "  v_mov_b32_e32 v67, s41\n" \
    "  v_fmac_f32_e64 v67, s42, v64\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v67\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v67, s41\n" \
    "  v_fmac_f32_e64 v67, s42, v64\n" \
    "  v_mul_f32_e32 v65, 0x4038aa3b, v67\n" \
    "  v_exp_f32_e32 v65, v65\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v66, 1.0, v65\n" \
    "  v_rcp_f32_e32 v66, v66\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v65, v66, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v67, s41\n" \
    "  v_fmac_f32_e64 v67, s42, v64\n" \
    "  v_mul_f32_e32 v65, 0xbfb8aa3b, v67\n" \
    "  v_exp_f32_e32 v65, v65\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v66, 1.0, v65\n" \
    "  v_rcp_f32_e32 v65, v66\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v67, s41\n" \
    "  v_fmac_f32_e64 v67, s42, v64\n" \
    "  v_maximum3_f32 v65, v67, 0, 0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v67, s41\n" \
    "  v_fmac_f32_e64 v67, s42, v64\n" \
    "  v_mul_f32_e32 v66, 0x3ea2f983, v67\n" \
    "  v_rndne_f32_e32 v66, v66\n" \
    "  v_fmamk_f32 v64, v66, 0xc0490fdb, v67\n" \
    "  v_fmac_f32_e32 v64, 0x33bbbd2e, v66\n" \
    "  v_cvt_i32_f32_e32 v66, v66\n" \
    "  v_mul_f32_e32 v67, v64, v64\n" \
    "  v_fmaak_f32 v69, v67, v68, 0xb2d7322b\n" \
    "  v_fmaak_f32 v69, v67, v69, 0x3638ef1d\n" \
    "  v_fmaak_f32 v69, v67, v69, 0xb9500d01\n" \
    "  v_fmaak_f32 v69, v67, v69, 0x3c088889\n" \
    "  v_fmaak_f32 v69, v67, v69, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v65, v64, v67\n" \
    "  v_fmac_f32_e32 v64, v65, v69\n" \
    "  v_lshl_add_u32 v65, v66, 31, v64\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v67, s41\n" \
    "  v_fmac_f32_e64 v67, s42, v64\n" \
    "  v_mul_f32_e32 v65, v67, v67\n" \
    "  v_mul_f32_e32 v65, 0xbfb8aa3b, v65\n" \
    "  v_exp_f32_e32 v66, v65\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v66\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v67, s41\n" \
    "  v_fmac_f32_e64 v67, s42, v64\n" \
    "  v_maximum3_f32 v65, v67, -v67, -v67\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_branch Ldone%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  v_mov_b32_e32 v64, 0\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v64, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v64, v0, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v64, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v64, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v64, v0, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v64, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v64, v0, s51\n" \
    "  s_set_gpr_idx_idx s52\n" \
    "  v_fmac_f32_e64 v64, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_fmac_f32_e64 v64, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v64, v0, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v64, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v64, v0, s51\n" \
    "  s_set_gpr_idx_idx s52\n" \
    "  v_fmac_f32_e64 v64, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_fmac_f32_e64 v64, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_branch Lovs_A%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v66, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v66, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v66, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v65\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v66, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v66, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v65\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v66, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v65\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v66, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v66, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v65\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v66, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v65\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_branch Lovp_A%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v66, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v65, v66, v66\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v66, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v65, v66, v66\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v66, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v64, v65, v66\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v66, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v65, v66, v66\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v66, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v64, v65, v66\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v66, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v64, v65, v66\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v66, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v65, v66, v66\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v66, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v64, v65, v66\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v66, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v64, v65, v66\n" \
    "  s_branch Lovm_A%=\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v67, s41, v64\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v67\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v67, s41, v64\n" \
    "  v_mul_f32_e32 v65, 0x4038aa3b, v67\n" \
    "  v_exp_f32_e32 v65, v65\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v66, 1.0, v65\n" \
    "  v_rcp_f32_e32 v66, v66\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v65, v66, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v67, s41, v64\n" \
    "  v_mul_f32_e32 v65, 0xbfb8aa3b, v67\n" \
    "  v_exp_f32_e32 v65, v65\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v66, 1.0, v65\n" \
    "  v_rcp_f32_e32 v65, v66\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v67, s41, v64\n" \
    "  v_maximum3_f32 v65, v67, 0, 0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v67, s41, v64\n" \
    "  v_mul_f32_e32 v66, 0x3ea2f983, v67\n" \
    "  v_rndne_f32_e32 v66, v66\n" \
    "  v_fmamk_f32 v64, v66, 0xc0490fdb, v67\n" \
    "  v_fmac_f32_e32 v64, 0x33bbbd2e, v66\n" \
    "  v_cvt_i32_f32_e32 v66, v66\n" \
    "  v_mul_f32_e32 v67, v64, v64\n" \
    "  v_fmaak_f32 v69, v67, v68, 0xb2d7322b\n" \
    "  v_fmaak_f32 v69, v67, v69, 0x3638ef1d\n" \
    "  v_fmaak_f32 v69, v67, v69, 0xb9500d01\n" \
    "  v_fmaak_f32 v69, v67, v69, 0x3c088889\n" \
    "  v_fmaak_f32 v69, v67, v69, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v65, v64, v67\n" \
    "  v_fmac_f32_e32 v64, v65, v69\n" \
    "  v_lshl_add_u32 v65, v66, 31, v64\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v67, s41, v64\n" \
    "  v_mul_f32_e32 v65, v67, v67\n" \
    "  v_mul_f32_e32 v65, 0xbfb8aa3b, v65\n" \
    "  v_exp_f32_e32 v66, v65\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v66\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v67, s41, v64\n" \
    "  v_maximum3_f32 v65, v67, -v67, -v67\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovs_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Los_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v64, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_fmac_f32_e64 v64, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovds_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v64, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_fmac_f32_e64 v64, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovds_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Los_A%=\n" \
    "Lovds_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovp_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lop_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v66, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v65\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdp_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v66, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v65\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdp_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lop_A%=\n" \
    "Lovdp_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovm_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lom_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v66, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v64, v65, v66\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdm_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v66, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v64, v65, v66\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdm_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lom_A%=\n" \
    "Lovdm_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "Ltab_B%=:\n" \
    "  v_mov_b32_e32 v67, s57\n" \
    "  v_fmac_f32_e64 v67, s58, v64\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v67\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v67, s57\n" \
    "  v_fmac_f32_e64 v67, s58, v64\n" \
    "  v_mul_f32_e32 v65, 0x4038aa3b, v67\n" \
    "  v_exp_f32_e32 v65, v65\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v66, 1.0, v65\n" \
    "  v_rcp_f32_e32 v66, v66\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v65, v66, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v67, s57\n" \
    "  v_fmac_f32_e64 v67, s58, v64\n" \
    "  v_mul_f32_e32 v65, 0xbfb8aa3b, v67\n" \
    "  v_exp_f32_e32 v65, v65\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v66, 1.0, v65\n" \
    "  v_rcp_f32_e32 v65, v66\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v67, s57\n" \
    "  v_fmac_f32_e64 v67, s58, v64\n" \
    "  v_maximum3_f32 v65, v67, 0, 0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v67, s57\n" \
    "  v_fmac_f32_e64 v67, s58, v64\n" \
    "  v_mul_f32_e32 v66, 0x3ea2f983, v67\n" \
    "  v_rndne_f32_e32 v66, v66\n" \
    "  v_fmamk_f32 v64, v66, 0xc0490fdb, v67\n" \
    "  v_fmac_f32_e32 v64, 0x33bbbd2e, v66\n" \
    "  v_cvt_i32_f32_e32 v66, v66\n" \
    "  v_mul_f32_e32 v67, v64, v64\n" \
    "  v_fmaak_f32 v69, v67, v68, 0xb2d7322b\n" \
    "  v_fmaak_f32 v69, v67, v69, 0x3638ef1d\n" \
    "  v_fmaak_f32 v69, v67, v69, 0xb9500d01\n" \
    "  v_fmaak_f32 v69, v67, v69, 0x3c088889\n" \
    "  v_fmaak_f32 v69, v67, v69, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v65, v64, v67\n" \
    "  v_fmac_f32_e32 v64, v65, v69\n" \
    "  v_lshl_add_u32 v65, v66, 31, v64\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v67, s57\n" \
    "  v_fmac_f32_e64 v67, s58, v64\n" \
    "  v_mul_f32_e32 v65, v67, v67\n" \
    "  v_mul_f32_e32 v65, 0xbfb8aa3b, v65\n" \
    "  v_exp_f32_e32 v66, v65\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v66\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v67, s57\n" \
    "  v_fmac_f32_e64 v67, s58, v64\n" \
    "  v_maximum3_f32 v65, v67, -v67, -v67\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_branch Ldone%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  v_mov_b32_e32 v64, 0\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v64, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v64, v0, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v64, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v64, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v64, v0, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v64, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v64, v0, s67\n" \
    "  s_set_gpr_idx_idx s68\n" \
    "  v_fmac_f32_e64 v64, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_fmac_f32_e64 v64, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v64, v0, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v64, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v64, v0, s67\n" \
    "  s_set_gpr_idx_idx s68\n" \
    "  v_fmac_f32_e64 v64, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_fmac_f32_e64 v64, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_branch Lovs_B%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v66, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v66, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v66, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v65\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v66, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v66, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v65\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v66, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v65\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v64, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v66, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v66, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v65\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v66, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v65\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_branch Lovp_B%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v66, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v65, v66, v66\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v66, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v65, v66, v66\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v66, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v64, v65, v66\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v66, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v65, v66, v66\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v66, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v64, v65, v66\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v66, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v64, v65, v66\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v66, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v65, v66, v66\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v66, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v64, v65, v66\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v66, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v64, v65, v66\n" \
    "  s_branch Lovm_B%=\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v67, s57, v64\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v67\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v67, s57, v64\n" \
    "  v_mul_f32_e32 v65, 0x4038aa3b, v67\n" \
    "  v_exp_f32_e32 v65, v65\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v66, 1.0, v65\n" \
    "  v_rcp_f32_e32 v66, v66\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v65, v66, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v67, s57, v64\n" \
    "  v_mul_f32_e32 v65, 0xbfb8aa3b, v67\n" \
    "  v_exp_f32_e32 v65, v65\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v66, 1.0, v65\n" \
    "  v_rcp_f32_e32 v65, v66\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v67, s57, v64\n" \
    "  v_maximum3_f32 v65, v67, 0, 0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v67, s57, v64\n" \
    "  v_mul_f32_e32 v66, 0x3ea2f983, v67\n" \
    "  v_rndne_f32_e32 v66, v66\n" \
    "  v_fmamk_f32 v64, v66, 0xc0490fdb, v67\n" \
    "  v_fmac_f32_e32 v64, 0x33bbbd2e, v66\n" \
    "  v_cvt_i32_f32_e32 v66, v66\n" \
    "  v_mul_f32_e32 v67, v64, v64\n" \
    "  v_fmaak_f32 v69, v67, v68, 0xb2d7322b\n" \
    "  v_fmaak_f32 v69, v67, v69, 0x3638ef1d\n" \
    "  v_fmaak_f32 v69, v67, v69, 0xb9500d01\n" \
    "  v_fmaak_f32 v69, v67, v69, 0x3c088889\n" \
    "  v_fmaak_f32 v69, v67, v69, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v65, v64, v67\n" \
    "  v_fmac_f32_e32 v64, v65, v69\n" \
    "  v_lshl_add_u32 v65, v66, 31, v64\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v67, s57, v64\n" \
    "  v_mul_f32_e32 v65, v67, v67\n" \
    "  v_mul_f32_e32 v65, 0xbfb8aa3b, v65\n" \
    "  v_exp_f32_e32 v66, v65\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v66\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v67, s57, v64\n" \
    "  v_maximum3_f32 v65, v67, -v67, -v67\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v65\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovs_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Los_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v64, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_fmac_f32_e64 v64, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovds_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v64, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_fmac_f32_e64 v64, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovds_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Los_B%=\n" \
    "Lovds_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovp_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lop_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v66, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v65\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdp_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v66, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v64, v64, v65\n" \
    "  v_mul_f32_e32 v64, v64, v66\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdp_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lop_B%=\n" \
    "Lovdp_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovm_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lom_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v66, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v64, v65, v66\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdm_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v65, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v66, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v64, v64, v65, v66\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdm_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lom_B%=\n" \
    "Lovdm_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Ldone%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_mov_b64 s[44:45], %[outs]\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_lshl_b32 s41, %[no], 2\n" \
    "  v_mul_u32_u24_e32 v72, s41, %[lane]\n" \
    "  v_add_u32_e32 v72, %[om0], v72\n" \
    "Lout%=:\n" \
    "  s_load_dwordx8 s[48:55], s[44:45], 0x0\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v64, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v72, v64 offset:0\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s49, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v65, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v72, v65 offset:4\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s50, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v66, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v72, v66 offset:8\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s51, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v67, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v72, v67 offset:12\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v68, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v72, v68 offset:16\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s53, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v69, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v72, v69 offset:20\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s54, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v70, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v72, v70 offset:24\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s55, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v71, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v72, v71 offset:28\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  v_add_u32_e32 v72, 32, v72\n" \
    "  s_add_u32 s44, s44, 32\n" \
    "  s_addc_u32 s45, s45, 0\n" \
    "  s_branch Lout%=\n" \
    "Lout_done%=:\n" \
    "  s_mov_b32 m0, s90\n"

#define NEAT_CLOB_S1_64 \
    "v0", "v1", "v2", "v3", "v4", "v5", "v6", "v7", "v8", "v9", "v10", "v11", \
    "v12", "v13", "v14", "v15", "v16", "v17", "v18", "v19", "v20", "v21", "v22", "v23", \
    "v24", "v25", "v26", "v27", "v28", "v29", "v30", "v31", "v32", "v33", "v34", "v35", \
    "v36", "v37", "v38", "v39", "v40", "v41", "v42", "v43", "v44", "v45", "v46", "v47", \
    "v48", "v49", "v50", "v51", "v52", "v53", "v54", "v55", "v56", "v57", "v58", "v59", \
    "v60", "v61", "v62", "v63", "v64", "v65", "v66", "v67", "v68", "v69", "v70", "v71", \
    "v72", "v73", "v74", "v75", "s40", "s41", "s42", "s43", "s44", "s45", "s46", "s47", \
    "s48", "s49", "s50", "s51", "s52", "s53", "s54", "s55", "s56", "s57", "s58", "s59", \
    "s60", "s61", "s62", "s63", "s64", "s65", "s66", "s67", "s68", "s69", "s70", "s71", \
    "s72", "s73", "s74", "s75", "s76", "s77", "s78", "s79", "s80", "s81", "s82", "s83", \
    "s84", "s85", "s86", "s87", "s88", "s89", "s90", "s91", "s92", "s93", "s94", "s95", \
    "vcc", "scc"

#define NEAT_SCRATCH_S1_64 64


// S2_64: 2 sample(s) per lane, value vectors at v0, v64, scratch v128..v147

#define NEAT_TILE_S2_64 \
    "  s_mov_b32 s90, m0\n" \
    "  s_lshl_b32 s41, %[ni], 2\n" \
    "  v_mul_u32_u24_e32 v144, s41, %[lane]\n" \
    "  v_add_u32_e32 v144, %[dm0], v144\n" \
    "  s_lshl_b32 s41, %[ni], 8\n" \
    "  v_add_u32_e32 v145, s41, v144\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_cmp_eq_u32 %[ni], 0\n" \
    "  s_cbranch_scc1 Lpl_done%=\n" \
    "Lpl%=:\n" \
    "  ds_read2_b32 v[128:129], v144 offset0:0 offset1:1\n" \
    "  ds_read2_b32 v[130:131], v144 offset0:2 offset1:3\n" \
    "  ds_read2_b32 v[132:133], v144 offset0:4 offset1:5\n" \
    "  ds_read2_b32 v[134:135], v144 offset0:6 offset1:7\n" \
    "  ds_read2_b32 v[136:137], v145 offset0:0 offset1:1\n" \
    "  ds_read2_b32 v[138:139], v145 offset0:2 offset1:3\n" \
    "  ds_read2_b32 v[140:141], v145 offset0:4 offset1:5\n" \
    "  ds_read2_b32 v[142:143], v145 offset0:6 offset1:7\n" \
    "  v_add_u32_e32 v144, 32, v144\n" \
    "  v_add_u32_e32 v145, 32, v145\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v128\n" \
    "  v_mov_b32_e32 v1, v129\n" \
    "  v_mov_b32_e32 v2, v130\n" \
    "  v_mov_b32_e32 v3, v131\n" \
    "  v_mov_b32_e32 v4, v132\n" \
    "  v_mov_b32_e32 v5, v133\n" \
    "  v_mov_b32_e32 v6, v134\n" \
    "  v_mov_b32_e32 v7, v135\n" \
    "  v_mov_b32_e32 v64, v136\n" \
    "  v_mov_b32_e32 v65, v137\n" \
    "  v_mov_b32_e32 v66, v138\n" \
    "  v_mov_b32_e32 v67, v139\n" \
    "  v_mov_b32_e32 v68, v140\n" \
    "  v_mov_b32_e32 v69, v141\n" \
    "  v_mov_b32_e32 v70, v142\n" \
    "  v_mov_b32_e32 v71, v143\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_add_u32 s40, s40, 8\n" \
    "  s_cmp_lt_u32 s40, %[ni]\n" \
    "  s_cbranch_scc1 Lpl%=\n" \
    "Lpl_done%=:\n" \
    "  s_set_gpr_idx_on %[zs], gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, 0\n" \
    "  v_mov_b32_e32 v1, 1.0\n" \
    "  v_mov_b32_e32 v64, 0\n" \
    "  v_mov_b32_e32 v65, 1.0\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 %[dn], 0\n" \
    "  s_cbranch_scc1 Ldma_done%=\n" \
    "  s_mov_b64 s[42:43], exec\n" \
    "  s_cmp_eq_u32 %[dvec], 0\n" \
    "  s_cselect_b32 s41, 2, 4\n" \
    "  v_lshlrev_b32_e32 v146, s41, %[lane]\n" \
    "  v_mov_b32_e32 v147, 0\n" \
    "  v_lshl_add_u64 v[146:147], v[146:147], 0, %[dsrc]\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_mov_b32 m0, %[dm0]\n" \
    "  s_cmp_eq_u32 %[dvec], 0\n" \
    "  s_cbranch_scc1 Ldma1%=\n" \
    "  s_mov_b64 s[46:47], 1024\n" \
    "Ldl4%=:\n" \
    "  s_sub_u32 s41, %[dn], s40\n" \
    "  v_cmp_gt_u32_e64 s[44:45], s41, %[lane]\n" \
    "  s_and_b64 exec, s[42:43], s[44:45]\n" \
    "  s_nop 0\n" \
    "  global_load_lds_dwordx4 v[146:147], off nt\n" \
    "  s_mov_b64 exec, s[42:43]\n" \
    "  v_lshl_add_u64 v[146:147], v[146:147], 0, s[46:47]\n" \
    "  s_add_u32 m0, m0, 1024\n" \
    "  s_add_u32 s40, s40, 64\n" \
    "  s_cmp_lt_u32 s40, %[dn]\n" \
    "  s_cbranch_scc1 Ldl4%=\n" \
    "  s_branch Ldma_done%=\n" \
    "Ldma1%=:\n" \
    "  s_mov_b64 s[46:47], 256\n" \
    "Ldl1%=:\n" \
    "  s_sub_u32 s41, %[dn], s40\n" \
    "  v_cmp_gt_u32_e64 s[44:45], s41, %[lane]\n" \
    "  s_and_b64 exec, s[42:43], s[44:45]\n" \
    "  s_nop 0\n" \
    "  global_load_lds_dword v[146:147], off nt\n" \
    "  s_mov_b64 exec, s[42:43]\n" \
    "  v_lshl_add_u64 v[146:147], v[146:147], 0, s[46:47]\n" \
    "  s_add_u32 m0, m0, 256\n" \
    "  s_add_u32 s40, s40, 64\n" \
    "  s_cmp_lt_u32 s40, %[dn]\n" \
    "  s_cbranch_scc1 Ldl1%=\n" \
    "  s_branch Ldma_done%=\n" \
    "Ldma_done%=:\n" \
    "  s_mov_b64 s[80:81], %[rec]\n" \
    "  s_mov_b64 s[84:85], %[edg]\n" \
    "  s_mov_b32 s86, 0\n" \
    "  v_mov_b32_e32 v136, 0x2f309231\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], 0x0\n" \
    "  s_getpc_b64 s[92:93]\n" \
    "Lpc%=:\n" \
    "  s_add_u32 s94, s92, Ltab_B%= - Lpc%=\n" \
    "  s_addc_u32 s95, s93, 0\n" \
    "  s_add_u32 s92, s92, Ltab_A%= - Lpc%=\n" \
    "  s_addc_u32 s93, s93, 0\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "Ltab_A%=:\n" \
    "  v_mov_b32_e32 v134, s41\n" \
    "  v_mov_b32_e32 v135, s41\n" \
    "  v_fmac_f32_e64 v134, s42, v128\n" \
    "  v_fmac_f32_e64 v135, s42, v129\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v134\n" \
    "  v_mov_b32_e32 v64, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v134, s41\n" \
    "  v_mov_b32_e32 v135, s41\n" \
    "  v_fmac_f32_e64 v134, s42, v128\n" \
    "  v_fmac_f32_e64 v135, s42, v129\n" \
    "  v_mul_f32_e32 v130, 0x4038aa3b, v134\n" \
    "  v_mul_f32_e32 v131, 0x4038aa3b, v135\n" \
    "  v_exp_f32_e32 v130, v130\n" \
    "  v_exp_f32_e32 v131, v131\n" \
    "  v_add_f32_e32 v132, 1.0, v130\n" \
    "  v_add_f32_e32 v133, 1.0, v131\n" \
    "  v_rcp_f32_e32 v132, v132\n" \
    "  v_rcp_f32_e32 v133, v133\n" \
    "  v_fma_f32 v130, v132, -2.0, 1.0\n" \
    "  v_fma_f32 v131, v133, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v134, s41\n" \
    "  v_mov_b32_e32 v135, s41\n" \
    "  v_fmac_f32_e64 v134, s42, v128\n" \
    "  v_fmac_f32_e64 v135, s42, v129\n" \
    "  v_mul_f32_e32 v130, 0xbfb8aa3b, v134\n" \
    "  v_mul_f32_e32 v131, 0xbfb8aa3b, v135\n" \
    "  v_exp_f32_e32 v130, v130\n" \
    "  v_exp_f32_e32 v131, v131\n" \
    "  v_add_f32_e32 v132, 1.0, v130\n" \
    "  v_add_f32_e32 v133, 1.0, v131\n" \
    "  v_rcp_f32_e32 v130, v132\n" \
    "  v_rcp_f32_e32 v131, v133\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v134, s41\n" \
    "  v_mov_b32_e32 v135, s41\n" \
    "  v_fmac_f32_e64 v134, s42, v128\n" \
    "  v_fmac_f32_e64 v135, s42, v129\n" \
    "  v_maximum3_f32 v130, v134, 0, 0\n" \
    "  v_maximum3_f32 v131, v135, 0, 0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v134, s41\n" \
    "  v_mov_b32_e32 v135, s41\n" \
    "  v_fmac_f32_e64 v134, s42, v128\n" \
    "  v_fmac_f32_e64 v135, s42, v129\n" \
    "  v_mul_f32_e32 v132, 0x3ea2f983, v134\n" \
    "  v_mul_f32_e32 v133, 0x3ea2f983, v135\n" \
    "  v_rndne_f32_e32 v132, v132\n" \
    "  v_rndne_f32_e32 v133, v133\n" \
    "  v_fmamk_f32 v128, v132, 0xc0490fdb, v134\n" \
    "  v_fmamk_f32 v129, v133, 0xc0490fdb, v135\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v132\n" \
    "  v_fmac_f32_e32 v129, 0x33bbbd2e, v133\n" \
    "  v_cvt_i32_f32_e32 v132, v132\n" \
    "  v_cvt_i32_f32_e32 v133, v133\n" \
    "  v_mul_f32_e32 v134, v128, v128\n" \
    "  v_mul_f32_e32 v135, v129, v129\n" \
    "  v_fmaak_f32 v137, v134, v136, 0xb2d7322b\n" \
    "  v_fmaak_f32 v138, v135, v136, 0xb2d7322b\n" \
    "  v_fmaak_f32 v137, v134, v137, 0x3638ef1d\n" \
    "  v_fmaak_f32 v138, v135, v138, 0x3638ef1d\n" \
    "  v_fmaak_f32 v137, v134, v137, 0xb9500d01\n" \
    "  v_fmaak_f32 v138, v135, v138, 0xb9500d01\n" \
    "  v_fmaak_f32 v137, v134, v137, 0x3c088889\n" \
    "  v_fmaak_f32 v138, v135, v138, 0x3c088889\n" \
    "  v_fmaak_f32 v137, v134, v137, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v138, v135, v138, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v130, v128, v134\n" \
    "  v_mul_f32_e32 v131, v129, v135\n" \
    "  v_fmac_f32_e32 v128, v130, v137\n" \
    "  v_fmac_f32_e32 v129, v131, v138\n" \
    "  v_lshl_add_u32 v130, v132, 31, v128\n" \
    "  v_lshl_add_u32 v131, v133, 31, v129\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v134, s41\n" \
    "  v_mov_b32_e32 v135, s41\n" \
    "  v_fmac_f32_e64 v134, s42, v128\n" \
    "  v_fmac_f32_e64 v135, s42, v129\n" \
    "  v_mul_f32_e32 v130, v134, v134\n" \
    "  v_mul_f32_e32 v131, v135, v135\n" \
    "  v_mul_f32_e32 v130, 0xbfb8aa3b, v130\n" \
    "  v_mul_f32_e32 v131, 0xbfb8aa3b, v131\n" \
    "  v_exp_f32_e32 v132, v130\n" \
    "  v_exp_f32_e32 v133, v131\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v64, v133\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v134, s41\n" \
    "  v_mov_b32_e32 v135, s41\n" \
    "  v_fmac_f32_e64 v134, s42, v128\n" \
    "  v_fmac_f32_e64 v135, s42, v129\n" \
    "  v_maximum3_f32 v130, v134, -v134, -v134\n" \
    "  v_maximum3_f32 v131, v135, -v135, -v135\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_branch Ldone%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  v_mov_b32_e32 v128, 0\n" \
    "  v_mov_b32_e32 v129, 0\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v64, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  v_fmac_f32_e64 v129, v64, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v64, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  v_fmac_f32_e64 v129, v64, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v128, v0, s49\n" \
    "  v_fmac_f32_e64 v129, v64, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v128, v0, s51\n" \
    "  v_fmac_f32_e64 v129, v64, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v64, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  v_fmac_f32_e64 v129, v64, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v128, v0, s49\n" \
    "  v_fmac_f32_e64 v129, v64, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v128, v0, s51\n" \
    "  v_fmac_f32_e64 v129, v64, s51\n" \
    "  s_set_gpr_idx_idx s52\n" \
    "  v_fmac_f32_e64 v128, v0, s53\n" \
    "  v_fmac_f32_e64 v129, v64, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_fmac_f32_e64 v128, v0, s55\n" \
    "  v_fmac_f32_e64 v129, v64, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v64, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  v_fmac_f32_e64 v129, v64, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v128, v0, s49\n" \
    "  v_fmac_f32_e64 v129, v64, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v128, v0, s51\n" \
    "  v_fmac_f32_e64 v129, v64, s51\n" \
    "  s_set_gpr_idx_idx s52\n" \
    "  v_fmac_f32_e64 v128, v0, s53\n" \
    "  v_fmac_f32_e64 v129, v64, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_fmac_f32_e64 v128, v0, s55\n" \
    "  v_fmac_f32_e64 v129, v64, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_branch Lovs_A%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v64, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v132, v0, s47\n" \
    "  v_mul_f32_e64 v133, v64, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v64, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v132, v0, s47\n" \
    "  v_mul_f32_e64 v133, v64, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s49\n" \
    "  v_mul_f32_e64 v131, v64, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v132, v0, s51\n" \
    "  v_mul_f32_e64 v133, v64, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  v_mul_f32_e32 v129, v129, v131\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v64, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v132, v0, s47\n" \
    "  v_mul_f32_e64 v133, v64, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s49\n" \
    "  v_mul_f32_e64 v131, v64, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v132, v0, s51\n" \
    "  v_mul_f32_e64 v133, v64, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  v_mul_f32_e32 v129, v129, v131\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s53\n" \
    "  v_mul_f32_e64 v131, v64, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v132, v0, s55\n" \
    "  v_mul_f32_e64 v133, v64, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  v_mul_f32_e32 v129, v129, v131\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v64, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v132, v0, s47\n" \
    "  v_mul_f32_e64 v133, v64, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s49\n" \
    "  v_mul_f32_e64 v131, v64, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v132, v0, s51\n" \
    "  v_mul_f32_e64 v133, v64, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  v_mul_f32_e32 v129, v129, v131\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s53\n" \
    "  v_mul_f32_e64 v131, v64, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v132, v0, s55\n" \
    "  v_mul_f32_e64 v133, v64, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  v_mul_f32_e32 v129, v129, v131\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_branch Lovp_A%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s45\n" \
    "  v_mul_f32_e64 v131, v64, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v132, v0, s47\n" \
    "  v_mul_f32_e64 v133, v64, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v130, v132, v132\n" \
    "  v_maximum3_f32 v129, v131, v133, v133\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s45\n" \
    "  v_mul_f32_e64 v131, v64, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v132, v0, s47\n" \
    "  v_mul_f32_e64 v133, v64, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v130, v132, v132\n" \
    "  v_maximum3_f32 v129, v131, v133, v133\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s49\n" \
    "  v_mul_f32_e64 v131, v64, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v132, v0, s51\n" \
    "  v_mul_f32_e64 v133, v64, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v130, v132\n" \
    "  v_maximum3_f32 v129, v129, v131, v133\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s45\n" \
    "  v_mul_f32_e64 v131, v64, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v132, v0, s47\n" \
    "  v_mul_f32_e64 v133, v64, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v130, v132, v132\n" \
    "  v_maximum3_f32 v129, v131, v133, v133\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s49\n" \
    "  v_mul_f32_e64 v131, v64, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v132, v0, s51\n" \
    "  v_mul_f32_e64 v133, v64, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v130, v132\n" \
    "  v_maximum3_f32 v129, v129, v131, v133\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s53\n" \
    "  v_mul_f32_e64 v131, v64, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v132, v0, s55\n" \
    "  v_mul_f32_e64 v133, v64, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v130, v132\n" \
    "  v_maximum3_f32 v129, v129, v131, v133\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s45\n" \
    "  v_mul_f32_e64 v131, v64, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v132, v0, s47\n" \
    "  v_mul_f32_e64 v133, v64, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v130, v132, v132\n" \
    "  v_maximum3_f32 v129, v131, v133, v133\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s49\n" \
    "  v_mul_f32_e64 v131, v64, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v132, v0, s51\n" \
    "  v_mul_f32_e64 v133, v64, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v130, v132\n" \
    "  v_maximum3_f32 v129, v129, v131, v133\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s53\n" \
    "  v_mul_f32_e64 v131, v64, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v132, v0, s55\n" \
    "  v_mul_f32_e64 v133, v64, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v130, v132\n" \
    "  v_maximum3_f32 v129, v129, v131, v133\n" \
    "  s_branch Lovm_A%=\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v134, s41, v128\n" \
    "  v_add_f32_e32 v135, s41, v129\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v134\n" \
    "  v_mov_b32_e32 v64, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v134, s41, v128\n" \
    "  v_add_f32_e32 v135, s41, v129\n" \
    "  v_mul_f32_e32 v130, 0x4038aa3b, v134\n" \
    "  v_mul_f32_e32 v131, 0x4038aa3b, v135\n" \
    "  v_exp_f32_e32 v130, v130\n" \
    "  v_exp_f32_e32 v131, v131\n" \
    "  v_add_f32_e32 v132, 1.0, v130\n" \
    "  v_add_f32_e32 v133, 1.0, v131\n" \
    "  v_rcp_f32_e32 v132, v132\n" \
    "  v_rcp_f32_e32 v133, v133\n" \
    "  v_fma_f32 v130, v132, -2.0, 1.0\n" \
    "  v_fma_f32 v131, v133, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v134, s41, v128\n" \
    "  v_add_f32_e32 v135, s41, v129\n" \
    "  v_mul_f32_e32 v130, 0xbfb8aa3b, v134\n" \
    "  v_mul_f32_e32 v131, 0xbfb8aa3b, v135\n" \
    "  v_exp_f32_e32 v130, v130\n" \
    "  v_exp_f32_e32 v131, v131\n" \
    "  v_add_f32_e32 v132, 1.0, v130\n" \
    "  v_add_f32_e32 v133, 1.0, v131\n" \
    "  v_rcp_f32_e32 v130, v132\n" \
    "  v_rcp_f32_e32 v131, v133\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v134, s41, v128\n" \
    "  v_add_f32_e32 v135, s41, v129\n" \
    "  v_maximum3_f32 v130, v134, 0, 0\n" \
    "  v_maximum3_f32 v131, v135, 0, 0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v134, s41, v128\n" \
    "  v_add_f32_e32 v135, s41, v129\n" \
    "  v_mul_f32_e32 v132, 0x3ea2f983, v134\n" \
    "  v_mul_f32_e32 v133, 0x3ea2f983, v135\n" \
    "  v_rndne_f32_e32 v132, v132\n" \
    "  v_rndne_f32_e32 v133, v133\n" \
    "  v_fmamk_f32 v128, v132, 0xc0490fdb, v134\n" \
    "  v_fmamk_f32 v129, v133, 0xc0490fdb, v135\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v132\n" \
    "  v_fmac_f32_e32 v129, 0x33bbbd2e, v133\n" \
    "  v_cvt_i32_f32_e32 v132, v132\n" \
    "  v_cvt_i32_f32_e32 v133, v133\n" \
    "  v_mul_f32_e32 v134, v128, v128\n" \
    "  v_mul_f32_e32 v135, v129, v129\n" \
    "  v_fmaak_f32 v137, v134, v136, 0xb2d7322b\n" \
    "  v_fmaak_f32 v138, v135, v136, 0xb2d7322b\n" \
    "  v_fmaak_f32 v137, v134, v137, 0x3638ef1d\n" \
    "  v_fmaak_f32 v138, v135, v138, 0x3638ef1d\n" \
    "  v_fmaak_f32 v137, v134, v137, 0xb9500d01\n" \
    "  v_fmaak_f32 v138, v135, v138, 0xb9500d01\n" \
    "  v_fmaak_f32 v137, v134, v137, 0x3c088889\n" \
    "  v_fmaak_f32 v138, v135, v138, 0x3c088889\n" \
    "  v_fmaak_f32 v137, v134, v137, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v138, v135, v138, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v130, v128, v134\n" \
    "  v_mul_f32_e32 v131, v129, v135\n" \
    "  v_fmac_f32_e32 v128, v130, v137\n" \
    "  v_fmac_f32_e32 v129, v131, v138\n" \
    "  v_lshl_add_u32 v130, v132, 31, v128\n" \
    "  v_lshl_add_u32 v131, v133, 31, v129\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v134, s41, v128\n" \
    "  v_add_f32_e32 v135, s41, v129\n" \
    "  v_mul_f32_e32 v130, v134, v134\n" \
    "  v_mul_f32_e32 v131, v135, v135\n" \
    "  v_mul_f32_e32 v130, 0xbfb8aa3b, v130\n" \
    "  v_mul_f32_e32 v131, 0xbfb8aa3b, v131\n" \
    "  v_exp_f32_e32 v132, v130\n" \
    "  v_exp_f32_e32 v133, v131\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v64, v133\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v134, s41, v128\n" \
    "  v_add_f32_e32 v135, s41, v129\n" \
    "  v_maximum3_f32 v130, v134, -v134, -v134\n" \
    "  v_maximum3_f32 v131, v135, -v135, -v135\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovs_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Los_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v128, v0, s73\n" \
    "  v_fmac_f32_e64 v129, v64, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_fmac_f32_e64 v128, v0, s75\n" \
    "  v_fmac_f32_e64 v129, v64, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovds_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v128, v0, s77\n" \
    "  v_fmac_f32_e64 v129, v64, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_fmac_f32_e64 v128, v0, s79\n" \
    "  v_fmac_f32_e64 v129, v64, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovds_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Los_A%=\n" \
    "Lovds_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovp_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lop_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s73\n" \
    "  v_mul_f32_e64 v131, v64, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v132, v0, s75\n" \
    "  v_mul_f32_e64 v133, v64, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  v_mul_f32_e32 v129, v129, v131\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdp_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s77\n" \
    "  v_mul_f32_e64 v131, v64, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v132, v0, s79\n" \
    "  v_mul_f32_e64 v133, v64, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  v_mul_f32_e32 v129, v129, v131\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdp_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lop_A%=\n" \
    "Lovdp_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovm_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lom_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s73\n" \
    "  v_mul_f32_e64 v131, v64, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v132, v0, s75\n" \
    "  v_mul_f32_e64 v133, v64, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v130, v132\n" \
    "  v_maximum3_f32 v129, v129, v131, v133\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdm_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s77\n" \
    "  v_mul_f32_e64 v131, v64, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v132, v0, s79\n" \
    "  v_mul_f32_e64 v133, v64, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v130, v132\n" \
    "  v_maximum3_f32 v129, v129, v131, v133\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdm_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lom_A%=\n" \
    "Lovdm_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "Ltab_B%=:\n" \
    "  v_mov_b32_e32 v134, s57\n" \
    "  v_mov_b32_e32 v135, s57\n" \
    "  v_fmac_f32_e64 v134, s58, v128\n" \
    "  v_fmac_f32_e64 v135, s58, v129\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v134\n" \
    "  v_mov_b32_e32 v64, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v134, s57\n" \
    "  v_mov_b32_e32 v135, s57\n" \
    "  v_fmac_f32_e64 v134, s58, v128\n" \
    "  v_fmac_f32_e64 v135, s58, v129\n" \
    "  v_mul_f32_e32 v130, 0x4038aa3b, v134\n" \
    "  v_mul_f32_e32 v131, 0x4038aa3b, v135\n" \
    "  v_exp_f32_e32 v130, v130\n" \
    "  v_exp_f32_e32 v131, v131\n" \
    "  v_add_f32_e32 v132, 1.0, v130\n" \
    "  v_add_f32_e32 v133, 1.0, v131\n" \
    "  v_rcp_f32_e32 v132, v132\n" \
    "  v_rcp_f32_e32 v133, v133\n" \
    "  v_fma_f32 v130, v132, -2.0, 1.0\n" \
    "  v_fma_f32 v131, v133, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v134, s57\n" \
    "  v_mov_b32_e32 v135, s57\n" \
    "  v_fmac_f32_e64 v134, s58, v128\n" \
    "  v_fmac_f32_e64 v135, s58, v129\n" \
    "  v_mul_f32_e32 v130, 0xbfb8aa3b, v134\n" \
    "  v_mul_f32_e32 v131, 0xbfb8aa3b, v135\n" \
    "  v_exp_f32_e32 v130, v130\n" \
    "  v_exp_f32_e32 v131, v131\n" \
    "  v_add_f32_e32 v132, 1.0, v130\n" \
    "  v_add_f32_e32 v133, 1.0, v131\n" \
    "  v_rcp_f32_e32 v130, v132\n" \
    "  v_rcp_f32_e32 v131, v133\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v134, s57\n" \
    "  v_mov_b32_e32 v135, s57\n" \
    "  v_fmac_f32_e64 v134, s58, v128\n" \
    "  v_fmac_f32_e64 v135, s58, v129\n" \
    "  v_maximum3_f32 v130, v134, 0, 0\n" \
    "  v_maximum3_f32 v131, v135, 0, 0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v134, s57\n" \
    "  v_mov_b32_e32 v135, s57\n" \
    "  v_fmac_f32_e64 v134, s58, v128\n" \
    "  v_fmac_f32_e64 v135, s58, v129\n" \
    "  v_mul_f32_e32 v132, 0x3ea2f983, v134\n" \
    "  v_mul_f32_e32 v133, 0x3ea2f983, v135\n" \
    "  v_rndne_f32_e32 v132, v132\n" \
    "  v_rndne_f32_e32 v133, v133\n" \
    "  v_fmamk_f32 v128, v132, 0xc0490fdb, v134\n" \
    "  v_fmamk_f32 v129, v133, 0xc0490fdb, v135\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v132\n" \
    "  v_fmac_f32_e32 v129, 0x33bbbd2e, v133\n" \
    "  v_cvt_i32_f32_e32 v132, v132\n" \
    "  v_cvt_i32_f32_e32 v133, v133\n" \
    "  v_mul_f32_e32 v134, v128, v128\n" \
    "  v_mul_f32_e32 v135, v129, v129\n" \
    "  v_fmaak_f32 v137, v134, v136, 0xb2d7322b\n" \
    "  v_fmaak_f32 v138, v135, v136, 0xb2d7322b\n" \
    "  v_fmaak_f32 v137, v134, v137, 0x3638ef1d\n" \
    "  v_fmaak_f32 v138, v135, v138, 0x3638ef1d\n" \
    "  v_fmaak_f32 v137, v134, v137, 0xb9500d01\n" \
    "  v_fmaak_f32 v138, v135, v138, 0xb9500d01\n" \
    "  v_fmaak_f32 v137, v134, v137, 0x3c088889\n" \
    "  v_fmaak_f32 v138, v135, v138, 0x3c088889\n" \
    "  v_fmaak_f32 v137, v134, v137, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v138, v135, v138, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v130, v128, v134\n" \
    "  v_mul_f32_e32 v131, v129, v135\n" \
    "  v_fmac_f32_e32 v128, v130, v137\n" \
    "  v_fmac_f32_e32 v129, v131, v138\n" \
    "  v_lshl_add_u32 v130, v132, 31, v128\n" \
    "  v_lshl_add_u32 v131, v133, 31, v129\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v134, s57\n" \
    "  v_mov_b32_e32 v135, s57\n" \
    "  v_fmac_f32_e64 v134, s58, v128\n" \
    "  v_fmac_f32_e64 v135, s58, v129\n" \
    "  v_mul_f32_e32 v130, v134, v134\n" \
    "  v_mul_f32_e32 v131, v135, v135\n" \
    "  v_mul_f32_e32 v130, 0xbfb8aa3b, v130\n" \
    "  v_mul_f32_e32 v131, 0xbfb8aa3b, v131\n" \
    "  v_exp_f32_e32 v132, v130\n" \
    "  v_exp_f32_e32 v133, v131\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v64, v133\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v134, s57\n" \
    "  v_mov_b32_e32 v135, s57\n" \
    "  v_fmac_f32_e64 v134, s58, v128\n" \
    "  v_fmac_f32_e64 v135, s58, v129\n" \
    "  v_maximum3_f32 v130, v134, -v134, -v134\n" \
    "  v_maximum3_f32 v131, v135, -v135, -v135\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_branch Ldone%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  v_mov_b32_e32 v128, 0\n" \
    "  v_mov_b32_e32 v129, 0\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v64, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  v_fmac_f32_e64 v129, v64, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v64, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  v_fmac_f32_e64 v129, v64, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v128, v0, s65\n" \
    "  v_fmac_f32_e64 v129, v64, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v128, v0, s67\n" \
    "  v_fmac_f32_e64 v129, v64, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v64, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  v_fmac_f32_e64 v129, v64, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v128, v0, s65\n" \
    "  v_fmac_f32_e64 v129, v64, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v128, v0, s67\n" \
    "  v_fmac_f32_e64 v129, v64, s67\n" \
    "  s_set_gpr_idx_idx s68\n" \
    "  v_fmac_f32_e64 v128, v0, s69\n" \
    "  v_fmac_f32_e64 v129, v64, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_fmac_f32_e64 v128, v0, s71\n" \
    "  v_fmac_f32_e64 v129, v64, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v64, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  v_fmac_f32_e64 v129, v64, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v128, v0, s65\n" \
    "  v_fmac_f32_e64 v129, v64, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v128, v0, s67\n" \
    "  v_fmac_f32_e64 v129, v64, s67\n" \
    "  s_set_gpr_idx_idx s68\n" \
    "  v_fmac_f32_e64 v128, v0, s69\n" \
    "  v_fmac_f32_e64 v129, v64, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_fmac_f32_e64 v128, v0, s71\n" \
    "  v_fmac_f32_e64 v129, v64, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_branch Lovs_B%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v64, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v132, v0, s63\n" \
    "  v_mul_f32_e64 v133, v64, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v64, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v132, v0, s63\n" \
    "  v_mul_f32_e64 v133, v64, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s65\n" \
    "  v_mul_f32_e64 v131, v64, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v132, v0, s67\n" \
    "  v_mul_f32_e64 v133, v64, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  v_mul_f32_e32 v129, v129, v131\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v64, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v132, v0, s63\n" \
    "  v_mul_f32_e64 v133, v64, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s65\n" \
    "  v_mul_f32_e64 v131, v64, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v132, v0, s67\n" \
    "  v_mul_f32_e64 v133, v64, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  v_mul_f32_e32 v129, v129, v131\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s69\n" \
    "  v_mul_f32_e64 v131, v64, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v132, v0, s71\n" \
    "  v_mul_f32_e64 v133, v64, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  v_mul_f32_e32 v129, v129, v131\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v64, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v132, v0, s63\n" \
    "  v_mul_f32_e64 v133, v64, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s65\n" \
    "  v_mul_f32_e64 v131, v64, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v132, v0, s67\n" \
    "  v_mul_f32_e64 v133, v64, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  v_mul_f32_e32 v129, v129, v131\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s69\n" \
    "  v_mul_f32_e64 v131, v64, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v132, v0, s71\n" \
    "  v_mul_f32_e64 v133, v64, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  v_mul_f32_e32 v129, v129, v131\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_branch Lovp_B%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s61\n" \
    "  v_mul_f32_e64 v131, v64, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v132, v0, s63\n" \
    "  v_mul_f32_e64 v133, v64, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v130, v132, v132\n" \
    "  v_maximum3_f32 v129, v131, v133, v133\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s61\n" \
    "  v_mul_f32_e64 v131, v64, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v132, v0, s63\n" \
    "  v_mul_f32_e64 v133, v64, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v130, v132, v132\n" \
    "  v_maximum3_f32 v129, v131, v133, v133\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s65\n" \
    "  v_mul_f32_e64 v131, v64, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v132, v0, s67\n" \
    "  v_mul_f32_e64 v133, v64, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v130, v132\n" \
    "  v_maximum3_f32 v129, v129, v131, v133\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s61\n" \
    "  v_mul_f32_e64 v131, v64, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v132, v0, s63\n" \
    "  v_mul_f32_e64 v133, v64, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v130, v132, v132\n" \
    "  v_maximum3_f32 v129, v131, v133, v133\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s65\n" \
    "  v_mul_f32_e64 v131, v64, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v132, v0, s67\n" \
    "  v_mul_f32_e64 v133, v64, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v130, v132\n" \
    "  v_maximum3_f32 v129, v129, v131, v133\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s69\n" \
    "  v_mul_f32_e64 v131, v64, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v132, v0, s71\n" \
    "  v_mul_f32_e64 v133, v64, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v130, v132\n" \
    "  v_maximum3_f32 v129, v129, v131, v133\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s61\n" \
    "  v_mul_f32_e64 v131, v64, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v132, v0, s63\n" \
    "  v_mul_f32_e64 v133, v64, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v130, v132, v132\n" \
    "  v_maximum3_f32 v129, v131, v133, v133\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s65\n" \
    "  v_mul_f32_e64 v131, v64, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v132, v0, s67\n" \
    "  v_mul_f32_e64 v133, v64, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v130, v132\n" \
    "  v_maximum3_f32 v129, v129, v131, v133\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s69\n" \
    "  v_mul_f32_e64 v131, v64, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v132, v0, s71\n" \
    "  v_mul_f32_e64 v133, v64, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v130, v132\n" \
    "  v_maximum3_f32 v129, v129, v131, v133\n" \
    "  s_branch Lovm_B%=\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v134, s57, v128\n" \
    "  v_add_f32_e32 v135, s57, v129\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v134\n" \
    "  v_mov_b32_e32 v64, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v134, s57, v128\n" \
    "  v_add_f32_e32 v135, s57, v129\n" \
    "  v_mul_f32_e32 v130, 0x4038aa3b, v134\n" \
    "  v_mul_f32_e32 v131, 0x4038aa3b, v135\n" \
    "  v_exp_f32_e32 v130, v130\n" \
    "  v_exp_f32_e32 v131, v131\n" \
    "  v_add_f32_e32 v132, 1.0, v130\n" \
    "  v_add_f32_e32 v133, 1.0, v131\n" \
    "  v_rcp_f32_e32 v132, v132\n" \
    "  v_rcp_f32_e32 v133, v133\n" \
    "  v_fma_f32 v130, v132, -2.0, 1.0\n" \
    "  v_fma_f32 v131, v133, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v134, s57, v128\n" \
    "  v_add_f32_e32 v135, s57, v129\n" \
    "  v_mul_f32_e32 v130, 0xbfb8aa3b, v134\n" \
    "  v_mul_f32_e32 v131, 0xbfb8aa3b, v135\n" \
    "  v_exp_f32_e32 v130, v130\n" \
    "  v_exp_f32_e32 v131, v131\n" \
    "  v_add_f32_e32 v132, 1.0, v130\n" \
    "  v_add_f32_e32 v133, 1.0, v131\n" \
    "  v_rcp_f32_e32 v130, v132\n" \
    "  v_rcp_f32_e32 v131, v133\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v134, s57, v128\n" \
    "  v_add_f32_e32 v135, s57, v129\n" \
    "  v_maximum3_f32 v130, v134, 0, 0\n" \
    "  v_maximum3_f32 v131, v135, 0, 0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v134, s57, v128\n" \
    "  v_add_f32_e32 v135, s57, v129\n" \
    "  v_mul_f32_e32 v132, 0x3ea2f983, v134\n" \
    "  v_mul_f32_e32 v133, 0x3ea2f983, v135\n" \
    "  v_rndne_f32_e32 v132, v132\n" \
    "  v_rndne_f32_e32 v133, v133\n" \
    "  v_fmamk_f32 v128, v132, 0xc0490fdb, v134\n" \
    "  v_fmamk_f32 v129, v133, 0xc0490fdb, v135\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v132\n" \
    "  v_fmac_f32_e32 v129, 0x33bbbd2e, v133\n" \
    "  v_cvt_i32_f32_e32 v132, v132\n" \
    "  v_cvt_i32_f32_e32 v133, v133\n" \
    "  v_mul_f32_e32 v134, v128, v128\n" \
    "  v_mul_f32_e32 v135, v129, v129\n" \
    "  v_fmaak_f32 v137, v134, v136, 0xb2d7322b\n" \
    "  v_fmaak_f32 v138, v135, v136, 0xb2d7322b\n" \
    "  v_fmaak_f32 v137, v134, v137, 0x3638ef1d\n" \
    "  v_fmaak_f32 v138, v135, v138, 0x3638ef1d\n" \
    "  v_fmaak_f32 v137, v134, v137, 0xb9500d01\n" \
    "  v_fmaak_f32 v138, v135, v138, 0xb9500d01\n" \
    "  v_fmaak_f32 v137, v134, v137, 0x3c088889\n" \
    "  v_fmaak_f32 v138, v135, v138, 0x3c088889\n" \
    "  v_fmaak_f32 v137, v134, v137, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v138, v135, v138, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v130, v128, v134\n" \
    "  v_mul_f32_e32 v131, v129, v135\n" \
    "  v_fmac_f32_e32 v128, v130, v137\n" \
    "  v_fmac_f32_e32 v129, v131, v138\n" \
    "  v_lshl_add_u32 v130, v132, 31, v128\n" \
    "  v_lshl_add_u32 v131, v133, 31, v129\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v134, s57, v128\n" \
    "  v_add_f32_e32 v135, s57, v129\n" \
    "  v_mul_f32_e32 v130, v134, v134\n" \
    "  v_mul_f32_e32 v131, v135, v135\n" \
    "  v_mul_f32_e32 v130, 0xbfb8aa3b, v130\n" \
    "  v_mul_f32_e32 v131, 0xbfb8aa3b, v131\n" \
    "  v_exp_f32_e32 v132, v130\n" \
    "  v_exp_f32_e32 v133, v131\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v64, v133\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v134, s57, v128\n" \
    "  v_add_f32_e32 v135, s57, v129\n" \
    "  v_maximum3_f32 v130, v134, -v134, -v134\n" \
    "  v_maximum3_f32 v131, v135, -v135, -v135\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovs_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Los_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v128, v0, s73\n" \
    "  v_fmac_f32_e64 v129, v64, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_fmac_f32_e64 v128, v0, s75\n" \
    "  v_fmac_f32_e64 v129, v64, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovds_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v128, v0, s77\n" \
    "  v_fmac_f32_e64 v129, v64, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_fmac_f32_e64 v128, v0, s79\n" \
    "  v_fmac_f32_e64 v129, v64, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovds_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Los_B%=\n" \
    "Lovds_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovp_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lop_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s73\n" \
    "  v_mul_f32_e64 v131, v64, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v132, v0, s75\n" \
    "  v_mul_f32_e64 v133, v64, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  v_mul_f32_e32 v129, v129, v131\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdp_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s77\n" \
    "  v_mul_f32_e64 v131, v64, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v132, v0, s79\n" \
    "  v_mul_f32_e64 v133, v64, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  v_mul_f32_e32 v129, v129, v131\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdp_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lop_B%=\n" \
    "Lovdp_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovm_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lom_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s73\n" \
    "  v_mul_f32_e64 v131, v64, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v132, v0, s75\n" \
    "  v_mul_f32_e64 v133, v64, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v130, v132\n" \
    "  v_maximum3_f32 v129, v129, v131, v133\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdm_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v130, v0, s77\n" \
    "  v_mul_f32_e64 v131, v64, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v132, v0, s79\n" \
    "  v_mul_f32_e64 v133, v64, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v130, v132\n" \
    "  v_maximum3_f32 v129, v129, v131, v133\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdm_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lom_B%=\n" \
    "Lovdm_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Ldone%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_mov_b64 s[44:45], %[outs]\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_lshl_b32 s41, %[no], 2\n" \
    "  v_mul_u32_u24_e32 v144, s41, %[lane]\n" \
    "  v_add_u32_e32 v144, %[om0], v144\n" \
    "  s_lshl_b32 s41, %[no], 8\n" \
    "  v_add_u32_e32 v145, s41, v144\n" \
    "Lout%=:\n" \
    "  s_load_dwordx8 s[48:55], s[44:45], 0x0\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v128, v0\n" \
    "  v_mov_b32_e32 v136, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v128 offset:0\n" \
    "  ds_write_b32 v145, v136 offset:0\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s49, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v129, v0\n" \
    "  v_mov_b32_e32 v137, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v129 offset:4\n" \
    "  ds_write_b32 v145, v137 offset:4\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s50, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v130, v0\n" \
    "  v_mov_b32_e32 v138, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v130 offset:8\n" \
    "  ds_write_b32 v145, v138 offset:8\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s51, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v131, v0\n" \
    "  v_mov_b32_e32 v139, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v131 offset:12\n" \
    "  ds_write_b32 v145, v139 offset:12\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v132, v0\n" \
    "  v_mov_b32_e32 v140, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v132 offset:16\n" \
    "  ds_write_b32 v145, v140 offset:16\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s53, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v133, v0\n" \
    "  v_mov_b32_e32 v141, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v133 offset:20\n" \
    "  ds_write_b32 v145, v141 offset:20\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s54, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v134, v0\n" \
    "  v_mov_b32_e32 v142, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v134 offset:24\n" \
    "  ds_write_b32 v145, v142 offset:24\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s55, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v135, v0\n" \
    "  v_mov_b32_e32 v143, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v135 offset:28\n" \
    "  ds_write_b32 v145, v143 offset:28\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  v_add_u32_e32 v144, 32, v144\n" \
    "  v_add_u32_e32 v145, 32, v145\n" \
    "  s_add_u32 s44, s44, 32\n" \
    "  s_addc_u32 s45, s45, 0\n" \
    "  s_branch Lout%=\n" \
    "Lout_done%=:\n" \
    "  s_mov_b32 m0, s90\n"

#define NEAT_CLOB_S2_64 \
    "v0", "v1", "v2", "v3", "v4", "v5", "v6", "v7", "v8", "v9", "v10", "v11", \
    "v12", "v13", "v14", "v15", "v16", "v17", "v18", "v19", "v20", "v21", "v22", "v23", \
    "v24", "v25", "v26", "v27", "v28", "v29", "v30", "v31", "v32", "v33", "v34", "v35", \
    "v36", "v37", "v38", "v39", "v40", "v41", "v42", "v43", "v44", "v45", "v46", "v47", \
    "v48", "v49", "v50", "v51", "v52", "v53", "v54", "v55", "v56", "v57", "v58", "v59", \
    "v60", "v61", "v62", "v63", "v64", "v65", "v66", "v67", "v68", "v69", "v70", "v71", \
    "v72", "v73", "v74", "v75", "v76", "v77", "v78", "v79", "v80", "v81", "v82", "v83", \
    "v84", "v85", "v86", "v87", "v88", "v89", "v90", "v91", "v92", "v93", "v94", "v95", \
    "v96", "v97", "v98", "v99", "v100", "v101", "v102", "v103", "v104", "v105", "v106", "v107", \
    "v108", "v109", "v110", "v111", "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", \
    "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127", "v128", "v129", "v130", "v131", \
    "v132", "v133", "v134", "v135", "v136", "v137", "v138", "v139", "v140", "v141", "v142", "v143", \
    "v144", "v145", "v146", "v147", "s40", "s41", "s42", "s43", "s44", "s45", "s46", "s47", \
    "s48", "s49", "s50", "s51", "s52", "s53", "s54", "s55", "s56", "s57", "s58", "s59", \
    "s60", "s61", "s62", "s63", "s64", "s65", "s66", "s67", "s68", "s69", "s70", "s71", \
    "s72", "s73", "s74", "s75", "s76", "s77", "s78", "s79", "s80", "s81", "s82", "s83", \
    "s84", "s85", "s86", "s87", "s88", "s89", "s90", "s91", "s92", "s93", "s94", "s95", \
    "vcc", "scc"

#define NEAT_SCRATCH_S2_64 128


// S1_128: 1 sample(s) per lane, value vectors at v0, scratch v128..v139

#define NEAT_TILE_S1_128 \
    "  s_mov_b32 s90, m0\n" \
    "  s_lshl_b32 s41, %[ni], 2\n" \
    "  v_mul_u32_u24_e32 v136, s41, %[lane]\n" \
    "  v_add_u32_e32 v136, %[dm0], v136\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_cmp_eq_u32 %[ni], 0\n" \
    "  s_cbranch_scc1 Lpl_done%=\n" \
    "Lpl%=:\n" \
    "  ds_read2_b32 v[128:129], v136 offset0:0 offset1:1\n" \
    "  ds_read2_b32 v[130:131], v136 offset0:2 offset1:3\n" \
    "  ds_read2_b32 v[132:133], v136 offset0:4 offset1:5\n" \
    "  ds_read2_b32 v[134:135], v136 offset0:6 offset1:7\n" \
    "  v_add_u32_e32 v136, 32, v136\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v128\n" \
    "  v_mov_b32_e32 v1, v129\n" \
    "  v_mov_b32_e32 v2, v130\n" \
    "  v_mov_b32_e32 v3, v131\n" \
    "  v_mov_b32_e32 v4, v132\n" \
    "  v_mov_b32_e32 v5, v133\n" \
    "  v_mov_b32_e32 v6, v134\n" \
    "  v_mov_b32_e32 v7, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_add_u32 s40, s40, 8\n" \
    "  s_cmp_lt_u32 s40, %[ni]\n" \
    "  s_cbranch_scc1 Lpl%=\n" \
    "Lpl_done%=:\n" \
    "  s_set_gpr_idx_on %[zs], gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, 0\n" \
    "  v_mov_b32_e32 v1, 1.0\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 %[dn], 0\n" \
    "  s_cbranch_scc1 Ldma_done%=\n" \
    "  s_mov_b64 s[42:43], exec\n" \
    "  s_cmp_eq_u32 %[dvec], 0\n" \
    "  s_cselect_b32 s41, 2, 4\n" \
    "  v_lshlrev_b32_e32 v138, s41, %[lane]\n" \
    "  v_mov_b32_e32 v139, 0\n" \
    "  v_lshl_add_u64 v[138:139], v[138:139], 0, %[dsrc]\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_mov_b32 m0, %[dm0]\n" \
    "  s_cmp_eq_u32 %[dvec], 0\n" \
    "  s_cbranch_scc1 Ldma1%=\n" \
    "  s_mov_b64 s[46:47], 1024\n" \
    "Ldl4%=:\n" \
    "  s_sub_u32 s41, %[dn], s40\n" \
    "  v_cmp_gt_u32_e64 s[44:45], s41, %[lane]\n" \
    "  s_and_b64 exec, s[42:43], s[44:45]\n" \
    "  s_nop 0\n" \
    "  global_load_lds_dwordx4 v[138:139], off nt\n" \
    "  s_mov_b64 exec, s[42:43]\n" \
    "  v_lshl_add_u64 v[138:139], v[138:139], 0, s[46:47]\n" \
    "  s_add_u32 m0, m0, 1024\n" \
    "  s_add_u32 s40, s40, 64\n" \
    "  s_cmp_lt_u32 s40, %[dn]\n" \
    "  s_cbranch_scc1 Ldl4%=\n" \
    "  s_branch Ldma_done%=\n" \
    "Ldma1%=:\n" \
    "  s_mov_b64 s[46:47], 256\n" \
    "Ldl1%=:\n" \
    "  s_sub_u32 s41, %[dn], s40\n" \
    "  v_cmp_gt_u32_e64 s[44:45], s41, %[lane]\n" \
    "  s_and_b64 exec, s[42:43], s[44:45]\n" \
    "  s_nop 0\n" \
    "  global_load_lds_dword v[138:139], off nt\n" \
    "  s_mov_b64 exec, s[42:43]\n" \
    "  v_lshl_add_u64 v[138:139], v[138:139], 0, s[46:47]\n" \
    "  s_add_u32 m0, m0, 256\n" \
    "  s_add_u32 s40, s40, 64\n" \
    "  s_cmp_lt_u32 s40, %[dn]\n" \
    "  s_cbranch_scc1 Ldl1%=\n" \
    "  s_branch Ldma_done%=\n" \
    "Ldma_done%=:\n" \
    "  s_mov_b64 s[80:81], %[rec]\n" \
    "  s_mov_b64 s[84:85], %[edg]\n" \
    "  s_mov_b32 s86, 0\n" \
    "  v_mov_b32_e32 v132, 0x2f309231\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], 0x0\n" \
    "  s_getpc_b64 s[92:93]\n" \
    "Lpc%=:\n" \
    "  s_add_u32 s94, s92, Ltab_B%= - Lpc%=\n" \
    "  s_addc_u32 s95, s93, 0\n" \
    "  s_add_u32 s92, s92, Ltab_A%= - Lpc%=\n" \
    "  s_addc_u32 s93, s93, 0\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "Ltab_A%=:\n" \
    "  v_mov_b32_e32 v131, s41\n" \
    "  v_fmac_f32_e64 v131, s42, v128\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s41\n" \
    "  v_fmac_f32_e64 v131, s42, v128\n" \
    "  v_mul_f32_e32 v129, 0x4038aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v130, v130\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v129, v130, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s41\n" \
    "  v_fmac_f32_e64 v131, s42, v128\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v129, v130\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s41\n" \
    "  v_fmac_f32_e64 v131, s42, v128\n" \
    "  v_maximum3_f32 v129, v131, 0, 0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s41\n" \
    "  v_fmac_f32_e64 v131, s42, v128\n" \
    "  v_mul_f32_e32 v130, 0x3ea2f983, v131\n" \
    "  v_rndne_f32_e32 v130, v130\n" \
    "  v_fmamk_f32 v128, v130, 0xc0490fdb, v131\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v130\n" \
    "  v_cvt_i32_f32_e32 v130, v130\n" \
    "  v_mul_f32_e32 v131, v128, v128\n" \
    "  v_fmaak_f32 v133, v131, v132, 0xb2d7322b\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3638ef1d\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xb9500d01\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3c088889\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v129, v128, v131\n" \
    "  v_fmac_f32_e32 v128, v129, v133\n" \
    "  v_lshl_add_u32 v129, v130, 31, v128\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s41\n" \
    "  v_fmac_f32_e64 v131, s42, v128\n" \
    "  v_mul_f32_e32 v129, v131, v131\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v129\n" \
    "  v_exp_f32_e32 v130, v129\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s41\n" \
    "  v_fmac_f32_e64 v131, s42, v128\n" \
    "  v_maximum3_f32 v129, v131, -v131, -v131\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_branch Ldone%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  v_mov_b32_e32 v128, 0\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v128, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v128, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v128, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v128, v0, s51\n" \
    "  s_set_gpr_idx_idx s52\n" \
    "  v_fmac_f32_e64 v128, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_fmac_f32_e64 v128, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v128, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v128, v0, s51\n" \
    "  s_set_gpr_idx_idx s52\n" \
    "  v_fmac_f32_e64 v128, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_fmac_f32_e64 v128, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_branch Lovs_A%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v130, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v130, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v130, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v130, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v130, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_branch Lovp_A%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v130, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v130, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v130, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v130, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v130, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_branch Lovm_A%=\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s41, v128\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s41, v128\n" \
    "  v_mul_f32_e32 v129, 0x4038aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v130, v130\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v129, v130, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s41, v128\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v129, v130\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s41, v128\n" \
    "  v_maximum3_f32 v129, v131, 0, 0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s41, v128\n" \
    "  v_mul_f32_e32 v130, 0x3ea2f983, v131\n" \
    "  v_rndne_f32_e32 v130, v130\n" \
    "  v_fmamk_f32 v128, v130, 0xc0490fdb, v131\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v130\n" \
    "  v_cvt_i32_f32_e32 v130, v130\n" \
    "  v_mul_f32_e32 v131, v128, v128\n" \
    "  v_fmaak_f32 v133, v131, v132, 0xb2d7322b\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3638ef1d\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xb9500d01\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3c088889\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v129, v128, v131\n" \
    "  v_fmac_f32_e32 v128, v129, v133\n" \
    "  v_lshl_add_u32 v129, v130, 31, v128\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s41, v128\n" \
    "  v_mul_f32_e32 v129, v131, v131\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v129\n" \
    "  v_exp_f32_e32 v130, v129\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s41, v128\n" \
    "  v_maximum3_f32 v129, v131, -v131, -v131\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovs_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Los_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v128, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_fmac_f32_e64 v128, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovds_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v128, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_fmac_f32_e64 v128, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovds_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Los_A%=\n" \
    "Lovds_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovp_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lop_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v130, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdp_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v130, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdp_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lop_A%=\n" \
    "Lovdp_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovm_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lom_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v130, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdm_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v130, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdm_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lom_A%=\n" \
    "Lovdm_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "Ltab_B%=:\n" \
    "  v_mov_b32_e32 v131, s57\n" \
    "  v_fmac_f32_e64 v131, s58, v128\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s57\n" \
    "  v_fmac_f32_e64 v131, s58, v128\n" \
    "  v_mul_f32_e32 v129, 0x4038aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v130, v130\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v129, v130, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s57\n" \
    "  v_fmac_f32_e64 v131, s58, v128\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v129, v130\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s57\n" \
    "  v_fmac_f32_e64 v131, s58, v128\n" \
    "  v_maximum3_f32 v129, v131, 0, 0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s57\n" \
    "  v_fmac_f32_e64 v131, s58, v128\n" \
    "  v_mul_f32_e32 v130, 0x3ea2f983, v131\n" \
    "  v_rndne_f32_e32 v130, v130\n" \
    "  v_fmamk_f32 v128, v130, 0xc0490fdb, v131\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v130\n" \
    "  v_cvt_i32_f32_e32 v130, v130\n" \
    "  v_mul_f32_e32 v131, v128, v128\n" \
    "  v_fmaak_f32 v133, v131, v132, 0xb2d7322b\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3638ef1d\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xb9500d01\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3c088889\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v129, v128, v131\n" \
    "  v_fmac_f32_e32 v128, v129, v133\n" \
    "  v_lshl_add_u32 v129, v130, 31, v128\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s57\n" \
    "  v_fmac_f32_e64 v131, s58, v128\n" \
    "  v_mul_f32_e32 v129, v131, v131\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v129\n" \
    "  v_exp_f32_e32 v130, v129\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s57\n" \
    "  v_fmac_f32_e64 v131, s58, v128\n" \
    "  v_maximum3_f32 v129, v131, -v131, -v131\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_branch Ldone%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  v_mov_b32_e32 v128, 0\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v128, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v128, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v128, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v128, v0, s67\n" \
    "  s_set_gpr_idx_idx s68\n" \
    "  v_fmac_f32_e64 v128, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_fmac_f32_e64 v128, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v128, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v128, v0, s67\n" \
    "  s_set_gpr_idx_idx s68\n" \
    "  v_fmac_f32_e64 v128, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_fmac_f32_e64 v128, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_branch Lovs_B%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v130, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v130, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v130, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v130, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v130, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_branch Lovp_B%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v130, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v130, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v130, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v130, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v130, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_branch Lovm_B%=\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s57, v128\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s57, v128\n" \
    "  v_mul_f32_e32 v129, 0x4038aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v130, v130\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v129, v130, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s57, v128\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v129, v130\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s57, v128\n" \
    "  v_maximum3_f32 v129, v131, 0, 0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s57, v128\n" \
    "  v_mul_f32_e32 v130, 0x3ea2f983, v131\n" \
    "  v_rndne_f32_e32 v130, v130\n" \
    "  v_fmamk_f32 v128, v130, 0xc0490fdb, v131\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v130\n" \
    "  v_cvt_i32_f32_e32 v130, v130\n" \
    "  v_mul_f32_e32 v131, v128, v128\n" \
    "  v_fmaak_f32 v133, v131, v132, 0xb2d7322b\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3638ef1d\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xb9500d01\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3c088889\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v129, v128, v131\n" \
    "  v_fmac_f32_e32 v128, v129, v133\n" \
    "  v_lshl_add_u32 v129, v130, 31, v128\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s57, v128\n" \
    "  v_mul_f32_e32 v129, v131, v131\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v129\n" \
    "  v_exp_f32_e32 v130, v129\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v130\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s57, v128\n" \
    "  v_maximum3_f32 v129, v131, -v131, -v131\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovs_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Los_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v128, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_fmac_f32_e64 v128, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovds_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v128, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_fmac_f32_e64 v128, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovds_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Los_B%=\n" \
    "Lovds_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovp_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lop_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v130, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdp_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v130, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdp_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lop_B%=\n" \
    "Lovdp_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovm_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lom_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v130, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdm_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v130, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdm_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lom_B%=\n" \
    "Lovdm_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Ldone%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_mov_b64 s[44:45], %[outs]\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_lshl_b32 s41, %[no], 2\n" \
    "  v_mul_u32_u24_e32 v136, s41, %[lane]\n" \
    "  v_add_u32_e32 v136, %[om0], v136\n" \
    "Lout%=:\n" \
    "  s_load_dwordx8 s[48:55], s[44:45], 0x0\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v128, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v128 offset:0\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s49, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v129, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v129 offset:4\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s50, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v130, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v130 offset:8\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s51, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v131, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v131 offset:12\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v132, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v132 offset:16\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s53, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v133, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v133 offset:20\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s54, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v134, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v134 offset:24\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s55, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v135, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v135 offset:28\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  v_add_u32_e32 v136, 32, v136\n" \
    "  s_add_u32 s44, s44, 32\n" \
    "  s_addc_u32 s45, s45, 0\n" \
    "  s_branch Lout%=\n" \
    "Lout_done%=:\n" \
    "  s_mov_b32 m0, s90\n"

#define NEAT_CLOB_S1_128 \
    "v0", "v1", "v2", "v3", "v4", "v5", "v6", "v7", "v8", "v9", "v10", "v11", \
    "v12", "v13", "v14", "v15", "v16", "v17", "v18", "v19", "v20", "v21", "v22", "v23", \
    "v24", "v25", "v26", "v27", "v28", "v29", "v30", "v31", "v32", "v33", "v34", "v35", \
    "v36", "v37", "v38", "v39", "v40", "v41", "v42", "v43", "v44", "v45", "v46", "v47", \
    "v48", "v49", "v50", "v51", "v52", "v53", "v54", "v55", "v56", "v57", "v58", "v59", \
    "v60", "v61", "v62", "v63", "v64", "v65", "v66", "v67", "v68", "v69", "v70", "v71", \
    "v72", "v73", "v74", "v75", "v76", "v77", "v78", "v79", "v80", "v81", "v82", "v83", \
    "v84", "v85", "v86", "v87", "v88", "v89", "v90", "v91", "v92", "v93", "v94", "v95", \
    "v96", "v97", "v98", "v99", "v100", "v101", "v102", "v103", "v104", "v105", "v106", "v107", \
    "v108", "v109", "v110", "v111", "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", \
    "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127", "v128", "v129", "v130", "v131", \
    "v132", "v133", "v134", "v135", "v136", "v137", "v138", "v139", "s40", "s41", "s42", "s43", \
    "s44", "s45", "s46", "s47", "s48", "s49", "s50", "s51", "s52", "s53", "s54", "s55", \
    "s56", "s57", "s58", "s59", "s60", "s61", "s62", "s63", "s64", "s65", "s66", "s67", \
    "s68", "s69", "s70", "s71", "s72", "s73", "s74", "s75", "s76", "s77", "s78", "s79", \
    "s80", "s81", "s82", "s83", "s84", "s85", "s86", "s87", "s88", "s89", "s90", "s91", \
    "s92", "s93", "s94", "s95", "vcc", "scc"

#define NEAT_SCRATCH_S1_128 128


// S1_224: 1 sample(s) per lane, value vectors at v0, scratch v224..v235

#define NEAT_TILE_S1_224 \
    "  s_mov_b32 s90, m0\n" \
    "  s_lshl_b32 s41, %[ni], 2\n" \
    "  v_mul_u32_u24_e32 v232, s41, %[lane]\n" \
    "  v_add_u32_e32 v232, %[dm0], v232\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_cmp_eq_u32 %[ni], 0\n" \
    "  s_cbranch_scc1 Lpl_done%=\n" \
    "Lpl%=:\n" \
    "  ds_read2_b32 v[224:225], v232 offset0:0 offset1:1\n" \
    "  ds_read2_b32 v[226:227], v232 offset0:2 offset1:3\n" \
    "  ds_read2_b32 v[228:229], v232 offset0:4 offset1:5\n" \
    "  ds_read2_b32 v[230:231], v232 offset0:6 offset1:7\n" \
    "  v_add_u32_e32 v232, 32, v232\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v224\n" \
    "  v_mov_b32_e32 v1, v225\n" \
    "  v_mov_b32_e32 v2, v226\n" \
    "  v_mov_b32_e32 v3, v227\n" \
    "  v_mov_b32_e32 v4, v228\n" \
    "  v_mov_b32_e32 v5, v229\n" \
    "  v_mov_b32_e32 v6, v230\n" \
    "  v_mov_b32_e32 v7, v231\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_add_u32 s40, s40, 8\n" \
    "  s_cmp_lt_u32 s40, %[ni]\n" \
    "  s_cbranch_scc1 Lpl%=\n" \
    "Lpl_done%=:\n" \
    "  s_set_gpr_idx_on %[zs], gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, 0\n" \
    "  v_mov_b32_e32 v1, 1.0\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 %[dn], 0\n" \
    "  s_cbranch_scc1 Ldma_done%=\n" \
    "  s_mov_b64 s[42:43], exec\n" \
    "  s_cmp_eq_u32 %[dvec], 0\n" \
    "  s_cselect_b32 s41, 2, 4\n" \
    "  v_lshlrev_b32_e32 v234, s41, %[lane]\n" \
    "  v_mov_b32_e32 v235, 0\n" \
    "  v_lshl_add_u64 v[234:235], v[234:235], 0, %[dsrc]\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_mov_b32 m0, %[dm0]\n" \
    "  s_cmp_eq_u32 %[dvec], 0\n" \
    "  s_cbranch_scc1 Ldma1%=\n" \
    "  s_mov_b64 s[46:47], 1024\n" \
    "Ldl4%=:\n" \
    "  s_sub_u32 s41, %[dn], s40\n" \
    "  v_cmp_gt_u32_e64 s[44:45], s41, %[lane]\n" \
    "  s_and_b64 exec, s[42:43], s[44:45]\n" \
    "  s_nop 0\n" \
    "  global_load_lds_dwordx4 v[234:235], off nt\n" \
    "  s_mov_b64 exec, s[42:43]\n" \
    "  v_lshl_add_u64 v[234:235], v[234:235], 0, s[46:47]\n" \
    "  s_add_u32 m0, m0, 1024\n" \
    "  s_add_u32 s40, s40, 64\n" \
    "  s_cmp_lt_u32 s40, %[dn]\n" \
    "  s_cbranch_scc1 Ldl4%=\n" \
    "  s_branch Ldma_done%=\n" \
    "Ldma1%=:\n" \
    "  s_mov_b64 s[46:47], 256\n" \
    "Ldl1%=:\n" \
    "  s_sub_u32 s41, %[dn], s40\n" \
    "  v_cmp_gt_u32_e64 s[44:45], s41, %[lane]\n" \
    "  s_and_b64 exec, s[42:43], s[44:45]\n" \
    "  s_nop 0\n" \
    "  global_load_lds_dword v[234:235], off nt\n" \
    "  s_mov_b64 exec, s[42:43]\n" \
    "  v_lshl_add_u64 v[234:235], v[234:235], 0, s[46:47]\n" \
    "  s_add_u32 m0, m0, 256\n" \
    "  s_add_u32 s40, s40, 64\n" \
    "  s_cmp_lt_u32 s40, %[dn]\n" \
    "  s_cbranch_scc1 Ldl1%=\n" \
    "  s_branch Ldma_done%=\n" \
    "Ldma_done%=:\n" \
    "  s_mov_b64 s[80:81], %[rec]\n" \
    "  s_mov_b64 s[84:85], %[edg]\n" \
    "  s_mov_b32 s86, 0\n" \
    "  v_mov_b32_e32 v228, 0x2f309231\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], 0x0\n" \
    "  s_getpc_b64 s[92:93]\n" \
    "Lpc%=:\n" \
    "  s_add_u32 s94, s92, Ltab_B%= - Lpc%=\n" \
    "  s_addc_u32 s95, s93, 0\n" \
    "  s_add_u32 s92, s92, Ltab_A%= - Lpc%=\n" \
    "  s_addc_u32 s93, s93, 0\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "Ltab_A%=:\n" \
    "  v_mov_b32_e32 v227, s41\n" \
    "  v_fmac_f32_e64 v227, s42, v224\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v227\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v227, s41\n" \
    "  v_fmac_f32_e64 v227, s42, v224\n" \
    "  v_mul_f32_e32 v225, 0x4038aa3b, v227\n" \
    "  v_exp_f32_e32 v225, v225\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v226, 1.0, v225\n" \
    "  v_rcp_f32_e32 v226, v226\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v225, v226, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v227, s41\n" \
    "  v_fmac_f32_e64 v227, s42, v224\n" \
    "  v_mul_f32_e32 v225, 0xbfb8aa3b, v227\n" \
    "  v_exp_f32_e32 v225, v225\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v226, 1.0, v225\n" \
    "  v_rcp_f32_e32 v225, v226\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v227, s41\n" \
    "  v_fmac_f32_e64 v227, s42, v224\n" \
    "  v_maximum3_f32 v225, v227, 0, 0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v227, s41\n" \
    "  v_fmac_f32_e64 v227, s42, v224\n" \
    "  v_mul_f32_e32 v226, 0x3ea2f983, v227\n" \
    "  v_rndne_f32_e32 v226, v226\n" \
    "  v_fmamk_f32 v224, v226, 0xc0490fdb, v227\n" \
    "  v_fmac_f32_e32 v224, 0x33bbbd2e, v226\n" \
    "  v_cvt_i32_f32_e32 v226, v226\n" \
    "  v_mul_f32_e32 v227, v224, v224\n" \
    "  v_fmaak_f32 v229, v227, v228, 0xb2d7322b\n" \
    "  v_fmaak_f32 v229, v227, v229, 0x3638ef1d\n" \
    "  v_fmaak_f32 v229, v227, v229, 0xb9500d01\n" \
    "  v_fmaak_f32 v229, v227, v229, 0x3c088889\n" \
    "  v_fmaak_f32 v229, v227, v229, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v225, v224, v227\n" \
    "  v_fmac_f32_e32 v224, v225, v229\n" \
    "  v_lshl_add_u32 v225, v226, 31, v224\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v227, s41\n" \
    "  v_fmac_f32_e64 v227, s42, v224\n" \
    "  v_mul_f32_e32 v225, v227, v227\n" \
    "  v_mul_f32_e32 v225, 0xbfb8aa3b, v225\n" \
    "  v_exp_f32_e32 v226, v225\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v226\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v227, s41\n" \
    "  v_fmac_f32_e64 v227, s42, v224\n" \
    "  v_maximum3_f32 v225, v227, -v227, -v227\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_branch Ldone%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  v_mov_b32_e32 v224, 0\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v224, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v224, v0, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v224, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v224, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v224, v0, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v224, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v224, v0, s51\n" \
    "  s_set_gpr_idx_idx s52\n" \
    "  v_fmac_f32_e64 v224, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_fmac_f32_e64 v224, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v224, v0, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v224, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v224, v0, s51\n" \
    "  s_set_gpr_idx_idx s52\n" \
    "  v_fmac_f32_e64 v224, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_fmac_f32_e64 v224, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_branch Lovs_A%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v226, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v226, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v226, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v225\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v226, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v226, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v225\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v226, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v225\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v226, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v226, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v225\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v226, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v225\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_branch Lovp_A%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v226, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v225, v226, v226\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v226, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v225, v226, v226\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v226, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v224, v225, v226\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v226, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v225, v226, v226\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v226, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v224, v225, v226\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v226, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v224, v225, v226\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v226, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v225, v226, v226\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v226, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v224, v225, v226\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v226, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v224, v225, v226\n" \
    "  s_branch Lovm_A%=\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v227, s41, v224\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v227\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v227, s41, v224\n" \
    "  v_mul_f32_e32 v225, 0x4038aa3b, v227\n" \
    "  v_exp_f32_e32 v225, v225\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v226, 1.0, v225\n" \
    "  v_rcp_f32_e32 v226, v226\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v225, v226, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v227, s41, v224\n" \
    "  v_mul_f32_e32 v225, 0xbfb8aa3b, v227\n" \
    "  v_exp_f32_e32 v225, v225\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v226, 1.0, v225\n" \
    "  v_rcp_f32_e32 v225, v226\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v227, s41, v224\n" \
    "  v_maximum3_f32 v225, v227, 0, 0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v227, s41, v224\n" \
    "  v_mul_f32_e32 v226, 0x3ea2f983, v227\n" \
    "  v_rndne_f32_e32 v226, v226\n" \
    "  v_fmamk_f32 v224, v226, 0xc0490fdb, v227\n" \
    "  v_fmac_f32_e32 v224, 0x33bbbd2e, v226\n" \
    "  v_cvt_i32_f32_e32 v226, v226\n" \
    "  v_mul_f32_e32 v227, v224, v224\n" \
    "  v_fmaak_f32 v229, v227, v228, 0xb2d7322b\n" \
    "  v_fmaak_f32 v229, v227, v229, 0x3638ef1d\n" \
    "  v_fmaak_f32 v229, v227, v229, 0xb9500d01\n" \
    "  v_fmaak_f32 v229, v227, v229, 0x3c088889\n" \
    "  v_fmaak_f32 v229, v227, v229, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v225, v224, v227\n" \
    "  v_fmac_f32_e32 v224, v225, v229\n" \
    "  v_lshl_add_u32 v225, v226, 31, v224\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v227, s41, v224\n" \
    "  v_mul_f32_e32 v225, v227, v227\n" \
    "  v_mul_f32_e32 v225, 0xbfb8aa3b, v225\n" \
    "  v_exp_f32_e32 v226, v225\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v226\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v227, s41, v224\n" \
    "  v_maximum3_f32 v225, v227, -v227, -v227\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovs_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Los_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v224, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_fmac_f32_e64 v224, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovds_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v224, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_fmac_f32_e64 v224, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovds_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Los_A%=\n" \
    "Lovds_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovp_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lop_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v226, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v225\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdp_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v226, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v225\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdp_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lop_A%=\n" \
    "Lovdp_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovm_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lom_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v226, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v224, v225, v226\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdm_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v226, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v224, v225, v226\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdm_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lom_A%=\n" \
    "Lovdm_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "Ltab_B%=:\n" \
    "  v_mov_b32_e32 v227, s57\n" \
    "  v_fmac_f32_e64 v227, s58, v224\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v227\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v227, s57\n" \
    "  v_fmac_f32_e64 v227, s58, v224\n" \
    "  v_mul_f32_e32 v225, 0x4038aa3b, v227\n" \
    "  v_exp_f32_e32 v225, v225\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v226, 1.0, v225\n" \
    "  v_rcp_f32_e32 v226, v226\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v225, v226, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v227, s57\n" \
    "  v_fmac_f32_e64 v227, s58, v224\n" \
    "  v_mul_f32_e32 v225, 0xbfb8aa3b, v227\n" \
    "  v_exp_f32_e32 v225, v225\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v226, 1.0, v225\n" \
    "  v_rcp_f32_e32 v225, v226\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v227, s57\n" \
    "  v_fmac_f32_e64 v227, s58, v224\n" \
    "  v_maximum3_f32 v225, v227, 0, 0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v227, s57\n" \
    "  v_fmac_f32_e64 v227, s58, v224\n" \
    "  v_mul_f32_e32 v226, 0x3ea2f983, v227\n" \
    "  v_rndne_f32_e32 v226, v226\n" \
    "  v_fmamk_f32 v224, v226, 0xc0490fdb, v227\n" \
    "  v_fmac_f32_e32 v224, 0x33bbbd2e, v226\n" \
    "  v_cvt_i32_f32_e32 v226, v226\n" \
    "  v_mul_f32_e32 v227, v224, v224\n" \
    "  v_fmaak_f32 v229, v227, v228, 0xb2d7322b\n" \
    "  v_fmaak_f32 v229, v227, v229, 0x3638ef1d\n" \
    "  v_fmaak_f32 v229, v227, v229, 0xb9500d01\n" \
    "  v_fmaak_f32 v229, v227, v229, 0x3c088889\n" \
    "  v_fmaak_f32 v229, v227, v229, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v225, v224, v227\n" \
    "  v_fmac_f32_e32 v224, v225, v229\n" \
    "  v_lshl_add_u32 v225, v226, 31, v224\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v227, s57\n" \
    "  v_fmac_f32_e64 v227, s58, v224\n" \
    "  v_mul_f32_e32 v225, v227, v227\n" \
    "  v_mul_f32_e32 v225, 0xbfb8aa3b, v225\n" \
    "  v_exp_f32_e32 v226, v225\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v226\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v227, s57\n" \
    "  v_fmac_f32_e64 v227, s58, v224\n" \
    "  v_maximum3_f32 v225, v227, -v227, -v227\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_branch Ldone%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  v_mov_b32_e32 v224, 0\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v224, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v224, v0, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v224, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v224, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v224, v0, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v224, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v224, v0, s67\n" \
    "  s_set_gpr_idx_idx s68\n" \
    "  v_fmac_f32_e64 v224, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_fmac_f32_e64 v224, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v224, v0, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v224, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v224, v0, s67\n" \
    "  s_set_gpr_idx_idx s68\n" \
    "  v_fmac_f32_e64 v224, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_fmac_f32_e64 v224, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_branch Lovs_B%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v226, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v226, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v226, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v225\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v226, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v226, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v225\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v226, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v225\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v224, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v226, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v226, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v225\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v226, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v225\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_branch Lovp_B%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v226, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v225, v226, v226\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v226, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v225, v226, v226\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v226, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v224, v225, v226\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v226, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v225, v226, v226\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v226, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v224, v225, v226\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v226, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v224, v225, v226\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v226, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v225, v226, v226\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v226, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v224, v225, v226\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v226, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v224, v225, v226\n" \
    "  s_branch Lovm_B%=\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v227, s57, v224\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v227\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v227, s57, v224\n" \
    "  v_mul_f32_e32 v225, 0x4038aa3b, v227\n" \
    "  v_exp_f32_e32 v225, v225\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v226, 1.0, v225\n" \
    "  v_rcp_f32_e32 v226, v226\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v225, v226, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v227, s57, v224\n" \
    "  v_mul_f32_e32 v225, 0xbfb8aa3b, v227\n" \
    "  v_exp_f32_e32 v225, v225\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v226, 1.0, v225\n" \
    "  v_rcp_f32_e32 v225, v226\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v227, s57, v224\n" \
    "  v_maximum3_f32 v225, v227, 0, 0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v227, s57, v224\n" \
    "  v_mul_f32_e32 v226, 0x3ea2f983, v227\n" \
    "  v_rndne_f32_e32 v226, v226\n" \
    "  v_fmamk_f32 v224, v226, 0xc0490fdb, v227\n" \
    "  v_fmac_f32_e32 v224, 0x33bbbd2e, v226\n" \
    "  v_cvt_i32_f32_e32 v226, v226\n" \
    "  v_mul_f32_e32 v227, v224, v224\n" \
    "  v_fmaak_f32 v229, v227, v228, 0xb2d7322b\n" \
    "  v_fmaak_f32 v229, v227, v229, 0x3638ef1d\n" \
    "  v_fmaak_f32 v229, v227, v229, 0xb9500d01\n" \
    "  v_fmaak_f32 v229, v227, v229, 0x3c088889\n" \
    "  v_fmaak_f32 v229, v227, v229, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v225, v224, v227\n" \
    "  v_fmac_f32_e32 v224, v225, v229\n" \
    "  v_lshl_add_u32 v225, v226, 31, v224\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v227, s57, v224\n" \
    "  v_mul_f32_e32 v225, v227, v227\n" \
    "  v_mul_f32_e32 v225, 0xbfb8aa3b, v225\n" \
    "  v_exp_f32_e32 v226, v225\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v226\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v227, s57, v224\n" \
    "  v_maximum3_f32 v225, v227, -v227, -v227\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v225\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovs_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Los_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v224, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_fmac_f32_e64 v224, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovds_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v224, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_fmac_f32_e64 v224, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovds_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Los_B%=\n" \
    "Lovds_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovp_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lop_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v226, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v225\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdp_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v226, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v224, v224, v225\n" \
    "  v_mul_f32_e32 v224, v224, v226\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdp_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lop_B%=\n" \
    "Lovdp_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovm_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lom_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v226, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v224, v225, v226\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdm_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v225, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v226, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v224, v224, v225, v226\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdm_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lom_B%=\n" \
    "Lovdm_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Ldone%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_mov_b64 s[44:45], %[outs]\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_lshl_b32 s41, %[no], 2\n" \
    "  v_mul_u32_u24_e32 v232, s41, %[lane]\n" \
    "  v_add_u32_e32 v232, %[om0], v232\n" \
    "Lout%=:\n" \
    "  s_load_dwordx8 s[48:55], s[44:45], 0x0\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v224, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v232, v224 offset:0\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s49, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v225, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v232, v225 offset:4\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s50, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v226, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v232, v226 offset:8\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s51, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v227, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v232, v227 offset:12\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v228, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v232, v228 offset:16\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s53, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v229, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v232, v229 offset:20\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s54, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v230, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v232, v230 offset:24\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s55, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v231, v0\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v232, v231 offset:28\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  v_add_u32_e32 v232, 32, v232\n" \
    "  s_add_u32 s44, s44, 32\n" \
    "  s_addc_u32 s45, s45, 0\n" \
    "  s_branch Lout%=\n" \
    "Lout_done%=:\n" \
    "  s_mov_b32 m0, s90\n"

#define NEAT_CLOB_S1_224 \
    "v0", "v1", "v2", "v3", "v4", "v5", "v6", "v7", "v8", "v9", "v10", "v11", \
    "v12", "v13", "v14", "v15", "v16", "v17", "v18", "v19", "v20", "v21", "v22", "v23", \
    "v24", "v25", "v26", "v27", "v28", "v29", "v30", "v31", "v32", "v33", "v34", "v35", \
    "v36", "v37", "v38", "v39", "v40", "v41", "v42", "v43", "v44", "v45", "v46", "v47", \
    "v48", "v49", "v50", "v51", "v52", "v53", "v54", "v55", "v56", "v57", "v58", "v59", \
    "v60", "v61", "v62", "v63", "v64", "v65", "v66", "v67", "v68", "v69", "v70", "v71", \
    "v72", "v73", "v74", "v75", "v76", "v77", "v78", "v79", "v80", "v81", "v82", "v83", \
    "v84", "v85", "v86", "v87", "v88", "v89", "v90", "v91", "v92", "v93", "v94", "v95", \
    "v96", "v97", "v98", "v99", "v100", "v101", "v102", "v103", "v104", "v105", "v106", "v107", \
    "v108", "v109", "v110", "v111", "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", \
    "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127", "v128", "v129", "v130", "v131", \
    "v132", "v133", "v134", "v135", "v136", "v137", "v138", "v139", "v140", "v141", "v142", "v143", \
    "v144", "v145", "v146", "v147", "v148", "v149", "v150", "v151", "v152", "v153", "v154", "v155", \
    "v156", "v157", "v158", "v159", "v160", "v161", "v162", "v163", "v164", "v165", "v166", "v167", \
    "v168", "v169", "v170", "v171", "v172", "v173", "v174", "v175", "v176", "v177", "v178", "v179", \
    "v180", "v181", "v182", "v183", "v184", "v185", "v186", "v187", "v188", "v189", "v190", "v191", \
    "v192", "v193", "v194", "v195", "v196", "v197", "v198", "v199", "v200", "v201", "v202", "v203", \
    "v204", "v205", "v206", "v207", "v208", "v209", "v210", "v211", "v212", "v213", "v214", "v215", \
    "v216", "v217", "v218", "v219", "v220", "v221", "v222", "v223", "v224", "v225", "v226", "v227", \
    "v228", "v229", "v230", "v231", "v232", "v233", "v234", "v235", "s40", "s41", "s42", "s43", \
    "s44", "s45", "s46", "s47", "s48", "s49", "s50", "s51", "s52", "s53", "s54", "s55", \
    "s56", "s57", "s58", "s59", "s60", "s61", "s62", "s63", "s64", "s65", "s66", "s67", \
    "s68", "s69", "s70", "s71", "s72", "s73", "s74", "s75", "s76", "s77", "s78", "s79", \
    "s80", "s81", "s82", "s83", "s84", "s85", "s86", "s87", "s88", "s89", "s90", "s91", \
    "s92", "s93", "s94", "s95", "vcc", "scc"

#define NEAT_SCRATCH_S1_224 224


// S1_64R: 1 sample(s) per lane, value vectors at v0, scratch v128..v139

#define NEAT_TILE_S1_64R \
    "  s_mov_b32 s90, m0\n" \
    "  s_add_u32 s41, %[n], %[ni]\n" \
    "  v_mov_b32_e32 v0, 0\n" \
    "  v_mov_b32_e32 v1, 0\n" \
    "  v_mov_b32_e32 v2, 0\n" \
    "  v_mov_b32_e32 v3, 0\n" \
    "  v_mov_b32_e32 v4, 0\n" \
    "  v_mov_b32_e32 v5, 0\n" \
    "  v_mov_b32_e32 v6, 0\n" \
    "  v_mov_b32_e32 v7, 0\n" \
    "  s_cmp_le_u32 s41, 8\n" \
    "  s_cbranch_scc1 Lzr%=\n" \
    "  v_mov_b32_e32 v8, 0\n" \
    "  v_mov_b32_e32 v9, 0\n" \
    "  v_mov_b32_e32 v10, 0\n" \
    "  v_mov_b32_e32 v11, 0\n" \
    "  v_mov_b32_e32 v12, 0\n" \
    "  v_mov_b32_e32 v13, 0\n" \
    "  v_mov_b32_e32 v14, 0\n" \
    "  v_mov_b32_e32 v15, 0\n" \
    "  s_cmp_le_u32 s41, 16\n" \
    "  s_cbranch_scc1 Lzr%=\n" \
    "  v_mov_b32_e32 v16, 0\n" \
    "  v_mov_b32_e32 v17, 0\n" \
    "  v_mov_b32_e32 v18, 0\n" \
    "  v_mov_b32_e32 v19, 0\n" \
    "  v_mov_b32_e32 v20, 0\n" \
    "  v_mov_b32_e32 v21, 0\n" \
    "  v_mov_b32_e32 v22, 0\n" \
    "  v_mov_b32_e32 v23, 0\n" \
    "  s_cmp_le_u32 s41, 24\n" \
    "  s_cbranch_scc1 Lzr%=\n" \
    "  v_mov_b32_e32 v24, 0\n" \
    "  v_mov_b32_e32 v25, 0\n" \
    "  v_mov_b32_e32 v26, 0\n" \
    "  v_mov_b32_e32 v27, 0\n" \
    "  v_mov_b32_e32 v28, 0\n" \
    "  v_mov_b32_e32 v29, 0\n" \
    "  v_mov_b32_e32 v30, 0\n" \
    "  v_mov_b32_e32 v31, 0\n" \
    "  s_cmp_le_u32 s41, 32\n" \
    "  s_cbranch_scc1 Lzr%=\n" \
    "  v_mov_b32_e32 v32, 0\n" \
    "  v_mov_b32_e32 v33, 0\n" \
    "  v_mov_b32_e32 v34, 0\n" \
    "  v_mov_b32_e32 v35, 0\n" \
    "  v_mov_b32_e32 v36, 0\n" \
    "  v_mov_b32_e32 v37, 0\n" \
    "  v_mov_b32_e32 v38, 0\n" \
    "  v_mov_b32_e32 v39, 0\n" \
    "  s_cmp_le_u32 s41, 40\n" \
    "  s_cbranch_scc1 Lzr%=\n" \
    "  v_mov_b32_e32 v40, 0\n" \
    "  v_mov_b32_e32 v41, 0\n" \
    "  v_mov_b32_e32 v42, 0\n" \
    "  v_mov_b32_e32 v43, 0\n" \
    "  v_mov_b32_e32 v44, 0\n" \
    "  v_mov_b32_e32 v45, 0\n" \
    "  v_mov_b32_e32 v46, 0\n" \
    "  v_mov_b32_e32 v47, 0\n" \
    "  s_cmp_le_u32 s41, 48\n" \
    "  s_cbranch_scc1 Lzr%=\n" \
    "  v_mov_b32_e32 v48, 0\n" \
    "  v_mov_b32_e32 v49, 0\n" \
    "  v_mov_b32_e32 v50, 0\n" \
    "  v_mov_b32_e32 v51, 0\n" \
    "  v_mov_b32_e32 v52, 0\n" \
    "  v_mov_b32_e32 v53, 0\n" \
    "  v_mov_b32_e32 v54, 0\n" \
    "  v_mov_b32_e32 v55, 0\n" \
    "  s_cmp_le_u32 s41, 56\n" \
    "  s_cbranch_scc1 Lzr%=\n" \
    "  v_mov_b32_e32 v56, 0\n" \
    "  v_mov_b32_e32 v57, 0\n" \
    "  v_mov_b32_e32 v58, 0\n" \
    "  v_mov_b32_e32 v59, 0\n" \
    "  v_mov_b32_e32 v60, 0\n" \
    "  v_mov_b32_e32 v61, 0\n" \
    "  v_mov_b32_e32 v62, 0\n" \
    "  v_mov_b32_e32 v63, 0\n" \
    "Lzr%=:\n" \
    "  s_cmp_lg_u32 %[nsw], 0\n" \
    "  s_cbranch_scc1 Lzw%=\n" \
    "  s_add_u32 s41, %[n], %[ni]\n" \
    "  v_mov_b32_e32 v64, 0\n" \
    "  v_mov_b32_e32 v65, 0\n" \
    "  v_mov_b32_e32 v66, 0\n" \
    "  v_mov_b32_e32 v67, 0\n" \
    "  v_mov_b32_e32 v68, 0\n" \
    "  v_mov_b32_e32 v69, 0\n" \
    "  v_mov_b32_e32 v70, 0\n" \
    "  v_mov_b32_e32 v71, 0\n" \
    "  s_cmp_le_u32 s41, 8\n" \
    "  s_cbranch_scc1 Lzw%=\n" \
    "  v_mov_b32_e32 v72, 0\n" \
    "  v_mov_b32_e32 v73, 0\n" \
    "  v_mov_b32_e32 v74, 0\n" \
    "  v_mov_b32_e32 v75, 0\n" \
    "  v_mov_b32_e32 v76, 0\n" \
    "  v_mov_b32_e32 v77, 0\n" \
    "  v_mov_b32_e32 v78, 0\n" \
    "  v_mov_b32_e32 v79, 0\n" \
    "  s_cmp_le_u32 s41, 16\n" \
    "  s_cbranch_scc1 Lzw%=\n" \
    "  v_mov_b32_e32 v80, 0\n" \
    "  v_mov_b32_e32 v81, 0\n" \
    "  v_mov_b32_e32 v82, 0\n" \
    "  v_mov_b32_e32 v83, 0\n" \
    "  v_mov_b32_e32 v84, 0\n" \
    "  v_mov_b32_e32 v85, 0\n" \
    "  v_mov_b32_e32 v86, 0\n" \
    "  v_mov_b32_e32 v87, 0\n" \
    "  s_cmp_le_u32 s41, 24\n" \
    "  s_cbranch_scc1 Lzw%=\n" \
    "  v_mov_b32_e32 v88, 0\n" \
    "  v_mov_b32_e32 v89, 0\n" \
    "  v_mov_b32_e32 v90, 0\n" \
    "  v_mov_b32_e32 v91, 0\n" \
    "  v_mov_b32_e32 v92, 0\n" \
    "  v_mov_b32_e32 v93, 0\n" \
    "  v_mov_b32_e32 v94, 0\n" \
    "  v_mov_b32_e32 v95, 0\n" \
    "  s_cmp_le_u32 s41, 32\n" \
    "  s_cbranch_scc1 Lzw%=\n" \
    "  v_mov_b32_e32 v96, 0\n" \
    "  v_mov_b32_e32 v97, 0\n" \
    "  v_mov_b32_e32 v98, 0\n" \
    "  v_mov_b32_e32 v99, 0\n" \
    "  v_mov_b32_e32 v100, 0\n" \
    "  v_mov_b32_e32 v101, 0\n" \
    "  v_mov_b32_e32 v102, 0\n" \
    "  v_mov_b32_e32 v103, 0\n" \
    "  s_cmp_le_u32 s41, 40\n" \
    "  s_cbranch_scc1 Lzw%=\n" \
    "  v_mov_b32_e32 v104, 0\n" \
    "  v_mov_b32_e32 v105, 0\n" \
    "  v_mov_b32_e32 v106, 0\n" \
    "  v_mov_b32_e32 v107, 0\n" \
    "  v_mov_b32_e32 v108, 0\n" \
    "  v_mov_b32_e32 v109, 0\n" \
    "  v_mov_b32_e32 v110, 0\n" \
    "  v_mov_b32_e32 v111, 0\n" \
    "  s_cmp_le_u32 s41, 48\n" \
    "  s_cbranch_scc1 Lzw%=\n" \
    "  v_mov_b32_e32 v112, 0\n" \
    "  v_mov_b32_e32 v113, 0\n" \
    "  v_mov_b32_e32 v114, 0\n" \
    "  v_mov_b32_e32 v115, 0\n" \
    "  v_mov_b32_e32 v116, 0\n" \
    "  v_mov_b32_e32 v117, 0\n" \
    "  v_mov_b32_e32 v118, 0\n" \
    "  v_mov_b32_e32 v119, 0\n" \
    "  s_cmp_le_u32 s41, 56\n" \
    "  s_cbranch_scc1 Lzw%=\n" \
    "  v_mov_b32_e32 v120, 0\n" \
    "  v_mov_b32_e32 v121, 0\n" \
    "  v_mov_b32_e32 v122, 0\n" \
    "  v_mov_b32_e32 v123, 0\n" \
    "  v_mov_b32_e32 v124, 0\n" \
    "  v_mov_b32_e32 v125, 0\n" \
    "  v_mov_b32_e32 v126, 0\n" \
    "  v_mov_b32_e32 v127, 0\n" \
    "Lzw%=:\n" \
    "  s_lshl_b32 s41, %[ni], 2\n" \
    "  v_mul_u32_u24_e32 v136, s41, %[lane]\n" \
    "  v_add_u32_e32 v136, %[dm0], v136\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_cmp_eq_u32 %[ni], 0\n" \
    "  s_cbranch_scc1 Lpl_done%=\n" \
    "Lpl%=:\n" \
    "  ds_read2_b32 v[128:129], v136 offset0:0 offset1:1\n" \
    "  ds_read2_b32 v[130:131], v136 offset0:2 offset1:3\n" \
    "  ds_read2_b32 v[132:133], v136 offset0:4 offset1:5\n" \
    "  ds_read2_b32 v[134:135], v136 offset0:6 offset1:7\n" \
    "  v_add_u32_e32 v136, 32, v136\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v128\n" \
    "  v_mov_b32_e32 v1, v129\n" \
    "  v_mov_b32_e32 v2, v130\n" \
    "  v_mov_b32_e32 v3, v131\n" \
    "  v_mov_b32_e32 v4, v132\n" \
    "  v_mov_b32_e32 v5, v133\n" \
    "  v_mov_b32_e32 v6, v134\n" \
    "  v_mov_b32_e32 v7, v135\n" \
    "  v_mov_b32_e32 v64, v128\n" \
    "  v_mov_b32_e32 v65, v129\n" \
    "  v_mov_b32_e32 v66, v130\n" \
    "  v_mov_b32_e32 v67, v131\n" \
    "  v_mov_b32_e32 v68, v132\n" \
    "  v_mov_b32_e32 v69, v133\n" \
    "  v_mov_b32_e32 v70, v134\n" \
    "  v_mov_b32_e32 v71, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_add_u32 s40, s40, 8\n" \
    "  s_cmp_lt_u32 s40, %[ni]\n" \
    "  s_cbranch_scc1 Lpl%=\n" \
    "Lpl_done%=:\n" \
    "  s_mov_b32 s41, %[ni]\n" \
    "Lcl%=:\n" \
    "  s_and_b32 s40, s41, 7\n" \
    "  s_cbranch_scc0 Lcl_done%=\n" \
    "  s_set_gpr_idx_on s41, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, 0\n" \
    "  v_mov_b32_e32 v64, 0\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_add_u32 s41, s41, 1\n" \
    "  s_branch Lcl%=\n" \
    "Lcl_done%=:\n" \
    "  s_set_gpr_idx_on %[zs], gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, 0\n" \
    "  v_mov_b32_e32 v1, 1.0\n" \
    "  v_mov_b32_e32 v64, 0\n" \
    "  v_mov_b32_e32 v65, 1.0\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 %[dn], 0\n" \
    "  s_cbranch_scc1 Ldma_done%=\n" \
    "  s_mov_b64 s[42:43], exec\n" \
    "  s_cmp_eq_u32 %[dvec], 0\n" \
    "  s_cselect_b32 s41, 2, 4\n" \
    "  v_lshlrev_b32_e32 v138, s41, %[lane]\n" \
    "  v_mov_b32_e32 v139, 0\n" \
    "  v_lshl_add_u64 v[138:139], v[138:139], 0, %[dsrc]\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_mov_b32 m0, %[dm0]\n" \
    "  s_cmp_eq_u32 %[dvec], 0\n" \
    "  s_cbranch_scc1 Ldma1%=\n" \
    "  s_mov_b64 s[46:47], 1024\n" \
    "Ldl4%=:\n" \
    "  s_sub_u32 s41, %[dn], s40\n" \
    "  v_cmp_gt_u32_e64 s[44:45], s41, %[lane]\n" \
    "  s_and_b64 exec, s[42:43], s[44:45]\n" \
    "  s_nop 0\n" \
    "  global_load_lds_dwordx4 v[138:139], off nt\n" \
    "  s_mov_b64 exec, s[42:43]\n" \
    "  v_lshl_add_u64 v[138:139], v[138:139], 0, s[46:47]\n" \
    "  s_add_u32 m0, m0, 1024\n" \
    "  s_add_u32 s40, s40, 64\n" \
    "  s_cmp_lt_u32 s40, %[dn]\n" \
    "  s_cbranch_scc1 Ldl4%=\n" \
    "  s_branch Ldma_done%=\n" \
    "Ldma1%=:\n" \
    "  s_mov_b64 s[46:47], 256\n" \
    "Ldl1%=:\n" \
    "  s_sub_u32 s41, %[dn], s40\n" \
    "  v_cmp_gt_u32_e64 s[44:45], s41, %[lane]\n" \
    "  s_and_b64 exec, s[42:43], s[44:45]\n" \
    "  s_nop 0\n" \
    "  global_load_lds_dword v[138:139], off nt\n" \
    "  s_mov_b64 exec, s[42:43]\n" \
    "  v_lshl_add_u64 v[138:139], v[138:139], 0, s[46:47]\n" \
    "  s_add_u32 m0, m0, 256\n" \
    "  s_add_u32 s40, s40, 64\n" \
    "  s_cmp_lt_u32 s40, %[dn]\n" \
    "  s_cbranch_scc1 Ldl1%=\n" \
    "  s_branch Ldma_done%=\n" \
    "Ldma_done%=:\n" \
    "  s_mov_b32 s91, %[nsw]\n" \
    "Lsw%=:\n" \
    "  s_cmp_eq_u32 s91, 0\n" \
    "  s_cbranch_scc1 Lsw_done%=\n" \
    "  s_mov_b64 s[80:81], %[rec]\n" \
    "  s_mov_b64 s[84:85], %[edg]\n" \
    "  s_mov_b32 s86, 0\n" \
    "  v_mov_b32_e32 v132, 0x2f309231\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], 0x0\n" \
    "  s_getpc_b64 s[92:93]\n" \
    "Lpc%=:\n" \
    "  s_add_u32 s94, s92, Ltab_B%= - Lpc%=\n" \
    "  s_addc_u32 s95, s93, 0\n" \
    "  s_add_u32 s92, s92, Ltab_A%= - Lpc%=\n" \
    "  s_addc_u32 s93, s93, 0\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "Ltab_A%=:\n" \
    "  v_mov_b32_e32 v131, s41\n" \
    "  v_fmac_f32_e64 v131, s42, v128\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s41\n" \
    "  v_fmac_f32_e64 v131, s42, v128\n" \
    "  v_mul_f32_e32 v129, 0x4038aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v130, v130\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v129, v130, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s41\n" \
    "  v_fmac_f32_e64 v131, s42, v128\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v129, v130\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s41\n" \
    "  v_fmac_f32_e64 v131, s42, v128\n" \
    "  v_maximum3_f32 v129, v131, 0, 0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s41\n" \
    "  v_fmac_f32_e64 v131, s42, v128\n" \
    "  v_mul_f32_e32 v130, 0x3ea2f983, v131\n" \
    "  v_rndne_f32_e32 v130, v130\n" \
    "  v_fmamk_f32 v128, v130, 0xc0490fdb, v131\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v130\n" \
    "  v_cvt_i32_f32_e32 v130, v130\n" \
    "  v_mul_f32_e32 v131, v128, v128\n" \
    "  v_fmaak_f32 v133, v131, v132, 0xb2d7322b\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3638ef1d\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xb9500d01\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3c088889\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v129, v128, v131\n" \
    "  v_fmac_f32_e32 v128, v129, v133\n" \
    "  v_lshl_add_u32 v129, v130, 31, v128\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s41\n" \
    "  v_fmac_f32_e64 v131, s42, v128\n" \
    "  v_mul_f32_e32 v129, v131, v131\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v129\n" \
    "  v_exp_f32_e32 v130, v129\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v130\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s41\n" \
    "  v_fmac_f32_e64 v131, s42, v128\n" \
    "  v_maximum3_f32 v129, v131, -v131, -v131\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_branch Ldone%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  v_mov_b32_e32 v128, 0\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v128, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v128, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v128, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v128, v0, s51\n" \
    "  s_set_gpr_idx_idx s52\n" \
    "  v_fmac_f32_e64 v128, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_fmac_f32_e64 v128, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v128, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v128, v0, s51\n" \
    "  s_set_gpr_idx_idx s52\n" \
    "  v_fmac_f32_e64 v128, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_fmac_f32_e64 v128, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_branch Lovs_A%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v130, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v130, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v130, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v130, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v130, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_branch Lovp_A%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v130, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v130, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v130, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v130, v0, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v130, v0, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v130, v0, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_branch Lovm_A%=\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s41, v128\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s41, v128\n" \
    "  v_mul_f32_e32 v129, 0x4038aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v130, v130\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v129, v130, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s41, v128\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v129, v130\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s41, v128\n" \
    "  v_maximum3_f32 v129, v131, 0, 0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s41, v128\n" \
    "  v_mul_f32_e32 v130, 0x3ea2f983, v131\n" \
    "  v_rndne_f32_e32 v130, v130\n" \
    "  v_fmamk_f32 v128, v130, 0xc0490fdb, v131\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v130\n" \
    "  v_cvt_i32_f32_e32 v130, v130\n" \
    "  v_mul_f32_e32 v131, v128, v128\n" \
    "  v_fmaak_f32 v133, v131, v132, 0xb2d7322b\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3638ef1d\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xb9500d01\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3c088889\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v129, v128, v131\n" \
    "  v_fmac_f32_e32 v128, v129, v133\n" \
    "  v_lshl_add_u32 v129, v130, 31, v128\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s41, v128\n" \
    "  v_mul_f32_e32 v129, v131, v131\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v129\n" \
    "  v_exp_f32_e32 v130, v129\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v130\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s41, v128\n" \
    "  v_maximum3_f32 v129, v131, -v131, -v131\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovs_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Los_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v128, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_fmac_f32_e64 v128, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovds_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v128, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_fmac_f32_e64 v128, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovds_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Los_A%=\n" \
    "Lovds_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovp_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lop_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v130, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdp_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v130, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdp_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lop_A%=\n" \
    "Lovdp_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovm_A%=:\n" \
    "  s_and_b32 s87, s43, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lom_A%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v130, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdm_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v130, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdm_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lom_A%=\n" \
    "Lovdm_A%=:\n" \
    "  s_lshr_b32 s88, s40, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "Ltab_B%=:\n" \
    "  v_mov_b32_e32 v131, s57\n" \
    "  v_fmac_f32_e64 v131, s58, v128\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s57\n" \
    "  v_fmac_f32_e64 v131, s58, v128\n" \
    "  v_mul_f32_e32 v129, 0x4038aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v130, v130\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v129, v130, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s57\n" \
    "  v_fmac_f32_e64 v131, s58, v128\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v129, v130\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s57\n" \
    "  v_fmac_f32_e64 v131, s58, v128\n" \
    "  v_maximum3_f32 v129, v131, 0, 0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s57\n" \
    "  v_fmac_f32_e64 v131, s58, v128\n" \
    "  v_mul_f32_e32 v130, 0x3ea2f983, v131\n" \
    "  v_rndne_f32_e32 v130, v130\n" \
    "  v_fmamk_f32 v128, v130, 0xc0490fdb, v131\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v130\n" \
    "  v_cvt_i32_f32_e32 v130, v130\n" \
    "  v_mul_f32_e32 v131, v128, v128\n" \
    "  v_fmaak_f32 v133, v131, v132, 0xb2d7322b\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3638ef1d\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xb9500d01\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3c088889\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v129, v128, v131\n" \
    "  v_fmac_f32_e32 v128, v129, v133\n" \
    "  v_lshl_add_u32 v129, v130, 31, v128\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s57\n" \
    "  v_fmac_f32_e64 v131, s58, v128\n" \
    "  v_mul_f32_e32 v129, v131, v131\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v129\n" \
    "  v_exp_f32_e32 v130, v129\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v130\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_mov_b32_e32 v131, s57\n" \
    "  v_fmac_f32_e64 v131, s58, v128\n" \
    "  v_maximum3_f32 v129, v131, -v131, -v131\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_branch Ldone%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  v_mov_b32_e32 v128, 0\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v128, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v128, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v128, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v128, v0, s67\n" \
    "  s_set_gpr_idx_idx s68\n" \
    "  v_fmac_f32_e64 v128, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_fmac_f32_e64 v128, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v128, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v128, v0, s67\n" \
    "  s_set_gpr_idx_idx s68\n" \
    "  v_fmac_f32_e64 v128, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_fmac_f32_e64 v128, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_branch Lovs_B%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v130, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v130, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v130, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v130, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v130, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_branch Lovp_B%=\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v130, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v130, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v130, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v130, v0, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v129, v130, v130\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v130, v0, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v130, v0, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_branch Lovm_B%=\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s57, v128\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v131\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s57, v128\n" \
    "  v_mul_f32_e32 v129, 0x4038aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v130, v130\n" \
    "  s_nop 0\n" \
    "  v_fma_f32 v129, v130, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s57, v128\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v131\n" \
    "  v_exp_f32_e32 v129, v129\n" \
    "  s_nop 0\n" \
    "  v_add_f32_e32 v130, 1.0, v129\n" \
    "  v_rcp_f32_e32 v129, v130\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s57, v128\n" \
    "  v_maximum3_f32 v129, v131, 0, 0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s57, v128\n" \
    "  v_mul_f32_e32 v130, 0x3ea2f983, v131\n" \
    "  v_rndne_f32_e32 v130, v130\n" \
    "  v_fmamk_f32 v128, v130, 0xc0490fdb, v131\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v130\n" \
    "  v_cvt_i32_f32_e32 v130, v130\n" \
    "  v_mul_f32_e32 v131, v128, v128\n" \
    "  v_fmaak_f32 v133, v131, v132, 0xb2d7322b\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3638ef1d\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xb9500d01\n" \
    "  v_fmaak_f32 v133, v131, v133, 0x3c088889\n" \
    "  v_fmaak_f32 v133, v131, v133, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v129, v128, v131\n" \
    "  v_fmac_f32_e32 v128, v129, v133\n" \
    "  v_lshl_add_u32 v129, v130, 31, v128\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s57, v128\n" \
    "  v_mul_f32_e32 v129, v131, v131\n" \
    "  v_mul_f32_e32 v129, 0xbfb8aa3b, v129\n" \
    "  v_exp_f32_e32 v130, v129\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v130\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 8\n" \
    "  v_add_f32_e32 v131, s57, v128\n" \
    "  v_maximum3_f32 v129, v131, -v131, -v131\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v64, v129\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 16\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovs_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Los_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v128, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_fmac_f32_e64 v128, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovds_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v128, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_fmac_f32_e64 v128, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovds_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Los_B%=\n" \
    "Lovds_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovp_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lop_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v130, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdp_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v130, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v129\n" \
    "  v_mul_f32_e32 v128, v128, v130\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdp_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lop_B%=\n" \
    "Lovdp_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Lovm_B%=:\n" \
    "  s_and_b32 s87, s59, 0x3fff\n" \
    "  s_sub_u32 s87, s87, 3\n" \
    "  s_mov_b64 s[82:83], s[84:85]\n" \
    "  s_lshl_b32 s89, s87, 4\n" \
    "  s_add_u32 s84, s84, s89\n" \
    "  s_addc_u32 s85, s85, 0\n" \
    "Lom_B%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s72, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v130, v0, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdm_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v129, v0, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v130, v0, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v129, v130\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdm_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lom_B%=\n" \
    "Lovdm_B%=:\n" \
    "  s_lshr_b32 s88, s56, 16\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "Ldone%=:\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_sub_u32 s91, s91, 1\n" \
    "  s_cmp_eq_u32 s91, 0\n" \
    "  s_cbranch_scc1 Lsw_done%=\n" \
    "  s_add_u32 s41, %[n], %[ni]\n" \
    "  v_mov_b32_e32 v0, v64\n" \
    "  v_mov_b32_e32 v1, v65\n" \
    "  v_mov_b32_e32 v2, v66\n" \
    "  v_mov_b32_e32 v3, v67\n" \
    "  v_mov_b32_e32 v4, v68\n" \
    "  v_mov_b32_e32 v5, v69\n" \
    "  v_mov_b32_e32 v6, v70\n" \
    "  v_mov_b32_e32 v7, v71\n" \
    "  s_cmp_le_u32 s41, 8\n" \
    "  s_cbranch_scc1 Lcp%=\n" \
    "  v_mov_b32_e32 v8, v72\n" \
    "  v_mov_b32_e32 v9, v73\n" \
    "  v_mov_b32_e32 v10, v74\n" \
    "  v_mov_b32_e32 v11, v75\n" \
    "  v_mov_b32_e32 v12, v76\n" \
    "  v_mov_b32_e32 v13, v77\n" \
    "  v_mov_b32_e32 v14, v78\n" \
    "  v_mov_b32_e32 v15, v79\n" \
    "  s_cmp_le_u32 s41, 16\n" \
    "  s_cbranch_scc1 Lcp%=\n" \
    "  v_mov_b32_e32 v16, v80\n" \
    "  v_mov_b32_e32 v17, v81\n" \
    "  v_mov_b32_e32 v18, v82\n" \
    "  v_mov_b32_e32 v19, v83\n" \
    "  v_mov_b32_e32 v20, v84\n" \
    "  v_mov_b32_e32 v21, v85\n" \
    "  v_mov_b32_e32 v22, v86\n" \
    "  v_mov_b32_e32 v23, v87\n" \
    "  s_cmp_le_u32 s41, 24\n" \
    "  s_cbranch_scc1 Lcp%=\n" \
    "  v_mov_b32_e32 v24, v88\n" \
    "  v_mov_b32_e32 v25, v89\n" \
    "  v_mov_b32_e32 v26, v90\n" \
    "  v_mov_b32_e32 v27, v91\n" \
    "  v_mov_b32_e32 v28, v92\n" \
    "  v_mov_b32_e32 v29, v93\n" \
    "  v_mov_b32_e32 v30, v94\n" \
    "  v_mov_b32_e32 v31, v95\n" \
    "  s_cmp_le_u32 s41, 32\n" \
    "  s_cbranch_scc1 Lcp%=\n" \
    "  v_mov_b32_e32 v32, v96\n" \
    "  v_mov_b32_e32 v33, v97\n" \
    "  v_mov_b32_e32 v34, v98\n" \
    "  v_mov_b32_e32 v35, v99\n" \
    "  v_mov_b32_e32 v36, v100\n" \
    "  v_mov_b32_e32 v37, v101\n" \
    "  v_mov_b32_e32 v38, v102\n" \
    "  v_mov_b32_e32 v39, v103\n" \
    "  s_cmp_le_u32 s41, 40\n" \
    "  s_cbranch_scc1 Lcp%=\n" \
    "  v_mov_b32_e32 v40, v104\n" \
    "  v_mov_b32_e32 v41, v105\n" \
    "  v_mov_b32_e32 v42, v106\n" \
    "  v_mov_b32_e32 v43, v107\n" \
    "  v_mov_b32_e32 v44, v108\n" \
    "  v_mov_b32_e32 v45, v109\n" \
    "  v_mov_b32_e32 v46, v110\n" \
    "  v_mov_b32_e32 v47, v111\n" \
    "  s_cmp_le_u32 s41, 48\n" \
    "  s_cbranch_scc1 Lcp%=\n" \
    "  v_mov_b32_e32 v48, v112\n" \
    "  v_mov_b32_e32 v49, v113\n" \
    "  v_mov_b32_e32 v50, v114\n" \
    "  v_mov_b32_e32 v51, v115\n" \
    "  v_mov_b32_e32 v52, v116\n" \
    "  v_mov_b32_e32 v53, v117\n" \
    "  v_mov_b32_e32 v54, v118\n" \
    "  v_mov_b32_e32 v55, v119\n" \
    "  s_cmp_le_u32 s41, 56\n" \
    "  s_cbranch_scc1 Lcp%=\n" \
    "  v_mov_b32_e32 v56, v120\n" \
    "  v_mov_b32_e32 v57, v121\n" \
    "  v_mov_b32_e32 v58, v122\n" \
    "  v_mov_b32_e32 v59, v123\n" \
    "  v_mov_b32_e32 v60, v124\n" \
    "  v_mov_b32_e32 v61, v125\n" \
    "  v_mov_b32_e32 v62, v126\n" \
    "  v_mov_b32_e32 v63, v127\n" \
    "Lcp%=:\n" \
    "  s_branch Lsw%=\n" \
    "Lsw_done%=:\n" \
    "  s_mov_b64 s[44:45], %[outs]\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_lshl_b32 s41, %[no], 2\n" \
    "  v_mul_u32_u24_e32 v136, s41, %[lane]\n" \
    "  v_add_u32_e32 v136, %[om0], v136\n" \
    "Lout%=:\n" \
    "  s_load_dwordx8 s[48:55], s[44:45], 0x0\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v128, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v128 offset:0\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s49, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v129, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v129 offset:4\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s50, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v130, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v130 offset:8\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s51, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v131, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v131 offset:12\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v132, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v132 offset:16\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s53, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v133, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v133 offset:20\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s54, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v134, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v134 offset:24\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s55, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v135, v64\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v136, v135 offset:28\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  v_add_u32_e32 v136, 32, v136\n" \
    "  s_add_u32 s44, s44, 32\n" \
    "  s_addc_u32 s45, s45, 0\n" \
    "  s_branch Lout%=\n" \
    "Lout_done%=:\n" \
    "  s_mov_b32 m0, s90\n"

#define NEAT_CLOB_S1_64R \
    "v0", "v1", "v2", "v3", "v4", "v5", "v6", "v7", "v8", "v9", "v10", "v11", \
    "v12", "v13", "v14", "v15", "v16", "v17", "v18", "v19", "v20", "v21", "v22", "v23", \
    "v24", "v25", "v26", "v27", "v28", "v29", "v30", "v31", "v32", "v33", "v34", "v35", \
    "v36", "v37", "v38", "v39", "v40", "v41", "v42", "v43", "v44", "v45", "v46", "v47", \
    "v48", "v49", "v50", "v51", "v52", "v53", "v54", "v55", "v56", "v57", "v58", "v59", \
    "v60", "v61", "v62", "v63", "v64", "v65", "v66", "v67", "v68", "v69", "v70", "v71", \
    "v72", "v73", "v74", "v75", "v76", "v77", "v78", "v79", "v80", "v81", "v82", "v83", \
    "v84", "v85", "v86", "v87", "v88", "v89", "v90", "v91", "v92", "v93", "v94", "v95", \
    "v96", "v97", "v98", "v99", "v100", "v101", "v102", "v103", "v104", "v105", "v106", "v107", \
    "v108", "v109", "v110", "v111", "v112", "v113", "v114", "v115", "v116", "v117", "v118", "v119", \
    "v120", "v121", "v122", "v123", "v124", "v125", "v126", "v127", "v128", "v129", "v130", "v131", \
    "v132", "v133", "v134", "v135", "v136", "v137", "v138", "v139", "s40", "s41", "s42", "s43", \
    "s44", "s45", "s46", "s47", "s48", "s49", "s50", "s51", "s52", "s53", "s54", "s55", \
    "s56", "s57", "s58", "s59", "s60", "s61", "s62", "s63", "s64", "s65", "s66", "s67", \
    "s68", "s69", "s70", "s71", "s72", "s73", "s74", "s75", "s76", "s77", "s78", "s79", \
    "s80", "s81", "s82", "s83", "s84", "s85", "s86", "s87", "s88", "s89", "s90", "s91", \
    "s92", "s93", "s94", "s95", "vcc", "scc"

#define NEAT_SCRATCH_S1_64R 128

