// node_loop_wide.h -- GENERATED by gen_node_loop.py; edit that script.
//
// Tile blocks as in node_loop_asm.h (which describes them) for populations
// of few node rows, with more samples per lane or fewer value registers.
#pragma once

// S4_32: 4 sample(s) per lane, value vectors at v0, v32, v64, v96, scratch v128..v149

#define NEAT_TILE_S4_32 \
    "  s_mov_b32 s90, m0\n" \
    "  s_lshl_b32 s41, %[ni], 2\n" \
    "  v_mul_u32_u24_e32 v144, s41, %[lane]\n" \
    "  v_add_u32_e32 v144, %[dm0], v144\n" \
    "  s_lshl_b32 s41, %[ni], 8\n" \
    "  v_add_u32_e32 v145, s41, v144\n" \
    "  v_add_u32_e32 v146, s41, v145\n" \
    "  v_add_u32_e32 v147, s41, v146\n" \
    "  s_mov_b32 s40, 0\n" \
    "  s_cmp_eq_u32 %[ni], 0\n" \
    "  s_cbranch_scc1 Lpl_done%=\n" \
    "Lpl%=:\n" \
    "  ds_read2_b32 v[128:129], v144 offset0:0 offset1:1\n" \
    "  ds_read2_b32 v[130:131], v144 offset0:2 offset1:3\n" \
    "  ds_read2_b32 v[132:133], v145 offset0:0 offset1:1\n" \
    "  ds_read2_b32 v[134:135], v145 offset0:2 offset1:3\n" \
    "  ds_read2_b32 v[136:137], v146 offset0:0 offset1:1\n" \
    "  ds_read2_b32 v[138:139], v146 offset0:2 offset1:3\n" \
    "  ds_read2_b32 v[140:141], v147 offset0:0 offset1:1\n" \
    "  ds_read2_b32 v[142:143], v147 offset0:2 offset1:3\n" \
    "  v_add_u32_e32 v144, 16, v144\n" \
    "  v_add_u32_e32 v145, 16, v145\n" \
    "  v_add_u32_e32 v146, 16, v146\n" \
    "  v_add_u32_e32 v147, 16, v147\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v128\n" \
    "  v_mov_b32_e32 v1, v129\n" \
    "  v_mov_b32_e32 v2, v130\n" \
    "  v_mov_b32_e32 v3, v131\n" \
    "  v_mov_b32_e32 v32, v132\n" \
    "  v_mov_b32_e32 v33, v133\n" \
    "  v_mov_b32_e32 v34, v134\n" \
    "  v_mov_b32_e32 v35, v135\n" \
    "  v_mov_b32_e32 v64, v136\n" \
    "  v_mov_b32_e32 v65, v137\n" \
    "  v_mov_b32_e32 v66, v138\n" \
    "  v_mov_b32_e32 v67, v139\n" \
    "  v_mov_b32_e32 v96, v140\n" \
    "  v_mov_b32_e32 v97, v141\n" \
    "  v_mov_b32_e32 v98, v142\n" \
    "  v_mov_b32_e32 v99, v143\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_add_u32 s40, s40, 4\n" \
    "  s_cmp_lt_u32 s40, %[ni]\n" \
    "  s_cbranch_scc1 Lpl%=\n" \
    "Lpl_done%=:\n" \
    "  s_set_gpr_idx_on %[zs], gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, 0\n" \
    "  v_mov_b32_e32 v1, 1.0\n" \
    "  v_mov_b32_e32 v32, 0\n" \
    "  v_mov_b32_e32 v33, 1.0\n" \
    "  v_mov_b32_e32 v64, 0\n" \
    "  v_mov_b32_e32 v65, 1.0\n" \
    "  v_mov_b32_e32 v96, 0\n" \
    "  v_mov_b32_e32 v97, 1.0\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 %[dn], 0\n" \
    "  s_cbranch_scc1 Ldma_done%=\n" \
    "  s_mov_b64 s[42:43], exec\n" \
    "  s_cmp_eq_u32 %[dvec], 0\n" \
    "  s_cselect_b32 s41, 2, 4\n" \
    "  v_lshlrev_b32_e32 v148, s41, %[lane]\n" \
    "  v_mov_b32_e32 v149, 0\n" \
    "  v_lshl_add_u64 v[148:149], v[148:149], 0, %[dsrc]\n" \
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
    "  global_load_lds_dwordx4 v[148:149], off nt\n" \
    "  s_mov_b64 exec, s[42:43]\n" \
    "  v_lshl_add_u64 v[148:149], v[148:149], 0, s[46:47]\n" \
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
    "  global_load_lds_dword v[148:149], off nt\n" \
    "  s_mov_b64 exec, s[42:43]\n" \
    "  v_lshl_add_u64 v[148:149], v[148:149], 0, s[46:47]\n" \
    "  s_add_u32 m0, m0, 256\n" \
    "  s_add_u32 s40, s40, 64\n" \
    "  s_cmp_lt_u32 s40, %[dn]\n" \
    "  s_cbranch_scc1 Ldl1%=\n" \
    "  s_branch Ldma_done%=\n" \
    "Ldma_done%=:\n" \
    "  s_mov_b64 s[80:81], %[rec]\n" \
    "  s_mov_b64 s[84:85], %[edg]\n" \
    "  s_mov_b32 s86, 0\n" \
    "  v_mov_b32_e32 v144, 0x2f309231\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], 0x0\n" \
    "  s_getpc_b64 s[92:93]\n" \
    "Lpc%=:\n" \
    "  s_add_u32 s94, s92, Ltab_B%= - Lpc%=\n" \
    "  s_addc_u32 s95, s93, 0\n" \
    "  s_add_u32 s92, s92, Ltab_A%= - Lpc%=\n" \
    "  s_addc_u32 s93, s93, 0\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "Ltab_A%=:\n" \
    "  v_mov_b32_e32 v140, s41\n" \
    "  v_mov_b32_e32 v141, s41\n" \
    "  v_mov_b32_e32 v142, s41\n" \
    "  v_mov_b32_e32 v143, s41\n" \
    "  v_fmac_f32_e64 v140, s42, v128\n" \
    "  v_fmac_f32_e64 v141, s42, v129\n" \
    "  v_fmac_f32_e64 v142, s42, v130\n" \
    "  v_fmac_f32_e64 v143, s42, v131\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v140\n" \
    "  v_mov_b32_e32 v32, v141\n" \
    "  v_mov_b32_e32 v64, v142\n" \
    "  v_mov_b32_e32 v96, v143\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_mov_b32_e32 v140, s41\n" \
    "  v_mov_b32_e32 v141, s41\n" \
    "  v_mov_b32_e32 v142, s41\n" \
    "  v_mov_b32_e32 v143, s41\n" \
    "  v_fmac_f32_e64 v140, s42, v128\n" \
    "  v_fmac_f32_e64 v141, s42, v129\n" \
    "  v_fmac_f32_e64 v142, s42, v130\n" \
    "  v_fmac_f32_e64 v143, s42, v131\n" \
    "  v_mul_f32_e32 v132, 0x4038aa3b, v140\n" \
    "  v_mul_f32_e32 v133, 0x4038aa3b, v141\n" \
    "  v_mul_f32_e32 v134, 0x4038aa3b, v142\n" \
    "  v_mul_f32_e32 v135, 0x4038aa3b, v143\n" \
    "  v_exp_f32_e32 v132, v132\n" \
    "  v_exp_f32_e32 v133, v133\n" \
    "  v_exp_f32_e32 v134, v134\n" \
    "  v_exp_f32_e32 v135, v135\n" \
    "  v_add_f32_e32 v136, 1.0, v132\n" \
    "  v_add_f32_e32 v137, 1.0, v133\n" \
    "  v_add_f32_e32 v138, 1.0, v134\n" \
    "  v_add_f32_e32 v139, 1.0, v135\n" \
    "  v_rcp_f32_e32 v136, v136\n" \
    "  v_rcp_f32_e32 v137, v137\n" \
    "  v_rcp_f32_e32 v138, v138\n" \
    "  v_rcp_f32_e32 v139, v139\n" \
    "  v_fma_f32 v132, v136, -2.0, 1.0\n" \
    "  v_fma_f32 v133, v137, -2.0, 1.0\n" \
    "  v_fma_f32 v134, v138, -2.0, 1.0\n" \
    "  v_fma_f32 v135, v139, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_mov_b32_e32 v140, s41\n" \
    "  v_mov_b32_e32 v141, s41\n" \
    "  v_mov_b32_e32 v142, s41\n" \
    "  v_mov_b32_e32 v143, s41\n" \
    "  v_fmac_f32_e64 v140, s42, v128\n" \
    "  v_fmac_f32_e64 v141, s42, v129\n" \
    "  v_fmac_f32_e64 v142, s42, v130\n" \
    "  v_fmac_f32_e64 v143, s42, v131\n" \
    "  v_mul_f32_e32 v132, 0xbfb8aa3b, v140\n" \
    "  v_mul_f32_e32 v133, 0xbfb8aa3b, v141\n" \
    "  v_mul_f32_e32 v134, 0xbfb8aa3b, v142\n" \
    "  v_mul_f32_e32 v135, 0xbfb8aa3b, v143\n" \
    "  v_exp_f32_e32 v132, v132\n" \
    "  v_exp_f32_e32 v133, v133\n" \
    "  v_exp_f32_e32 v134, v134\n" \
    "  v_exp_f32_e32 v135, v135\n" \
    "  v_add_f32_e32 v136, 1.0, v132\n" \
    "  v_add_f32_e32 v137, 1.0, v133\n" \
    "  v_add_f32_e32 v138, 1.0, v134\n" \
    "  v_add_f32_e32 v139, 1.0, v135\n" \
    "  v_rcp_f32_e32 v132, v136\n" \
    "  v_rcp_f32_e32 v133, v137\n" \
    "  v_rcp_f32_e32 v134, v138\n" \
    "  v_rcp_f32_e32 v135, v139\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_mov_b32_e32 v140, s41\n" \
    "  v_mov_b32_e32 v141, s41\n" \
    "  v_mov_b32_e32 v142, s41\n" \
    "  v_mov_b32_e32 v143, s41\n" \
    "  v_fmac_f32_e64 v140, s42, v128\n" \
    "  v_fmac_f32_e64 v141, s42, v129\n" \
    "  v_fmac_f32_e64 v142, s42, v130\n" \
    "  v_fmac_f32_e64 v143, s42, v131\n" \
    "  v_maximum3_f32 v132, v140, 0, 0\n" \
    "  v_maximum3_f32 v133, v141, 0, 0\n" \
    "  v_maximum3_f32 v134, v142, 0, 0\n" \
    "  v_maximum3_f32 v135, v143, 0, 0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_mov_b32_e32 v140, s41\n" \
    "  v_mov_b32_e32 v141, s41\n" \
    "  v_mov_b32_e32 v142, s41\n" \
    "  v_mov_b32_e32 v143, s41\n" \
    "  v_fmac_f32_e64 v140, s42, v128\n" \
    "  v_fmac_f32_e64 v141, s42, v129\n" \
    "  v_fmac_f32_e64 v142, s42, v130\n" \
    "  v_fmac_f32_e64 v143, s42, v131\n" \
    "  v_mul_f32_e32 v136, 0x3ea2f983, v140\n" \
    "  v_mul_f32_e32 v137, 0x3ea2f983, v141\n" \
    "  v_mul_f32_e32 v138, 0x3ea2f983, v142\n" \
    "  v_mul_f32_e32 v139, 0x3ea2f983, v143\n" \
    "  v_rndne_f32_e32 v136, v136\n" \
    "  v_rndne_f32_e32 v137, v137\n" \
    "  v_rndne_f32_e32 v138, v138\n" \
    "  v_rndne_f32_e32 v139, v139\n" \
    "  v_fmamk_f32 v128, v136, 0xc0490fdb, v140\n" \
    "  v_fmamk_f32 v129, v137, 0xc0490fdb, v141\n" \
    "  v_fmamk_f32 v130, v138, 0xc0490fdb, v142\n" \
    "  v_fmamk_f32 v131, v139, 0xc0490fdb, v143\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v136\n" \
    "  v_fmac_f32_e32 v129, 0x33bbbd2e, v137\n" \
    "  v_fmac_f32_e32 v130, 0x33bbbd2e, v138\n" \
    "  v_fmac_f32_e32 v131, 0x33bbbd2e, v139\n" \
    "  v_cvt_i32_f32_e32 v136, v136\n" \
    "  v_cvt_i32_f32_e32 v137, v137\n" \
    "  v_cvt_i32_f32_e32 v138, v138\n" \
    "  v_cvt_i32_f32_e32 v139, v139\n" \
    "  v_mul_f32_e32 v140, v128, v128\n" \
    "  v_mul_f32_e32 v141, v129, v129\n" \
    "  v_mul_f32_e32 v142, v130, v130\n" \
    "  v_mul_f32_e32 v143, v131, v131\n" \
    "  v_fmaak_f32 v145, v140, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v146, v141, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v147, v142, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v148, v143, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v145, v140, v145, 0x3638ef1d\n" \
    "  v_fmaak_f32 v146, v141, v146, 0x3638ef1d\n" \
    "  v_fmaak_f32 v147, v142, v147, 0x3638ef1d\n" \
    "  v_fmaak_f32 v148, v143, v148, 0x3638ef1d\n" \
    "  v_fmaak_f32 v145, v140, v145, 0xb9500d01\n" \
    "  v_fmaak_f32 v146, v141, v146, 0xb9500d01\n" \
    "  v_fmaak_f32 v147, v142, v147, 0xb9500d01\n" \
    "  v_fmaak_f32 v148, v143, v148, 0xb9500d01\n" \
    "  v_fmaak_f32 v145, v140, v145, 0x3c088889\n" \
    "  v_fmaak_f32 v146, v141, v146, 0x3c088889\n" \
    "  v_fmaak_f32 v147, v142, v147, 0x3c088889\n" \
    "  v_fmaak_f32 v148, v143, v148, 0x3c088889\n" \
    "  v_fmaak_f32 v145, v140, v145, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v146, v141, v146, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v147, v142, v147, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v148, v143, v148, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v132, v128, v140\n" \
    "  v_mul_f32_e32 v133, v129, v141\n" \
    "  v_mul_f32_e32 v134, v130, v142\n" \
    "  v_mul_f32_e32 v135, v131, v143\n" \
    "  v_fmac_f32_e32 v128, v132, v145\n" \
    "  v_fmac_f32_e32 v129, v133, v146\n" \
    "  v_fmac_f32_e32 v130, v134, v147\n" \
    "  v_fmac_f32_e32 v131, v135, v148\n" \
    "  v_lshl_add_u32 v132, v136, 31, v128\n" \
    "  v_lshl_add_u32 v133, v137, 31, v129\n" \
    "  v_lshl_add_u32 v134, v138, 31, v130\n" \
    "  v_lshl_add_u32 v135, v139, 31, v131\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_mov_b32_e32 v140, s41\n" \
    "  v_mov_b32_e32 v141, s41\n" \
    "  v_mov_b32_e32 v142, s41\n" \
    "  v_mov_b32_e32 v143, s41\n" \
    "  v_fmac_f32_e64 v140, s42, v128\n" \
    "  v_fmac_f32_e64 v141, s42, v129\n" \
    "  v_fmac_f32_e64 v142, s42, v130\n" \
    "  v_fmac_f32_e64 v143, s42, v131\n" \
    "  v_mul_f32_e32 v132, v140, v140\n" \
    "  v_mul_f32_e32 v133, v141, v141\n" \
    "  v_mul_f32_e32 v134, v142, v142\n" \
    "  v_mul_f32_e32 v135, v143, v143\n" \
    "  v_mul_f32_e32 v132, 0xbfb8aa3b, v132\n" \
    "  v_mul_f32_e32 v133, 0xbfb8aa3b, v133\n" \
    "  v_mul_f32_e32 v134, 0xbfb8aa3b, v134\n" \
    "  v_mul_f32_e32 v135, 0xbfb8aa3b, v135\n" \
    "  v_exp_f32_e32 v136, v132\n" \
    "  v_exp_f32_e32 v137, v133\n" \
    "  v_exp_f32_e32 v138, v134\n" \
    "  v_exp_f32_e32 v139, v135\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v136\n" \
    "  v_mov_b32_e32 v32, v137\n" \
    "  v_mov_b32_e32 v64, v138\n" \
    "  v_mov_b32_e32 v96, v139\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_mov_b32_e32 v140, s41\n" \
    "  v_mov_b32_e32 v141, s41\n" \
    "  v_mov_b32_e32 v142, s41\n" \
    "  v_mov_b32_e32 v143, s41\n" \
    "  v_fmac_f32_e64 v140, s42, v128\n" \
    "  v_fmac_f32_e64 v141, s42, v129\n" \
    "  v_fmac_f32_e64 v142, s42, v130\n" \
    "  v_fmac_f32_e64 v143, s42, v131\n" \
    "  v_maximum3_f32 v132, v140, -v140, -v140\n" \
    "  v_maximum3_f32 v133, v141, -v141, -v141\n" \
    "  v_maximum3_f32 v134, v142, -v142, -v142\n" \
    "  v_maximum3_f32 v135, v143, -v143, -v143\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_branch Ldone%=\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  v_mov_b32_e32 v128, 0\n" \
    "  v_mov_b32_e32 v129, 0\n" \
    "  v_mov_b32_e32 v130, 0\n" \
    "  v_mov_b32_e32 v131, 0\n" \
    "  s_lshr_b32 s88, s40, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v32, s45\n" \
    "  v_mul_f32_e64 v130, v64, s45\n" \
    "  v_mul_f32_e64 v131, v96, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  v_fmac_f32_e64 v129, v32, s47\n" \
    "  v_fmac_f32_e64 v130, v64, s47\n" \
    "  v_fmac_f32_e64 v131, v96, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v32, s45\n" \
    "  v_mul_f32_e64 v130, v64, s45\n" \
    "  v_mul_f32_e64 v131, v96, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  v_fmac_f32_e64 v129, v32, s47\n" \
    "  v_fmac_f32_e64 v130, v64, s47\n" \
    "  v_fmac_f32_e64 v131, v96, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v128, v0, s49\n" \
    "  v_fmac_f32_e64 v129, v32, s49\n" \
    "  v_fmac_f32_e64 v130, v64, s49\n" \
    "  v_fmac_f32_e64 v131, v96, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v128, v0, s51\n" \
    "  v_fmac_f32_e64 v129, v32, s51\n" \
    "  v_fmac_f32_e64 v130, v64, s51\n" \
    "  v_fmac_f32_e64 v131, v96, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v32, s45\n" \
    "  v_mul_f32_e64 v130, v64, s45\n" \
    "  v_mul_f32_e64 v131, v96, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  v_fmac_f32_e64 v129, v32, s47\n" \
    "  v_fmac_f32_e64 v130, v64, s47\n" \
    "  v_fmac_f32_e64 v131, v96, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v128, v0, s49\n" \
    "  v_fmac_f32_e64 v129, v32, s49\n" \
    "  v_fmac_f32_e64 v130, v64, s49\n" \
    "  v_fmac_f32_e64 v131, v96, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v128, v0, s51\n" \
    "  v_fmac_f32_e64 v129, v32, s51\n" \
    "  v_fmac_f32_e64 v130, v64, s51\n" \
    "  v_fmac_f32_e64 v131, v96, s51\n" \
    "  s_set_gpr_idx_idx s52\n" \
    "  v_fmac_f32_e64 v128, v0, s53\n" \
    "  v_fmac_f32_e64 v129, v32, s53\n" \
    "  v_fmac_f32_e64 v130, v64, s53\n" \
    "  v_fmac_f32_e64 v131, v96, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_fmac_f32_e64 v128, v0, s55\n" \
    "  v_fmac_f32_e64 v129, v32, s55\n" \
    "  v_fmac_f32_e64 v130, v64, s55\n" \
    "  v_fmac_f32_e64 v131, v96, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s40, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v32, s45\n" \
    "  v_mul_f32_e64 v130, v64, s45\n" \
    "  v_mul_f32_e64 v131, v96, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_fmac_f32_e64 v128, v0, s47\n" \
    "  v_fmac_f32_e64 v129, v32, s47\n" \
    "  v_fmac_f32_e64 v130, v64, s47\n" \
    "  v_fmac_f32_e64 v131, v96, s47\n" \
    "  s_set_gpr_idx_idx s48\n" \
    "  v_fmac_f32_e64 v128, v0, s49\n" \
    "  v_fmac_f32_e64 v129, v32, s49\n" \
    "  v_fmac_f32_e64 v130, v64, s49\n" \
    "  v_fmac_f32_e64 v131, v96, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_fmac_f32_e64 v128, v0, s51\n" \
    "  v_fmac_f32_e64 v129, v32, s51\n" \
    "  v_fmac_f32_e64 v130, v64, s51\n" \
    "  v_fmac_f32_e64 v131, v96, s51\n" \
    "  s_set_gpr_idx_idx s52\n" \
    "  v_fmac_f32_e64 v128, v0, s53\n" \
    "  v_fmac_f32_e64 v129, v32, s53\n" \
    "  v_fmac_f32_e64 v130, v64, s53\n" \
    "  v_fmac_f32_e64 v131, v96, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_fmac_f32_e64 v128, v0, s55\n" \
    "  v_fmac_f32_e64 v129, v32, s55\n" \
    "  v_fmac_f32_e64 v130, v64, s55\n" \
    "  v_fmac_f32_e64 v131, v96, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_branch Lovs_A%=\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v32, s45\n" \
    "  v_mul_f32_e64 v130, v64, s45\n" \
    "  v_mul_f32_e64 v131, v96, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v136, v0, s47\n" \
    "  v_mul_f32_e64 v137, v32, s47\n" \
    "  v_mul_f32_e64 v138, v64, s47\n" \
    "  v_mul_f32_e64 v139, v96, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_lshr_b32 s88, s40, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v32, s45\n" \
    "  v_mul_f32_e64 v130, v64, s45\n" \
    "  v_mul_f32_e64 v131, v96, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v136, v0, s47\n" \
    "  v_mul_f32_e64 v137, v32, s47\n" \
    "  v_mul_f32_e64 v138, v64, s47\n" \
    "  v_mul_f32_e64 v139, v96, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s49\n" \
    "  v_mul_f32_e64 v133, v32, s49\n" \
    "  v_mul_f32_e64 v134, v64, s49\n" \
    "  v_mul_f32_e64 v135, v96, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v136, v0, s51\n" \
    "  v_mul_f32_e64 v137, v32, s51\n" \
    "  v_mul_f32_e64 v138, v64, s51\n" \
    "  v_mul_f32_e64 v139, v96, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  v_mul_f32_e32 v130, v130, v134\n" \
    "  v_mul_f32_e32 v131, v131, v135\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_lshr_b32 s88, s40, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v32, s45\n" \
    "  v_mul_f32_e64 v130, v64, s45\n" \
    "  v_mul_f32_e64 v131, v96, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v136, v0, s47\n" \
    "  v_mul_f32_e64 v137, v32, s47\n" \
    "  v_mul_f32_e64 v138, v64, s47\n" \
    "  v_mul_f32_e64 v139, v96, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s49\n" \
    "  v_mul_f32_e64 v133, v32, s49\n" \
    "  v_mul_f32_e64 v134, v64, s49\n" \
    "  v_mul_f32_e64 v135, v96, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v136, v0, s51\n" \
    "  v_mul_f32_e64 v137, v32, s51\n" \
    "  v_mul_f32_e64 v138, v64, s51\n" \
    "  v_mul_f32_e64 v139, v96, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  v_mul_f32_e32 v130, v130, v134\n" \
    "  v_mul_f32_e32 v131, v131, v135\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s53\n" \
    "  v_mul_f32_e64 v133, v32, s53\n" \
    "  v_mul_f32_e64 v134, v64, s53\n" \
    "  v_mul_f32_e64 v135, v96, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v136, v0, s55\n" \
    "  v_mul_f32_e64 v137, v32, s55\n" \
    "  v_mul_f32_e64 v138, v64, s55\n" \
    "  v_mul_f32_e64 v139, v96, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  v_mul_f32_e32 v130, v130, v134\n" \
    "  v_mul_f32_e32 v131, v131, v135\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_lshr_b32 s88, s40, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s45\n" \
    "  v_mul_f32_e64 v129, v32, s45\n" \
    "  v_mul_f32_e64 v130, v64, s45\n" \
    "  v_mul_f32_e64 v131, v96, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v136, v0, s47\n" \
    "  v_mul_f32_e64 v137, v32, s47\n" \
    "  v_mul_f32_e64 v138, v64, s47\n" \
    "  v_mul_f32_e64 v139, v96, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s49\n" \
    "  v_mul_f32_e64 v133, v32, s49\n" \
    "  v_mul_f32_e64 v134, v64, s49\n" \
    "  v_mul_f32_e64 v135, v96, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v136, v0, s51\n" \
    "  v_mul_f32_e64 v137, v32, s51\n" \
    "  v_mul_f32_e64 v138, v64, s51\n" \
    "  v_mul_f32_e64 v139, v96, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  v_mul_f32_e32 v130, v130, v134\n" \
    "  v_mul_f32_e32 v131, v131, v135\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s53\n" \
    "  v_mul_f32_e64 v133, v32, s53\n" \
    "  v_mul_f32_e64 v134, v64, s53\n" \
    "  v_mul_f32_e64 v135, v96, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v136, v0, s55\n" \
    "  v_mul_f32_e64 v137, v32, s55\n" \
    "  v_mul_f32_e64 v138, v64, s55\n" \
    "  v_mul_f32_e64 v139, v96, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  v_mul_f32_e32 v130, v130, v134\n" \
    "  v_mul_f32_e32 v131, v131, v135\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_branch Lovp_A%=\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s45\n" \
    "  v_mul_f32_e64 v133, v32, s45\n" \
    "  v_mul_f32_e64 v134, v64, s45\n" \
    "  v_mul_f32_e64 v135, v96, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v136, v0, s47\n" \
    "  v_mul_f32_e64 v137, v32, s47\n" \
    "  v_mul_f32_e64 v138, v64, s47\n" \
    "  v_mul_f32_e64 v139, v96, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v132, v136, v136\n" \
    "  v_maximum3_f32 v129, v133, v137, v137\n" \
    "  v_maximum3_f32 v130, v134, v138, v138\n" \
    "  v_maximum3_f32 v131, v135, v139, v139\n" \
    "  s_lshr_b32 s88, s40, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s45\n" \
    "  v_mul_f32_e64 v133, v32, s45\n" \
    "  v_mul_f32_e64 v134, v64, s45\n" \
    "  v_mul_f32_e64 v135, v96, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v136, v0, s47\n" \
    "  v_mul_f32_e64 v137, v32, s47\n" \
    "  v_mul_f32_e64 v138, v64, s47\n" \
    "  v_mul_f32_e64 v139, v96, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v132, v136, v136\n" \
    "  v_maximum3_f32 v129, v133, v137, v137\n" \
    "  v_maximum3_f32 v130, v134, v138, v138\n" \
    "  v_maximum3_f32 v131, v135, v139, v139\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s49\n" \
    "  v_mul_f32_e64 v133, v32, s49\n" \
    "  v_mul_f32_e64 v134, v64, s49\n" \
    "  v_mul_f32_e64 v135, v96, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v136, v0, s51\n" \
    "  v_mul_f32_e64 v137, v32, s51\n" \
    "  v_mul_f32_e64 v138, v64, s51\n" \
    "  v_mul_f32_e64 v139, v96, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v132, v136\n" \
    "  v_maximum3_f32 v129, v129, v133, v137\n" \
    "  v_maximum3_f32 v130, v130, v134, v138\n" \
    "  v_maximum3_f32 v131, v131, v135, v139\n" \
    "  s_lshr_b32 s88, s40, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s45\n" \
    "  v_mul_f32_e64 v133, v32, s45\n" \
    "  v_mul_f32_e64 v134, v64, s45\n" \
    "  v_mul_f32_e64 v135, v96, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v136, v0, s47\n" \
    "  v_mul_f32_e64 v137, v32, s47\n" \
    "  v_mul_f32_e64 v138, v64, s47\n" \
    "  v_mul_f32_e64 v139, v96, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v132, v136, v136\n" \
    "  v_maximum3_f32 v129, v133, v137, v137\n" \
    "  v_maximum3_f32 v130, v134, v138, v138\n" \
    "  v_maximum3_f32 v131, v135, v139, v139\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s49\n" \
    "  v_mul_f32_e64 v133, v32, s49\n" \
    "  v_mul_f32_e64 v134, v64, s49\n" \
    "  v_mul_f32_e64 v135, v96, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v136, v0, s51\n" \
    "  v_mul_f32_e64 v137, v32, s51\n" \
    "  v_mul_f32_e64 v138, v64, s51\n" \
    "  v_mul_f32_e64 v139, v96, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v132, v136\n" \
    "  v_maximum3_f32 v129, v129, v133, v137\n" \
    "  v_maximum3_f32 v130, v130, v134, v138\n" \
    "  v_maximum3_f32 v131, v131, v135, v139\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s53\n" \
    "  v_mul_f32_e64 v133, v32, s53\n" \
    "  v_mul_f32_e64 v134, v64, s53\n" \
    "  v_mul_f32_e64 v135, v96, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v136, v0, s55\n" \
    "  v_mul_f32_e64 v137, v32, s55\n" \
    "  v_mul_f32_e64 v138, v64, s55\n" \
    "  v_mul_f32_e64 v139, v96, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v132, v136\n" \
    "  v_maximum3_f32 v129, v129, v133, v137\n" \
    "  v_maximum3_f32 v130, v130, v134, v138\n" \
    "  v_maximum3_f32 v131, v131, v135, v139\n" \
    "  s_lshr_b32 s88, s40, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[56:71], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s44, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s45\n" \
    "  v_mul_f32_e64 v133, v32, s45\n" \
    "  v_mul_f32_e64 v134, v64, s45\n" \
    "  v_mul_f32_e64 v135, v96, s45\n" \
    "  s_set_gpr_idx_idx s46\n" \
    "  v_mul_f32_e64 v136, v0, s47\n" \
    "  v_mul_f32_e64 v137, v32, s47\n" \
    "  v_mul_f32_e64 v138, v64, s47\n" \
    "  v_mul_f32_e64 v139, v96, s47\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v132, v136, v136\n" \
    "  v_maximum3_f32 v129, v133, v137, v137\n" \
    "  v_maximum3_f32 v130, v134, v138, v138\n" \
    "  v_maximum3_f32 v131, v135, v139, v139\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s49\n" \
    "  v_mul_f32_e64 v133, v32, s49\n" \
    "  v_mul_f32_e64 v134, v64, s49\n" \
    "  v_mul_f32_e64 v135, v96, s49\n" \
    "  s_set_gpr_idx_idx s50\n" \
    "  v_mul_f32_e64 v136, v0, s51\n" \
    "  v_mul_f32_e64 v137, v32, s51\n" \
    "  v_mul_f32_e64 v138, v64, s51\n" \
    "  v_mul_f32_e64 v139, v96, s51\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v132, v136\n" \
    "  v_maximum3_f32 v129, v129, v133, v137\n" \
    "  v_maximum3_f32 v130, v130, v134, v138\n" \
    "  v_maximum3_f32 v131, v131, v135, v139\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s53\n" \
    "  v_mul_f32_e64 v133, v32, s53\n" \
    "  v_mul_f32_e64 v134, v64, s53\n" \
    "  v_mul_f32_e64 v135, v96, s53\n" \
    "  s_set_gpr_idx_idx s54\n" \
    "  v_mul_f32_e64 v136, v0, s55\n" \
    "  v_mul_f32_e64 v137, v32, s55\n" \
    "  v_mul_f32_e64 v138, v64, s55\n" \
    "  v_mul_f32_e64 v139, v96, s55\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v132, v136\n" \
    "  v_maximum3_f32 v129, v129, v133, v137\n" \
    "  v_maximum3_f32 v130, v130, v134, v138\n" \
    "  v_maximum3_f32 v131, v131, v135, v139\n" \
    "  s_branch Lovm_A%=\n" \
    "  .p2align 9\n" \
    "  v_add_f32_e32 v140, s41, v128\n" \
    "  v_add_f32_e32 v141, s41, v129\n" \
    "  v_add_f32_e32 v142, s41, v130\n" \
    "  v_add_f32_e32 v143, s41, v131\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v140\n" \
    "  v_mov_b32_e32 v32, v141\n" \
    "  v_mov_b32_e32 v64, v142\n" \
    "  v_mov_b32_e32 v96, v143\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_add_f32_e32 v140, s41, v128\n" \
    "  v_add_f32_e32 v141, s41, v129\n" \
    "  v_add_f32_e32 v142, s41, v130\n" \
    "  v_add_f32_e32 v143, s41, v131\n" \
    "  v_mul_f32_e32 v132, 0x4038aa3b, v140\n" \
    "  v_mul_f32_e32 v133, 0x4038aa3b, v141\n" \
    "  v_mul_f32_e32 v134, 0x4038aa3b, v142\n" \
    "  v_mul_f32_e32 v135, 0x4038aa3b, v143\n" \
    "  v_exp_f32_e32 v132, v132\n" \
    "  v_exp_f32_e32 v133, v133\n" \
    "  v_exp_f32_e32 v134, v134\n" \
    "  v_exp_f32_e32 v135, v135\n" \
    "  v_add_f32_e32 v136, 1.0, v132\n" \
    "  v_add_f32_e32 v137, 1.0, v133\n" \
    "  v_add_f32_e32 v138, 1.0, v134\n" \
    "  v_add_f32_e32 v139, 1.0, v135\n" \
    "  v_rcp_f32_e32 v136, v136\n" \
    "  v_rcp_f32_e32 v137, v137\n" \
    "  v_rcp_f32_e32 v138, v138\n" \
    "  v_rcp_f32_e32 v139, v139\n" \
    "  v_fma_f32 v132, v136, -2.0, 1.0\n" \
    "  v_fma_f32 v133, v137, -2.0, 1.0\n" \
    "  v_fma_f32 v134, v138, -2.0, 1.0\n" \
    "  v_fma_f32 v135, v139, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_add_f32_e32 v140, s41, v128\n" \
    "  v_add_f32_e32 v141, s41, v129\n" \
    "  v_add_f32_e32 v142, s41, v130\n" \
    "  v_add_f32_e32 v143, s41, v131\n" \
    "  v_mul_f32_e32 v132, 0xbfb8aa3b, v140\n" \
    "  v_mul_f32_e32 v133, 0xbfb8aa3b, v141\n" \
    "  v_mul_f32_e32 v134, 0xbfb8aa3b, v142\n" \
    "  v_mul_f32_e32 v135, 0xbfb8aa3b, v143\n" \
    "  v_exp_f32_e32 v132, v132\n" \
    "  v_exp_f32_e32 v133, v133\n" \
    "  v_exp_f32_e32 v134, v134\n" \
    "  v_exp_f32_e32 v135, v135\n" \
    "  v_add_f32_e32 v136, 1.0, v132\n" \
    "  v_add_f32_e32 v137, 1.0, v133\n" \
    "  v_add_f32_e32 v138, 1.0, v134\n" \
    "  v_add_f32_e32 v139, 1.0, v135\n" \
    "  v_rcp_f32_e32 v132, v136\n" \
    "  v_rcp_f32_e32 v133, v137\n" \
    "  v_rcp_f32_e32 v134, v138\n" \
    "  v_rcp_f32_e32 v135, v139\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_add_f32_e32 v140, s41, v128\n" \
    "  v_add_f32_e32 v141, s41, v129\n" \
    "  v_add_f32_e32 v142, s41, v130\n" \
    "  v_add_f32_e32 v143, s41, v131\n" \
    "  v_maximum3_f32 v132, v140, 0, 0\n" \
    "  v_maximum3_f32 v133, v141, 0, 0\n" \
    "  v_maximum3_f32 v134, v142, 0, 0\n" \
    "  v_maximum3_f32 v135, v143, 0, 0\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_add_f32_e32 v140, s41, v128\n" \
    "  v_add_f32_e32 v141, s41, v129\n" \
    "  v_add_f32_e32 v142, s41, v130\n" \
    "  v_add_f32_e32 v143, s41, v131\n" \
    "  v_mul_f32_e32 v136, 0x3ea2f983, v140\n" \
    "  v_mul_f32_e32 v137, 0x3ea2f983, v141\n" \
    "  v_mul_f32_e32 v138, 0x3ea2f983, v142\n" \
    "  v_mul_f32_e32 v139, 0x3ea2f983, v143\n" \
    "  v_rndne_f32_e32 v136, v136\n" \
    "  v_rndne_f32_e32 v137, v137\n" \
    "  v_rndne_f32_e32 v138, v138\n" \
    "  v_rndne_f32_e32 v139, v139\n" \
    "  v_fmamk_f32 v128, v136, 0xc0490fdb, v140\n" \
    "  v_fmamk_f32 v129, v137, 0xc0490fdb, v141\n" \
    "  v_fmamk_f32 v130, v138, 0xc0490fdb, v142\n" \
    "  v_fmamk_f32 v131, v139, 0xc0490fdb, v143\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v136\n" \
    "  v_fmac_f32_e32 v129, 0x33bbbd2e, v137\n" \
    "  v_fmac_f32_e32 v130, 0x33bbbd2e, v138\n" \
    "  v_fmac_f32_e32 v131, 0x33bbbd2e, v139\n" \
    "  v_cvt_i32_f32_e32 v136, v136\n" \
    "  v_cvt_i32_f32_e32 v137, v137\n" \
    "  v_cvt_i32_f32_e32 v138, v138\n" \
    "  v_cvt_i32_f32_e32 v139, v139\n" \
    "  v_mul_f32_e32 v140, v128, v128\n" \
    "  v_mul_f32_e32 v141, v129, v129\n" \
    "  v_mul_f32_e32 v142, v130, v130\n" \
    "  v_mul_f32_e32 v143, v131, v131\n" \
    "  v_fmaak_f32 v145, v140, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v146, v141, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v147, v142, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v148, v143, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v145, v140, v145, 0x3638ef1d\n" \
    "  v_fmaak_f32 v146, v141, v146, 0x3638ef1d\n" \
    "  v_fmaak_f32 v147, v142, v147, 0x3638ef1d\n" \
    "  v_fmaak_f32 v148, v143, v148, 0x3638ef1d\n" \
    "  v_fmaak_f32 v145, v140, v145, 0xb9500d01\n" \
    "  v_fmaak_f32 v146, v141, v146, 0xb9500d01\n" \
    "  v_fmaak_f32 v147, v142, v147, 0xb9500d01\n" \
    "  v_fmaak_f32 v148, v143, v148, 0xb9500d01\n" \
    "  v_fmaak_f32 v145, v140, v145, 0x3c088889\n" \
    "  v_fmaak_f32 v146, v141, v146, 0x3c088889\n" \
    "  v_fmaak_f32 v147, v142, v147, 0x3c088889\n" \
    "  v_fmaak_f32 v148, v143, v148, 0x3c088889\n" \
    "  v_fmaak_f32 v145, v140, v145, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v146, v141, v146, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v147, v142, v147, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v148, v143, v148, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v132, v128, v140\n" \
    "  v_mul_f32_e32 v133, v129, v141\n" \
    "  v_mul_f32_e32 v134, v130, v142\n" \
    "  v_mul_f32_e32 v135, v131, v143\n" \
    "  v_fmac_f32_e32 v128, v132, v145\n" \
    "  v_fmac_f32_e32 v129, v133, v146\n" \
    "  v_fmac_f32_e32 v130, v134, v147\n" \
    "  v_fmac_f32_e32 v131, v135, v148\n" \
    "  v_lshl_add_u32 v132, v136, 31, v128\n" \
    "  v_lshl_add_u32 v133, v137, 31, v129\n" \
    "  v_lshl_add_u32 v134, v138, 31, v130\n" \
    "  v_lshl_add_u32 v135, v139, 31, v131\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_add_f32_e32 v140, s41, v128\n" \
    "  v_add_f32_e32 v141, s41, v129\n" \
    "  v_add_f32_e32 v142, s41, v130\n" \
    "  v_add_f32_e32 v143, s41, v131\n" \
    "  v_mul_f32_e32 v132, v140, v140\n" \
    "  v_mul_f32_e32 v133, v141, v141\n" \
    "  v_mul_f32_e32 v134, v142, v142\n" \
    "  v_mul_f32_e32 v135, v143, v143\n" \
    "  v_mul_f32_e32 v132, 0xbfb8aa3b, v132\n" \
    "  v_mul_f32_e32 v133, 0xbfb8aa3b, v133\n" \
    "  v_mul_f32_e32 v134, 0xbfb8aa3b, v134\n" \
    "  v_mul_f32_e32 v135, 0xbfb8aa3b, v135\n" \
    "  v_exp_f32_e32 v136, v132\n" \
    "  v_exp_f32_e32 v137, v133\n" \
    "  v_exp_f32_e32 v138, v134\n" \
    "  v_exp_f32_e32 v139, v135\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v136\n" \
    "  v_mov_b32_e32 v32, v137\n" \
    "  v_mov_b32_e32 v64, v138\n" \
    "  v_mov_b32_e32 v96, v139\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_add_f32_e32 v140, s41, v128\n" \
    "  v_add_f32_e32 v141, s41, v129\n" \
    "  v_add_f32_e32 v142, s41, v130\n" \
    "  v_add_f32_e32 v143, s41, v131\n" \
    "  v_maximum3_f32 v132, v140, -v140, -v140\n" \
    "  v_maximum3_f32 v133, v141, -v141, -v141\n" \
    "  v_maximum3_f32 v134, v142, -v142, -v142\n" \
    "  v_maximum3_f32 v135, v143, -v143, -v143\n" \
    "  s_set_gpr_idx_on s40, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s59, 15\n" \
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
    "  v_fmac_f32_e64 v129, v32, s73\n" \
    "  v_fmac_f32_e64 v130, v64, s73\n" \
    "  v_fmac_f32_e64 v131, v96, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_fmac_f32_e64 v128, v0, s75\n" \
    "  v_fmac_f32_e64 v129, v32, s75\n" \
    "  v_fmac_f32_e64 v130, v64, s75\n" \
    "  v_fmac_f32_e64 v131, v96, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovds_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v128, v0, s77\n" \
    "  v_fmac_f32_e64 v129, v32, s77\n" \
    "  v_fmac_f32_e64 v130, v64, s77\n" \
    "  v_fmac_f32_e64 v131, v96, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_fmac_f32_e64 v128, v0, s79\n" \
    "  v_fmac_f32_e64 v129, v32, s79\n" \
    "  v_fmac_f32_e64 v130, v64, s79\n" \
    "  v_fmac_f32_e64 v131, v96, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovds_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Los_A%=\n" \
    "Lovds_A%=:\n" \
    "  s_lshr_b32 s88, s40, 15\n" \
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
    "  v_mul_f32_e64 v132, v0, s73\n" \
    "  v_mul_f32_e64 v133, v32, s73\n" \
    "  v_mul_f32_e64 v134, v64, s73\n" \
    "  v_mul_f32_e64 v135, v96, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v136, v0, s75\n" \
    "  v_mul_f32_e64 v137, v32, s75\n" \
    "  v_mul_f32_e64 v138, v64, s75\n" \
    "  v_mul_f32_e64 v139, v96, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  v_mul_f32_e32 v130, v130, v134\n" \
    "  v_mul_f32_e32 v131, v131, v135\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdp_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s77\n" \
    "  v_mul_f32_e64 v133, v32, s77\n" \
    "  v_mul_f32_e64 v134, v64, s77\n" \
    "  v_mul_f32_e64 v135, v96, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v136, v0, s79\n" \
    "  v_mul_f32_e64 v137, v32, s79\n" \
    "  v_mul_f32_e64 v138, v64, s79\n" \
    "  v_mul_f32_e64 v139, v96, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  v_mul_f32_e32 v130, v130, v134\n" \
    "  v_mul_f32_e32 v131, v131, v135\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdp_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lop_A%=\n" \
    "Lovdp_A%=:\n" \
    "  s_lshr_b32 s88, s40, 15\n" \
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
    "  v_mul_f32_e64 v132, v0, s73\n" \
    "  v_mul_f32_e64 v133, v32, s73\n" \
    "  v_mul_f32_e64 v134, v64, s73\n" \
    "  v_mul_f32_e64 v135, v96, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v136, v0, s75\n" \
    "  v_mul_f32_e64 v137, v32, s75\n" \
    "  v_mul_f32_e64 v138, v64, s75\n" \
    "  v_mul_f32_e64 v139, v96, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v132, v136\n" \
    "  v_maximum3_f32 v129, v129, v133, v137\n" \
    "  v_maximum3_f32 v130, v130, v134, v138\n" \
    "  v_maximum3_f32 v131, v131, v135, v139\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdm_A%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s77\n" \
    "  v_mul_f32_e64 v133, v32, s77\n" \
    "  v_mul_f32_e64 v134, v64, s77\n" \
    "  v_mul_f32_e64 v135, v96, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v136, v0, s79\n" \
    "  v_mul_f32_e64 v137, v32, s79\n" \
    "  v_mul_f32_e64 v138, v64, s79\n" \
    "  v_mul_f32_e64 v139, v96, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v132, v136\n" \
    "  v_maximum3_f32 v129, v129, v133, v137\n" \
    "  v_maximum3_f32 v130, v130, v134, v138\n" \
    "  v_maximum3_f32 v131, v131, v135, v139\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdm_A%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lom_A%=\n" \
    "Lovdm_A%=:\n" \
    "  s_lshr_b32 s88, s40, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "Ltab_B%=:\n" \
    "  v_mov_b32_e32 v140, s57\n" \
    "  v_mov_b32_e32 v141, s57\n" \
    "  v_mov_b32_e32 v142, s57\n" \
    "  v_mov_b32_e32 v143, s57\n" \
    "  v_fmac_f32_e64 v140, s58, v128\n" \
    "  v_fmac_f32_e64 v141, s58, v129\n" \
    "  v_fmac_f32_e64 v142, s58, v130\n" \
    "  v_fmac_f32_e64 v143, s58, v131\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v140\n" \
    "  v_mov_b32_e32 v32, v141\n" \
    "  v_mov_b32_e32 v64, v142\n" \
    "  v_mov_b32_e32 v96, v143\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_mov_b32_e32 v140, s57\n" \
    "  v_mov_b32_e32 v141, s57\n" \
    "  v_mov_b32_e32 v142, s57\n" \
    "  v_mov_b32_e32 v143, s57\n" \
    "  v_fmac_f32_e64 v140, s58, v128\n" \
    "  v_fmac_f32_e64 v141, s58, v129\n" \
    "  v_fmac_f32_e64 v142, s58, v130\n" \
    "  v_fmac_f32_e64 v143, s58, v131\n" \
    "  v_mul_f32_e32 v132, 0x4038aa3b, v140\n" \
    "  v_mul_f32_e32 v133, 0x4038aa3b, v141\n" \
    "  v_mul_f32_e32 v134, 0x4038aa3b, v142\n" \
    "  v_mul_f32_e32 v135, 0x4038aa3b, v143\n" \
    "  v_exp_f32_e32 v132, v132\n" \
    "  v_exp_f32_e32 v133, v133\n" \
    "  v_exp_f32_e32 v134, v134\n" \
    "  v_exp_f32_e32 v135, v135\n" \
    "  v_add_f32_e32 v136, 1.0, v132\n" \
    "  v_add_f32_e32 v137, 1.0, v133\n" \
    "  v_add_f32_e32 v138, 1.0, v134\n" \
    "  v_add_f32_e32 v139, 1.0, v135\n" \
    "  v_rcp_f32_e32 v136, v136\n" \
    "  v_rcp_f32_e32 v137, v137\n" \
    "  v_rcp_f32_e32 v138, v138\n" \
    "  v_rcp_f32_e32 v139, v139\n" \
    "  v_fma_f32 v132, v136, -2.0, 1.0\n" \
    "  v_fma_f32 v133, v137, -2.0, 1.0\n" \
    "  v_fma_f32 v134, v138, -2.0, 1.0\n" \
    "  v_fma_f32 v135, v139, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_mov_b32_e32 v140, s57\n" \
    "  v_mov_b32_e32 v141, s57\n" \
    "  v_mov_b32_e32 v142, s57\n" \
    "  v_mov_b32_e32 v143, s57\n" \
    "  v_fmac_f32_e64 v140, s58, v128\n" \
    "  v_fmac_f32_e64 v141, s58, v129\n" \
    "  v_fmac_f32_e64 v142, s58, v130\n" \
    "  v_fmac_f32_e64 v143, s58, v131\n" \
    "  v_mul_f32_e32 v132, 0xbfb8aa3b, v140\n" \
    "  v_mul_f32_e32 v133, 0xbfb8aa3b, v141\n" \
    "  v_mul_f32_e32 v134, 0xbfb8aa3b, v142\n" \
    "  v_mul_f32_e32 v135, 0xbfb8aa3b, v143\n" \
    "  v_exp_f32_e32 v132, v132\n" \
    "  v_exp_f32_e32 v133, v133\n" \
    "  v_exp_f32_e32 v134, v134\n" \
    "  v_exp_f32_e32 v135, v135\n" \
    "  v_add_f32_e32 v136, 1.0, v132\n" \
    "  v_add_f32_e32 v137, 1.0, v133\n" \
    "  v_add_f32_e32 v138, 1.0, v134\n" \
    "  v_add_f32_e32 v139, 1.0, v135\n" \
    "  v_rcp_f32_e32 v132, v136\n" \
    "  v_rcp_f32_e32 v133, v137\n" \
    "  v_rcp_f32_e32 v134, v138\n" \
    "  v_rcp_f32_e32 v135, v139\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_mov_b32_e32 v140, s57\n" \
    "  v_mov_b32_e32 v141, s57\n" \
    "  v_mov_b32_e32 v142, s57\n" \
    "  v_mov_b32_e32 v143, s57\n" \
    "  v_fmac_f32_e64 v140, s58, v128\n" \
    "  v_fmac_f32_e64 v141, s58, v129\n" \
    "  v_fmac_f32_e64 v142, s58, v130\n" \
    "  v_fmac_f32_e64 v143, s58, v131\n" \
    "  v_maximum3_f32 v132, v140, 0, 0\n" \
    "  v_maximum3_f32 v133, v141, 0, 0\n" \
    "  v_maximum3_f32 v134, v142, 0, 0\n" \
    "  v_maximum3_f32 v135, v143, 0, 0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_mov_b32_e32 v140, s57\n" \
    "  v_mov_b32_e32 v141, s57\n" \
    "  v_mov_b32_e32 v142, s57\n" \
    "  v_mov_b32_e32 v143, s57\n" \
    "  v_fmac_f32_e64 v140, s58, v128\n" \
    "  v_fmac_f32_e64 v141, s58, v129\n" \
    "  v_fmac_f32_e64 v142, s58, v130\n" \
    "  v_fmac_f32_e64 v143, s58, v131\n" \
    "  v_mul_f32_e32 v136, 0x3ea2f983, v140\n" \
    "  v_mul_f32_e32 v137, 0x3ea2f983, v141\n" \
    "  v_mul_f32_e32 v138, 0x3ea2f983, v142\n" \
    "  v_mul_f32_e32 v139, 0x3ea2f983, v143\n" \
    "  v_rndne_f32_e32 v136, v136\n" \
    "  v_rndne_f32_e32 v137, v137\n" \
    "  v_rndne_f32_e32 v138, v138\n" \
    "  v_rndne_f32_e32 v139, v139\n" \
    "  v_fmamk_f32 v128, v136, 0xc0490fdb, v140\n" \
    "  v_fmamk_f32 v129, v137, 0xc0490fdb, v141\n" \
    "  v_fmamk_f32 v130, v138, 0xc0490fdb, v142\n" \
    "  v_fmamk_f32 v131, v139, 0xc0490fdb, v143\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v136\n" \
    "  v_fmac_f32_e32 v129, 0x33bbbd2e, v137\n" \
    "  v_fmac_f32_e32 v130, 0x33bbbd2e, v138\n" \
    "  v_fmac_f32_e32 v131, 0x33bbbd2e, v139\n" \
    "  v_cvt_i32_f32_e32 v136, v136\n" \
    "  v_cvt_i32_f32_e32 v137, v137\n" \
    "  v_cvt_i32_f32_e32 v138, v138\n" \
    "  v_cvt_i32_f32_e32 v139, v139\n" \
    "  v_mul_f32_e32 v140, v128, v128\n" \
    "  v_mul_f32_e32 v141, v129, v129\n" \
    "  v_mul_f32_e32 v142, v130, v130\n" \
    "  v_mul_f32_e32 v143, v131, v131\n" \
    "  v_fmaak_f32 v145, v140, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v146, v141, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v147, v142, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v148, v143, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v145, v140, v145, 0x3638ef1d\n" \
    "  v_fmaak_f32 v146, v141, v146, 0x3638ef1d\n" \
    "  v_fmaak_f32 v147, v142, v147, 0x3638ef1d\n" \
    "  v_fmaak_f32 v148, v143, v148, 0x3638ef1d\n" \
    "  v_fmaak_f32 v145, v140, v145, 0xb9500d01\n" \
    "  v_fmaak_f32 v146, v141, v146, 0xb9500d01\n" \
    "  v_fmaak_f32 v147, v142, v147, 0xb9500d01\n" \
    "  v_fmaak_f32 v148, v143, v148, 0xb9500d01\n" \
    "  v_fmaak_f32 v145, v140, v145, 0x3c088889\n" \
    "  v_fmaak_f32 v146, v141, v146, 0x3c088889\n" \
    "  v_fmaak_f32 v147, v142, v147, 0x3c088889\n" \
    "  v_fmaak_f32 v148, v143, v148, 0x3c088889\n" \
    "  v_fmaak_f32 v145, v140, v145, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v146, v141, v146, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v147, v142, v147, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v148, v143, v148, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v132, v128, v140\n" \
    "  v_mul_f32_e32 v133, v129, v141\n" \
    "  v_mul_f32_e32 v134, v130, v142\n" \
    "  v_mul_f32_e32 v135, v131, v143\n" \
    "  v_fmac_f32_e32 v128, v132, v145\n" \
    "  v_fmac_f32_e32 v129, v133, v146\n" \
    "  v_fmac_f32_e32 v130, v134, v147\n" \
    "  v_fmac_f32_e32 v131, v135, v148\n" \
    "  v_lshl_add_u32 v132, v136, 31, v128\n" \
    "  v_lshl_add_u32 v133, v137, 31, v129\n" \
    "  v_lshl_add_u32 v134, v138, 31, v130\n" \
    "  v_lshl_add_u32 v135, v139, 31, v131\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_mov_b32_e32 v140, s57\n" \
    "  v_mov_b32_e32 v141, s57\n" \
    "  v_mov_b32_e32 v142, s57\n" \
    "  v_mov_b32_e32 v143, s57\n" \
    "  v_fmac_f32_e64 v140, s58, v128\n" \
    "  v_fmac_f32_e64 v141, s58, v129\n" \
    "  v_fmac_f32_e64 v142, s58, v130\n" \
    "  v_fmac_f32_e64 v143, s58, v131\n" \
    "  v_mul_f32_e32 v132, v140, v140\n" \
    "  v_mul_f32_e32 v133, v141, v141\n" \
    "  v_mul_f32_e32 v134, v142, v142\n" \
    "  v_mul_f32_e32 v135, v143, v143\n" \
    "  v_mul_f32_e32 v132, 0xbfb8aa3b, v132\n" \
    "  v_mul_f32_e32 v133, 0xbfb8aa3b, v133\n" \
    "  v_mul_f32_e32 v134, 0xbfb8aa3b, v134\n" \
    "  v_mul_f32_e32 v135, 0xbfb8aa3b, v135\n" \
    "  v_exp_f32_e32 v136, v132\n" \
    "  v_exp_f32_e32 v137, v133\n" \
    "  v_exp_f32_e32 v138, v134\n" \
    "  v_exp_f32_e32 v139, v135\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v136\n" \
    "  v_mov_b32_e32 v32, v137\n" \
    "  v_mov_b32_e32 v64, v138\n" \
    "  v_mov_b32_e32 v96, v139\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_mov_b32_e32 v140, s57\n" \
    "  v_mov_b32_e32 v141, s57\n" \
    "  v_mov_b32_e32 v142, s57\n" \
    "  v_mov_b32_e32 v143, s57\n" \
    "  v_fmac_f32_e64 v140, s58, v128\n" \
    "  v_fmac_f32_e64 v141, s58, v129\n" \
    "  v_fmac_f32_e64 v142, s58, v130\n" \
    "  v_fmac_f32_e64 v143, s58, v131\n" \
    "  v_maximum3_f32 v132, v140, -v140, -v140\n" \
    "  v_maximum3_f32 v133, v141, -v141, -v141\n" \
    "  v_maximum3_f32 v134, v142, -v142, -v142\n" \
    "  v_maximum3_f32 v135, v143, -v143, -v143\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_branch Ldone%=\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  v_mov_b32_e32 v128, 0\n" \
    "  v_mov_b32_e32 v129, 0\n" \
    "  v_mov_b32_e32 v130, 0\n" \
    "  v_mov_b32_e32 v131, 0\n" \
    "  s_lshr_b32 s88, s56, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v32, s61\n" \
    "  v_mul_f32_e64 v130, v64, s61\n" \
    "  v_mul_f32_e64 v131, v96, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  v_fmac_f32_e64 v129, v32, s63\n" \
    "  v_fmac_f32_e64 v130, v64, s63\n" \
    "  v_fmac_f32_e64 v131, v96, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v32, s61\n" \
    "  v_mul_f32_e64 v130, v64, s61\n" \
    "  v_mul_f32_e64 v131, v96, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  v_fmac_f32_e64 v129, v32, s63\n" \
    "  v_fmac_f32_e64 v130, v64, s63\n" \
    "  v_fmac_f32_e64 v131, v96, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v128, v0, s65\n" \
    "  v_fmac_f32_e64 v129, v32, s65\n" \
    "  v_fmac_f32_e64 v130, v64, s65\n" \
    "  v_fmac_f32_e64 v131, v96, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v128, v0, s67\n" \
    "  v_fmac_f32_e64 v129, v32, s67\n" \
    "  v_fmac_f32_e64 v130, v64, s67\n" \
    "  v_fmac_f32_e64 v131, v96, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v32, s61\n" \
    "  v_mul_f32_e64 v130, v64, s61\n" \
    "  v_mul_f32_e64 v131, v96, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  v_fmac_f32_e64 v129, v32, s63\n" \
    "  v_fmac_f32_e64 v130, v64, s63\n" \
    "  v_fmac_f32_e64 v131, v96, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v128, v0, s65\n" \
    "  v_fmac_f32_e64 v129, v32, s65\n" \
    "  v_fmac_f32_e64 v130, v64, s65\n" \
    "  v_fmac_f32_e64 v131, v96, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v128, v0, s67\n" \
    "  v_fmac_f32_e64 v129, v32, s67\n" \
    "  v_fmac_f32_e64 v130, v64, s67\n" \
    "  v_fmac_f32_e64 v131, v96, s67\n" \
    "  s_set_gpr_idx_idx s68\n" \
    "  v_fmac_f32_e64 v128, v0, s69\n" \
    "  v_fmac_f32_e64 v129, v32, s69\n" \
    "  v_fmac_f32_e64 v130, v64, s69\n" \
    "  v_fmac_f32_e64 v131, v96, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_fmac_f32_e64 v128, v0, s71\n" \
    "  v_fmac_f32_e64 v129, v32, s71\n" \
    "  v_fmac_f32_e64 v130, v64, s71\n" \
    "  v_fmac_f32_e64 v131, v96, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_lshr_b32 s88, s56, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v32, s61\n" \
    "  v_mul_f32_e64 v130, v64, s61\n" \
    "  v_mul_f32_e64 v131, v96, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_fmac_f32_e64 v128, v0, s63\n" \
    "  v_fmac_f32_e64 v129, v32, s63\n" \
    "  v_fmac_f32_e64 v130, v64, s63\n" \
    "  v_fmac_f32_e64 v131, v96, s63\n" \
    "  s_set_gpr_idx_idx s64\n" \
    "  v_fmac_f32_e64 v128, v0, s65\n" \
    "  v_fmac_f32_e64 v129, v32, s65\n" \
    "  v_fmac_f32_e64 v130, v64, s65\n" \
    "  v_fmac_f32_e64 v131, v96, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_fmac_f32_e64 v128, v0, s67\n" \
    "  v_fmac_f32_e64 v129, v32, s67\n" \
    "  v_fmac_f32_e64 v130, v64, s67\n" \
    "  v_fmac_f32_e64 v131, v96, s67\n" \
    "  s_set_gpr_idx_idx s68\n" \
    "  v_fmac_f32_e64 v128, v0, s69\n" \
    "  v_fmac_f32_e64 v129, v32, s69\n" \
    "  v_fmac_f32_e64 v130, v64, s69\n" \
    "  v_fmac_f32_e64 v131, v96, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_fmac_f32_e64 v128, v0, s71\n" \
    "  v_fmac_f32_e64 v129, v32, s71\n" \
    "  v_fmac_f32_e64 v130, v64, s71\n" \
    "  v_fmac_f32_e64 v131, v96, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_branch Lovs_B%=\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v32, s61\n" \
    "  v_mul_f32_e64 v130, v64, s61\n" \
    "  v_mul_f32_e64 v131, v96, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v136, v0, s63\n" \
    "  v_mul_f32_e64 v137, v32, s63\n" \
    "  v_mul_f32_e64 v138, v64, s63\n" \
    "  v_mul_f32_e64 v139, v96, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_lshr_b32 s88, s56, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v32, s61\n" \
    "  v_mul_f32_e64 v130, v64, s61\n" \
    "  v_mul_f32_e64 v131, v96, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v136, v0, s63\n" \
    "  v_mul_f32_e64 v137, v32, s63\n" \
    "  v_mul_f32_e64 v138, v64, s63\n" \
    "  v_mul_f32_e64 v139, v96, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s65\n" \
    "  v_mul_f32_e64 v133, v32, s65\n" \
    "  v_mul_f32_e64 v134, v64, s65\n" \
    "  v_mul_f32_e64 v135, v96, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v136, v0, s67\n" \
    "  v_mul_f32_e64 v137, v32, s67\n" \
    "  v_mul_f32_e64 v138, v64, s67\n" \
    "  v_mul_f32_e64 v139, v96, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  v_mul_f32_e32 v130, v130, v134\n" \
    "  v_mul_f32_e32 v131, v131, v135\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_lshr_b32 s88, s56, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v32, s61\n" \
    "  v_mul_f32_e64 v130, v64, s61\n" \
    "  v_mul_f32_e64 v131, v96, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v136, v0, s63\n" \
    "  v_mul_f32_e64 v137, v32, s63\n" \
    "  v_mul_f32_e64 v138, v64, s63\n" \
    "  v_mul_f32_e64 v139, v96, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s65\n" \
    "  v_mul_f32_e64 v133, v32, s65\n" \
    "  v_mul_f32_e64 v134, v64, s65\n" \
    "  v_mul_f32_e64 v135, v96, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v136, v0, s67\n" \
    "  v_mul_f32_e64 v137, v32, s67\n" \
    "  v_mul_f32_e64 v138, v64, s67\n" \
    "  v_mul_f32_e64 v139, v96, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  v_mul_f32_e32 v130, v130, v134\n" \
    "  v_mul_f32_e32 v131, v131, v135\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s69\n" \
    "  v_mul_f32_e64 v133, v32, s69\n" \
    "  v_mul_f32_e64 v134, v64, s69\n" \
    "  v_mul_f32_e64 v135, v96, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v136, v0, s71\n" \
    "  v_mul_f32_e64 v137, v32, s71\n" \
    "  v_mul_f32_e64 v138, v64, s71\n" \
    "  v_mul_f32_e64 v139, v96, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  v_mul_f32_e32 v130, v130, v134\n" \
    "  v_mul_f32_e32 v131, v131, v135\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_lshr_b32 s88, s56, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v128, v0, s61\n" \
    "  v_mul_f32_e64 v129, v32, s61\n" \
    "  v_mul_f32_e64 v130, v64, s61\n" \
    "  v_mul_f32_e64 v131, v96, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v136, v0, s63\n" \
    "  v_mul_f32_e64 v137, v32, s63\n" \
    "  v_mul_f32_e64 v138, v64, s63\n" \
    "  v_mul_f32_e64 v139, v96, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s65\n" \
    "  v_mul_f32_e64 v133, v32, s65\n" \
    "  v_mul_f32_e64 v134, v64, s65\n" \
    "  v_mul_f32_e64 v135, v96, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v136, v0, s67\n" \
    "  v_mul_f32_e64 v137, v32, s67\n" \
    "  v_mul_f32_e64 v138, v64, s67\n" \
    "  v_mul_f32_e64 v139, v96, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  v_mul_f32_e32 v130, v130, v134\n" \
    "  v_mul_f32_e32 v131, v131, v135\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s69\n" \
    "  v_mul_f32_e64 v133, v32, s69\n" \
    "  v_mul_f32_e64 v134, v64, s69\n" \
    "  v_mul_f32_e64 v135, v96, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v136, v0, s71\n" \
    "  v_mul_f32_e64 v137, v32, s71\n" \
    "  v_mul_f32_e64 v138, v64, s71\n" \
    "  v_mul_f32_e64 v139, v96, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  v_mul_f32_e32 v130, v130, v134\n" \
    "  v_mul_f32_e32 v131, v131, v135\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_branch Lovp_B%=\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s61\n" \
    "  v_mul_f32_e64 v133, v32, s61\n" \
    "  v_mul_f32_e64 v134, v64, s61\n" \
    "  v_mul_f32_e64 v135, v96, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v136, v0, s63\n" \
    "  v_mul_f32_e64 v137, v32, s63\n" \
    "  v_mul_f32_e64 v138, v64, s63\n" \
    "  v_mul_f32_e64 v139, v96, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v132, v136, v136\n" \
    "  v_maximum3_f32 v129, v133, v137, v137\n" \
    "  v_maximum3_f32 v130, v134, v138, v138\n" \
    "  v_maximum3_f32 v131, v135, v139, v139\n" \
    "  s_lshr_b32 s88, s56, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s61\n" \
    "  v_mul_f32_e64 v133, v32, s61\n" \
    "  v_mul_f32_e64 v134, v64, s61\n" \
    "  v_mul_f32_e64 v135, v96, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v136, v0, s63\n" \
    "  v_mul_f32_e64 v137, v32, s63\n" \
    "  v_mul_f32_e64 v138, v64, s63\n" \
    "  v_mul_f32_e64 v139, v96, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v132, v136, v136\n" \
    "  v_maximum3_f32 v129, v133, v137, v137\n" \
    "  v_maximum3_f32 v130, v134, v138, v138\n" \
    "  v_maximum3_f32 v131, v135, v139, v139\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s65\n" \
    "  v_mul_f32_e64 v133, v32, s65\n" \
    "  v_mul_f32_e64 v134, v64, s65\n" \
    "  v_mul_f32_e64 v135, v96, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v136, v0, s67\n" \
    "  v_mul_f32_e64 v137, v32, s67\n" \
    "  v_mul_f32_e64 v138, v64, s67\n" \
    "  v_mul_f32_e64 v139, v96, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v132, v136\n" \
    "  v_maximum3_f32 v129, v129, v133, v137\n" \
    "  v_maximum3_f32 v130, v130, v134, v138\n" \
    "  v_maximum3_f32 v131, v131, v135, v139\n" \
    "  s_lshr_b32 s88, s56, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s61\n" \
    "  v_mul_f32_e64 v133, v32, s61\n" \
    "  v_mul_f32_e64 v134, v64, s61\n" \
    "  v_mul_f32_e64 v135, v96, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v136, v0, s63\n" \
    "  v_mul_f32_e64 v137, v32, s63\n" \
    "  v_mul_f32_e64 v138, v64, s63\n" \
    "  v_mul_f32_e64 v139, v96, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v132, v136, v136\n" \
    "  v_maximum3_f32 v129, v133, v137, v137\n" \
    "  v_maximum3_f32 v130, v134, v138, v138\n" \
    "  v_maximum3_f32 v131, v135, v139, v139\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s65\n" \
    "  v_mul_f32_e64 v133, v32, s65\n" \
    "  v_mul_f32_e64 v134, v64, s65\n" \
    "  v_mul_f32_e64 v135, v96, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v136, v0, s67\n" \
    "  v_mul_f32_e64 v137, v32, s67\n" \
    "  v_mul_f32_e64 v138, v64, s67\n" \
    "  v_mul_f32_e64 v139, v96, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v132, v136\n" \
    "  v_maximum3_f32 v129, v129, v133, v137\n" \
    "  v_maximum3_f32 v130, v130, v134, v138\n" \
    "  v_maximum3_f32 v131, v131, v135, v139\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s69\n" \
    "  v_mul_f32_e64 v133, v32, s69\n" \
    "  v_mul_f32_e64 v134, v64, s69\n" \
    "  v_mul_f32_e64 v135, v96, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v136, v0, s71\n" \
    "  v_mul_f32_e64 v137, v32, s71\n" \
    "  v_mul_f32_e64 v138, v64, s71\n" \
    "  v_mul_f32_e64 v139, v96, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v132, v136\n" \
    "  v_maximum3_f32 v129, v129, v133, v137\n" \
    "  v_maximum3_f32 v130, v130, v134, v138\n" \
    "  v_maximum3_f32 v131, v131, v135, v139\n" \
    "  s_lshr_b32 s88, s56, 15\n" \
    "  s_add_u32 s88, s88, s94\n" \
    "  s_addc_u32 s89, s95, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  s_add_u32 s86, s86, 64\n" \
    "  s_load_dwordx16 s[40:55], s[80:81], s86\n" \
    "  s_load_dwordx8 s[72:79], s[84:85], 0x0\n" \
    "  s_set_gpr_idx_on s60, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s61\n" \
    "  v_mul_f32_e64 v133, v32, s61\n" \
    "  v_mul_f32_e64 v134, v64, s61\n" \
    "  v_mul_f32_e64 v135, v96, s61\n" \
    "  s_set_gpr_idx_idx s62\n" \
    "  v_mul_f32_e64 v136, v0, s63\n" \
    "  v_mul_f32_e64 v137, v32, s63\n" \
    "  v_mul_f32_e64 v138, v64, s63\n" \
    "  v_mul_f32_e64 v139, v96, s63\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v132, v136, v136\n" \
    "  v_maximum3_f32 v129, v133, v137, v137\n" \
    "  v_maximum3_f32 v130, v134, v138, v138\n" \
    "  v_maximum3_f32 v131, v135, v139, v139\n" \
    "  s_set_gpr_idx_on s64, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s65\n" \
    "  v_mul_f32_e64 v133, v32, s65\n" \
    "  v_mul_f32_e64 v134, v64, s65\n" \
    "  v_mul_f32_e64 v135, v96, s65\n" \
    "  s_set_gpr_idx_idx s66\n" \
    "  v_mul_f32_e64 v136, v0, s67\n" \
    "  v_mul_f32_e64 v137, v32, s67\n" \
    "  v_mul_f32_e64 v138, v64, s67\n" \
    "  v_mul_f32_e64 v139, v96, s67\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v132, v136\n" \
    "  v_maximum3_f32 v129, v129, v133, v137\n" \
    "  v_maximum3_f32 v130, v130, v134, v138\n" \
    "  v_maximum3_f32 v131, v131, v135, v139\n" \
    "  s_set_gpr_idx_on s68, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s69\n" \
    "  v_mul_f32_e64 v133, v32, s69\n" \
    "  v_mul_f32_e64 v134, v64, s69\n" \
    "  v_mul_f32_e64 v135, v96, s69\n" \
    "  s_set_gpr_idx_idx s70\n" \
    "  v_mul_f32_e64 v136, v0, s71\n" \
    "  v_mul_f32_e64 v137, v32, s71\n" \
    "  v_mul_f32_e64 v138, v64, s71\n" \
    "  v_mul_f32_e64 v139, v96, s71\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v132, v136\n" \
    "  v_maximum3_f32 v129, v129, v133, v137\n" \
    "  v_maximum3_f32 v130, v130, v134, v138\n" \
    "  v_maximum3_f32 v131, v131, v135, v139\n" \
    "  s_branch Lovm_B%=\n" \
    "  .p2align 9\n" \
    "  v_add_f32_e32 v140, s57, v128\n" \
    "  v_add_f32_e32 v141, s57, v129\n" \
    "  v_add_f32_e32 v142, s57, v130\n" \
    "  v_add_f32_e32 v143, s57, v131\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v140\n" \
    "  v_mov_b32_e32 v32, v141\n" \
    "  v_mov_b32_e32 v64, v142\n" \
    "  v_mov_b32_e32 v96, v143\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_add_f32_e32 v140, s57, v128\n" \
    "  v_add_f32_e32 v141, s57, v129\n" \
    "  v_add_f32_e32 v142, s57, v130\n" \
    "  v_add_f32_e32 v143, s57, v131\n" \
    "  v_mul_f32_e32 v132, 0x4038aa3b, v140\n" \
    "  v_mul_f32_e32 v133, 0x4038aa3b, v141\n" \
    "  v_mul_f32_e32 v134, 0x4038aa3b, v142\n" \
    "  v_mul_f32_e32 v135, 0x4038aa3b, v143\n" \
    "  v_exp_f32_e32 v132, v132\n" \
    "  v_exp_f32_e32 v133, v133\n" \
    "  v_exp_f32_e32 v134, v134\n" \
    "  v_exp_f32_e32 v135, v135\n" \
    "  v_add_f32_e32 v136, 1.0, v132\n" \
    "  v_add_f32_e32 v137, 1.0, v133\n" \
    "  v_add_f32_e32 v138, 1.0, v134\n" \
    "  v_add_f32_e32 v139, 1.0, v135\n" \
    "  v_rcp_f32_e32 v136, v136\n" \
    "  v_rcp_f32_e32 v137, v137\n" \
    "  v_rcp_f32_e32 v138, v138\n" \
    "  v_rcp_f32_e32 v139, v139\n" \
    "  v_fma_f32 v132, v136, -2.0, 1.0\n" \
    "  v_fma_f32 v133, v137, -2.0, 1.0\n" \
    "  v_fma_f32 v134, v138, -2.0, 1.0\n" \
    "  v_fma_f32 v135, v139, -2.0, 1.0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_add_f32_e32 v140, s57, v128\n" \
    "  v_add_f32_e32 v141, s57, v129\n" \
    "  v_add_f32_e32 v142, s57, v130\n" \
    "  v_add_f32_e32 v143, s57, v131\n" \
    "  v_mul_f32_e32 v132, 0xbfb8aa3b, v140\n" \
    "  v_mul_f32_e32 v133, 0xbfb8aa3b, v141\n" \
    "  v_mul_f32_e32 v134, 0xbfb8aa3b, v142\n" \
    "  v_mul_f32_e32 v135, 0xbfb8aa3b, v143\n" \
    "  v_exp_f32_e32 v132, v132\n" \
    "  v_exp_f32_e32 v133, v133\n" \
    "  v_exp_f32_e32 v134, v134\n" \
    "  v_exp_f32_e32 v135, v135\n" \
    "  v_add_f32_e32 v136, 1.0, v132\n" \
    "  v_add_f32_e32 v137, 1.0, v133\n" \
    "  v_add_f32_e32 v138, 1.0, v134\n" \
    "  v_add_f32_e32 v139, 1.0, v135\n" \
    "  v_rcp_f32_e32 v132, v136\n" \
    "  v_rcp_f32_e32 v133, v137\n" \
    "  v_rcp_f32_e32 v134, v138\n" \
    "  v_rcp_f32_e32 v135, v139\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_add_f32_e32 v140, s57, v128\n" \
    "  v_add_f32_e32 v141, s57, v129\n" \
    "  v_add_f32_e32 v142, s57, v130\n" \
    "  v_add_f32_e32 v143, s57, v131\n" \
    "  v_maximum3_f32 v132, v140, 0, 0\n" \
    "  v_maximum3_f32 v133, v141, 0, 0\n" \
    "  v_maximum3_f32 v134, v142, 0, 0\n" \
    "  v_maximum3_f32 v135, v143, 0, 0\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_add_f32_e32 v140, s57, v128\n" \
    "  v_add_f32_e32 v141, s57, v129\n" \
    "  v_add_f32_e32 v142, s57, v130\n" \
    "  v_add_f32_e32 v143, s57, v131\n" \
    "  v_mul_f32_e32 v136, 0x3ea2f983, v140\n" \
    "  v_mul_f32_e32 v137, 0x3ea2f983, v141\n" \
    "  v_mul_f32_e32 v138, 0x3ea2f983, v142\n" \
    "  v_mul_f32_e32 v139, 0x3ea2f983, v143\n" \
    "  v_rndne_f32_e32 v136, v136\n" \
    "  v_rndne_f32_e32 v137, v137\n" \
    "  v_rndne_f32_e32 v138, v138\n" \
    "  v_rndne_f32_e32 v139, v139\n" \
    "  v_fmamk_f32 v128, v136, 0xc0490fdb, v140\n" \
    "  v_fmamk_f32 v129, v137, 0xc0490fdb, v141\n" \
    "  v_fmamk_f32 v130, v138, 0xc0490fdb, v142\n" \
    "  v_fmamk_f32 v131, v139, 0xc0490fdb, v143\n" \
    "  v_fmac_f32_e32 v128, 0x33bbbd2e, v136\n" \
    "  v_fmac_f32_e32 v129, 0x33bbbd2e, v137\n" \
    "  v_fmac_f32_e32 v130, 0x33bbbd2e, v138\n" \
    "  v_fmac_f32_e32 v131, 0x33bbbd2e, v139\n" \
    "  v_cvt_i32_f32_e32 v136, v136\n" \
    "  v_cvt_i32_f32_e32 v137, v137\n" \
    "  v_cvt_i32_f32_e32 v138, v138\n" \
    "  v_cvt_i32_f32_e32 v139, v139\n" \
    "  v_mul_f32_e32 v140, v128, v128\n" \
    "  v_mul_f32_e32 v141, v129, v129\n" \
    "  v_mul_f32_e32 v142, v130, v130\n" \
    "  v_mul_f32_e32 v143, v131, v131\n" \
    "  v_fmaak_f32 v145, v140, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v146, v141, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v147, v142, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v148, v143, v144, 0xb2d7322b\n" \
    "  v_fmaak_f32 v145, v140, v145, 0x3638ef1d\n" \
    "  v_fmaak_f32 v146, v141, v146, 0x3638ef1d\n" \
    "  v_fmaak_f32 v147, v142, v147, 0x3638ef1d\n" \
    "  v_fmaak_f32 v148, v143, v148, 0x3638ef1d\n" \
    "  v_fmaak_f32 v145, v140, v145, 0xb9500d01\n" \
    "  v_fmaak_f32 v146, v141, v146, 0xb9500d01\n" \
    "  v_fmaak_f32 v147, v142, v147, 0xb9500d01\n" \
    "  v_fmaak_f32 v148, v143, v148, 0xb9500d01\n" \
    "  v_fmaak_f32 v145, v140, v145, 0x3c088889\n" \
    "  v_fmaak_f32 v146, v141, v146, 0x3c088889\n" \
    "  v_fmaak_f32 v147, v142, v147, 0x3c088889\n" \
    "  v_fmaak_f32 v148, v143, v148, 0x3c088889\n" \
    "  v_fmaak_f32 v145, v140, v145, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v146, v141, v146, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v147, v142, v147, 0xbe2aaaab\n" \
    "  v_fmaak_f32 v148, v143, v148, 0xbe2aaaab\n" \
    "  v_mul_f32_e32 v132, v128, v140\n" \
    "  v_mul_f32_e32 v133, v129, v141\n" \
    "  v_mul_f32_e32 v134, v130, v142\n" \
    "  v_mul_f32_e32 v135, v131, v143\n" \
    "  v_fmac_f32_e32 v128, v132, v145\n" \
    "  v_fmac_f32_e32 v129, v133, v146\n" \
    "  v_fmac_f32_e32 v130, v134, v147\n" \
    "  v_fmac_f32_e32 v131, v135, v148\n" \
    "  v_lshl_add_u32 v132, v136, 31, v128\n" \
    "  v_lshl_add_u32 v133, v137, 31, v129\n" \
    "  v_lshl_add_u32 v134, v138, 31, v130\n" \
    "  v_lshl_add_u32 v135, v139, 31, v131\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_add_f32_e32 v140, s57, v128\n" \
    "  v_add_f32_e32 v141, s57, v129\n" \
    "  v_add_f32_e32 v142, s57, v130\n" \
    "  v_add_f32_e32 v143, s57, v131\n" \
    "  v_mul_f32_e32 v132, v140, v140\n" \
    "  v_mul_f32_e32 v133, v141, v141\n" \
    "  v_mul_f32_e32 v134, v142, v142\n" \
    "  v_mul_f32_e32 v135, v143, v143\n" \
    "  v_mul_f32_e32 v132, 0xbfb8aa3b, v132\n" \
    "  v_mul_f32_e32 v133, 0xbfb8aa3b, v133\n" \
    "  v_mul_f32_e32 v134, 0xbfb8aa3b, v134\n" \
    "  v_mul_f32_e32 v135, 0xbfb8aa3b, v135\n" \
    "  v_exp_f32_e32 v136, v132\n" \
    "  v_exp_f32_e32 v137, v133\n" \
    "  v_exp_f32_e32 v138, v134\n" \
    "  v_exp_f32_e32 v139, v135\n" \
    "  s_nop 1\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v136\n" \
    "  v_mov_b32_e32 v32, v137\n" \
    "  v_mov_b32_e32 v64, v138\n" \
    "  v_mov_b32_e32 v96, v139\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
    "  s_add_u32 s88, s88, s92\n" \
    "  s_addc_u32 s89, s93, 0\n" \
    "  s_setpc_b64 s[88:89]\n" \
    "  .p2align 9\n" \
    "  v_add_f32_e32 v140, s57, v128\n" \
    "  v_add_f32_e32 v141, s57, v129\n" \
    "  v_add_f32_e32 v142, s57, v130\n" \
    "  v_add_f32_e32 v143, s57, v131\n" \
    "  v_maximum3_f32 v132, v140, -v140, -v140\n" \
    "  v_maximum3_f32 v133, v141, -v141, -v141\n" \
    "  v_maximum3_f32 v134, v142, -v142, -v142\n" \
    "  v_maximum3_f32 v135, v143, -v143, -v143\n" \
    "  s_set_gpr_idx_on s56, gpr_idx(DST)\n" \
    "  v_mov_b32_e32 v0, v132\n" \
    "  v_mov_b32_e32 v32, v133\n" \
    "  v_mov_b32_e32 v64, v134\n" \
    "  v_mov_b32_e32 v96, v135\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_lshr_b32 s88, s43, 15\n" \
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
    "  v_fmac_f32_e64 v129, v32, s73\n" \
    "  v_fmac_f32_e64 v130, v64, s73\n" \
    "  v_fmac_f32_e64 v131, v96, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_fmac_f32_e64 v128, v0, s75\n" \
    "  v_fmac_f32_e64 v129, v32, s75\n" \
    "  v_fmac_f32_e64 v130, v64, s75\n" \
    "  v_fmac_f32_e64 v131, v96, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovds_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_fmac_f32_e64 v128, v0, s77\n" \
    "  v_fmac_f32_e64 v129, v32, s77\n" \
    "  v_fmac_f32_e64 v130, v64, s77\n" \
    "  v_fmac_f32_e64 v131, v96, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_fmac_f32_e64 v128, v0, s79\n" \
    "  v_fmac_f32_e64 v129, v32, s79\n" \
    "  v_fmac_f32_e64 v130, v64, s79\n" \
    "  v_fmac_f32_e64 v131, v96, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovds_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Los_B%=\n" \
    "Lovds_B%=:\n" \
    "  s_lshr_b32 s88, s56, 15\n" \
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
    "  v_mul_f32_e64 v132, v0, s73\n" \
    "  v_mul_f32_e64 v133, v32, s73\n" \
    "  v_mul_f32_e64 v134, v64, s73\n" \
    "  v_mul_f32_e64 v135, v96, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v136, v0, s75\n" \
    "  v_mul_f32_e64 v137, v32, s75\n" \
    "  v_mul_f32_e64 v138, v64, s75\n" \
    "  v_mul_f32_e64 v139, v96, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  v_mul_f32_e32 v130, v130, v134\n" \
    "  v_mul_f32_e32 v131, v131, v135\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdp_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s77\n" \
    "  v_mul_f32_e64 v133, v32, s77\n" \
    "  v_mul_f32_e64 v134, v64, s77\n" \
    "  v_mul_f32_e64 v135, v96, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v136, v0, s79\n" \
    "  v_mul_f32_e64 v137, v32, s79\n" \
    "  v_mul_f32_e64 v138, v64, s79\n" \
    "  v_mul_f32_e64 v139, v96, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_mul_f32_e32 v128, v128, v132\n" \
    "  v_mul_f32_e32 v129, v129, v133\n" \
    "  v_mul_f32_e32 v130, v130, v134\n" \
    "  v_mul_f32_e32 v131, v131, v135\n" \
    "  v_mul_f32_e32 v128, v128, v136\n" \
    "  v_mul_f32_e32 v129, v129, v137\n" \
    "  v_mul_f32_e32 v130, v130, v138\n" \
    "  v_mul_f32_e32 v131, v131, v139\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdp_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lop_B%=\n" \
    "Lovdp_B%=:\n" \
    "  s_lshr_b32 s88, s56, 15\n" \
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
    "  v_mul_f32_e64 v132, v0, s73\n" \
    "  v_mul_f32_e64 v133, v32, s73\n" \
    "  v_mul_f32_e64 v134, v64, s73\n" \
    "  v_mul_f32_e64 v135, v96, s73\n" \
    "  s_set_gpr_idx_idx s74\n" \
    "  v_mul_f32_e64 v136, v0, s75\n" \
    "  v_mul_f32_e64 v137, v32, s75\n" \
    "  v_mul_f32_e64 v138, v64, s75\n" \
    "  v_mul_f32_e64 v139, v96, s75\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v132, v136\n" \
    "  v_maximum3_f32 v129, v129, v133, v137\n" \
    "  v_maximum3_f32 v130, v130, v134, v138\n" \
    "  v_maximum3_f32 v131, v131, v135, v139\n" \
    "  s_cmp_eq_u32 s87, 1\n" \
    "  s_cbranch_scc1 Lovdm_B%=\n" \
    "  s_set_gpr_idx_on s76, gpr_idx(SRC0)\n" \
    "  v_mul_f32_e64 v132, v0, s77\n" \
    "  v_mul_f32_e64 v133, v32, s77\n" \
    "  v_mul_f32_e64 v134, v64, s77\n" \
    "  v_mul_f32_e64 v135, v96, s77\n" \
    "  s_set_gpr_idx_idx s78\n" \
    "  v_mul_f32_e64 v136, v0, s79\n" \
    "  v_mul_f32_e64 v137, v32, s79\n" \
    "  v_mul_f32_e64 v138, v64, s79\n" \
    "  v_mul_f32_e64 v139, v96, s79\n" \
    "  s_set_gpr_idx_off\n" \
    "  v_maximum3_f32 v128, v128, v132, v136\n" \
    "  v_maximum3_f32 v129, v129, v133, v137\n" \
    "  v_maximum3_f32 v130, v130, v134, v138\n" \
    "  v_maximum3_f32 v131, v131, v135, v139\n" \
    "  s_sub_u32 s87, s87, 2\n" \
    "  s_cmp_eq_u32 s87, 0\n" \
    "  s_cbranch_scc1 Lovdm_B%=\n" \
    "  s_add_u32 s82, s82, 32\n" \
    "  s_addc_u32 s83, s83, 0\n" \
    "  s_load_dwordx8 s[72:79], s[82:83], 0x0\n" \
    "  s_branch Lom_B%=\n" \
    "Lovdm_B%=:\n" \
    "  s_lshr_b32 s88, s56, 15\n" \
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
    "  v_add_u32_e32 v146, s41, v145\n" \
    "  v_add_u32_e32 v147, s41, v146\n" \
    "Lout%=:\n" \
    "  s_load_dwordx8 s[48:55], s[44:45], 0x0\n" \
    "  s_waitcnt lgkmcnt(0)\n" \
    "  s_set_gpr_idx_on s48, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v128, v0\n" \
    "  v_mov_b32_e32 v132, v32\n" \
    "  v_mov_b32_e32 v136, v64\n" \
    "  v_mov_b32_e32 v140, v96\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v128 offset:0\n" \
    "  ds_write_b32 v145, v132 offset:0\n" \
    "  ds_write_b32 v146, v136 offset:0\n" \
    "  ds_write_b32 v147, v140 offset:0\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s49, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v129, v0\n" \
    "  v_mov_b32_e32 v133, v32\n" \
    "  v_mov_b32_e32 v137, v64\n" \
    "  v_mov_b32_e32 v141, v96\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v129 offset:4\n" \
    "  ds_write_b32 v145, v133 offset:4\n" \
    "  ds_write_b32 v146, v137 offset:4\n" \
    "  ds_write_b32 v147, v141 offset:4\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s50, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v130, v0\n" \
    "  v_mov_b32_e32 v134, v32\n" \
    "  v_mov_b32_e32 v138, v64\n" \
    "  v_mov_b32_e32 v142, v96\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v130 offset:8\n" \
    "  ds_write_b32 v145, v134 offset:8\n" \
    "  ds_write_b32 v146, v138 offset:8\n" \
    "  ds_write_b32 v147, v142 offset:8\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s51, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v131, v0\n" \
    "  v_mov_b32_e32 v135, v32\n" \
    "  v_mov_b32_e32 v139, v64\n" \
    "  v_mov_b32_e32 v143, v96\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v131 offset:12\n" \
    "  ds_write_b32 v145, v135 offset:12\n" \
    "  ds_write_b32 v146, v139 offset:12\n" \
    "  ds_write_b32 v147, v143 offset:12\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s52, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v128, v0\n" \
    "  v_mov_b32_e32 v132, v32\n" \
    "  v_mov_b32_e32 v136, v64\n" \
    "  v_mov_b32_e32 v140, v96\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v128 offset:16\n" \
    "  ds_write_b32 v145, v132 offset:16\n" \
    "  ds_write_b32 v146, v136 offset:16\n" \
    "  ds_write_b32 v147, v140 offset:16\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s53, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v129, v0\n" \
    "  v_mov_b32_e32 v133, v32\n" \
    "  v_mov_b32_e32 v137, v64\n" \
    "  v_mov_b32_e32 v141, v96\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v129 offset:20\n" \
    "  ds_write_b32 v145, v133 offset:20\n" \
    "  ds_write_b32 v146, v137 offset:20\n" \
    "  ds_write_b32 v147, v141 offset:20\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s54, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v130, v0\n" \
    "  v_mov_b32_e32 v134, v32\n" \
    "  v_mov_b32_e32 v138, v64\n" \
    "  v_mov_b32_e32 v142, v96\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v130 offset:24\n" \
    "  ds_write_b32 v145, v134 offset:24\n" \
    "  ds_write_b32 v146, v138 offset:24\n" \
    "  ds_write_b32 v147, v142 offset:24\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  s_set_gpr_idx_on s55, gpr_idx(SRC0)\n" \
    "  v_mov_b32_e32 v131, v0\n" \
    "  v_mov_b32_e32 v135, v32\n" \
    "  v_mov_b32_e32 v139, v64\n" \
    "  v_mov_b32_e32 v143, v96\n" \
    "  s_set_gpr_idx_off\n" \
    "  ds_write_b32 v144, v131 offset:28\n" \
    "  ds_write_b32 v145, v135 offset:28\n" \
    "  ds_write_b32 v146, v139 offset:28\n" \
    "  ds_write_b32 v147, v143 offset:28\n" \
    "  s_add_u32 s40, s40, 1\n" \
    "  s_cmp_ge_u32 s40, %[no]\n" \
    "  s_cbranch_scc1 Lout_done%=\n" \
    "  v_add_u32_e32 v144, 32, v144\n" \
    "  v_add_u32_e32 v145, 32, v145\n" \
    "  v_add_u32_e32 v146, 32, v146\n" \
    "  v_add_u32_e32 v147, 32, v147\n" \
    "  s_add_u32 s44, s44, 32\n" \
    "  s_addc_u32 s45, s45, 0\n" \
    "  s_branch Lout%=\n" \
    "Lout_done%=:\n" \
    "  s_mov_b32 m0, s90\n"

#define NEAT_CLOB_S4_32 \
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
    "v144", "v145", "v146", "v147", "v148", "v149", "s40", "s41", "s42", "s43", "s44", "s45", \
    "s46", "s47", "s48", "s49", "s50", "s51", "s52", "s53", "s54", "s55", "s56", "s57", \
    "s58", "s59", "s60", "s61", "s62", "s63", "s64", "s65", "s66", "s67", "s68", "s69", \
    "s70", "s71", "s72", "s73", "s74", "s75", "s76", "s77", "s78", "s79", "s80", "s81", \
    "s82", "s83", "s84", "s85", "s86", "s87", "s88", "s89", "s90", "s91", "s92", "s93", \
    "s94", "s95", "vcc", "scc"

#define NEAT_SCRATCH_S4_32 128

