// forward.hip -- the calculation stage (Section 3.3) over population x inputs.
//
// Mapping "lane per sample": a 64-lane wave evaluates one genome on a run of
// sample tiles, one, two or four samples per lane.  The genome's program is
// uniform across the wave, so it is read with scalar loads and every branch
// on a node's activation or aggregation is a scalar branch.  A workgroup
// holds up to four waves working on the same genome, so they share the
// CU's scalar cache.
//
// Value stores (the value vector v of Section 3.3, slots and slot classes
// in program.h), one kernel per store:
//   R64    v0..v63, one sample per lane            (class R64)
//   R64X2  v0..v63 and v64..v127, two samples       (class R64)
//   R32X4  v0..v31 ... v96..v127, four samples      (class R64, N_max <= 30)
//   R128   v0..v127, one sample                     (class R128)
//   R224   v0..v223, one sample                     (class R224)
//   LDS    one LDS row of 64 lanes per slot         (class LDS; any class
//          when chosen explicitly)
// The register stores run one assembly block per tile (node_loop_asm.h):
// inputs from the LDS staging area into the registers, the DMA of the next
// tile's inputs, the node loop in GPR-index mode with the program's uniform
// slots, and the outputs into an LDS output area, which the C++ code then
// writes to HBM with coalesced 16-byte stores.  The LDS store runs the same
// node operations in C++.
//
// Work units.  A launch covers one or more populations ("items"); item j
// contributes P_j x chunks_j wave units (chunks_j from the item's wave
// target, or the launch's for several items of a kernel with more than one
// sample per lane), unit (i, c) being run c of the tiles of the i-th genome of
// the item's list for the kernel's class (the class list the transformation
// wrote, or all genomes).  Each wave of a workgroup takes its own unit, so
// consecutive waves share a genome when it has several chunks and take
// different genomes when it has one.  Units past the list's length exit at
// once.  Workgroups are remapped so consecutive ones share an XCD (workgroups
// are dealt to the 8 XCDs round robin).
//
// Inputs of the next tile are copied HBM -> LDS by the DMA path of
// global_load_lds (16-byte pieces when aligned) while the current tile
// computes; each lane then moves its own samples' inputs into v.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cstdio>
#include <cstdlib>

#include "act.h"
#include "launch.h"
#include "neat.h"
#include "node_loop_asm.h"
#include "node_loop_wide.h"
#include "program.h"

namespace neat {
namespace {

constexpr int WAVE = 64;

typedef float f32x32 __attribute__((ext_vector_type(32)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef int i32x16 __attribute__((ext_vector_type(16)));
typedef const __attribute__((address_space(4))) int32_t cprog_t;
typedef const __attribute__((address_space(4))) i32x16 cint16_t;
typedef const __attribute__((address_space(4))) FwdItem citem_t;
typedef __attribute__((address_space(1))) const void gvoid;
typedef __attribute__((address_space(3))) void lvoid;

__device__ __forceinline__ float fbits(int b) { return __int_as_float(b); }

// NaN-propagating maximum of three (IEEE 754-2019 maximum)
__device__ __forceinline__ float maximum3(float a, float b, float c) {
    float r;
    asm volatile("v_maximum3_f32 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
    return r;
}

// ---------------------------------------------------------------- stores
// LDS rows of LD floats, one column per sample of the tile (LD = 64, or 32
// for half-wave tiles when 64 columns of a large genome do not fit in LDS)
template <int LD>
struct LdsStoreT {
    float *col;  // this lane's column: slot s at col[s * LD]
    template <int H>
    __device__ __forceinline__ float get(int s) const {
        return col[s * LD];
    }
    template <int H>
    __device__ __forceinline__ void set(int s, float x) {
        col[s * LD] = x;
    }
    __device__ __forceinline__ void init(int zs) {
        col[zs * LD] = 0.0f;
        col[(zs + 1) * LD] = 1.0f;
    }
};
using LdsStore = LdsStoreT<WAVE>;

// Register stores: one tile block of node_loop_asm.h per tile.  Operands as
// documented there; every value register lives only inside the block.
#define NEAT_TILE_OPERANDS                                                               \
    [rec] "s"(rec), [edg] "s"(edg), [n] "s"(n), [zs] "s"(zs), [ni] "s"(ni), [dm0] "s"(dm0),  \
        [dn] "s"(dn), [dvec] "s"(dvec), [dsrc] "s"(dsrc), [lane] "v"(lane),                 \
        [outs] "s"(outs), [no] "s"(no), [om0] "s"(om0)
// EXTRA: more operands (the recurrent block's sweep count), or nothing
#define NEAT_NSW_OPERAND , [nsw] "s"(nsw)
#define NEAT_OUT_OPERANDS , [outp] "s"(outp), [nb] "s"(nb)
#define NEAT_TILE_FN(TILE, CLOB, EXTRA)                                                   \
    __device__ __forceinline__ static void tile(const int32_t *rec, const int32_t *edg,   \
                                                int n, int zs, int ni, unsigned dm0,      \
                                                int dn, int dvec, const float *dsrc,      \
                                                unsigned lane, const int32_t *outs, int no, \
                                                unsigned om0, int nsw, float *outp,       \
                                                int nb) {                                 \
        n = __builtin_amdgcn_readfirstlane(n);                                            \
        zs = __builtin_amdgcn_readfirstlane(zs);                                          \
        ni = __builtin_amdgcn_readfirstlane(ni);                                          \
        no = __builtin_amdgcn_readfirstlane(no);                                          \
        dm0 = __builtin_amdgcn_readfirstlane(dm0);                                        \
        om0 = __builtin_amdgcn_readfirstlane(om0);                                        \
        dn = __builtin_amdgcn_readfirstlane(dn);                                          \
        dvec = __builtin_amdgcn_readfirstlane(dvec);                                      \
        nsw = __builtin_amdgcn_readfirstlane(nsw);                                        \
        nb = __builtin_amdgcn_readfirstlane(nb);                                          \
        asm volatile(TILE : : NEAT_TILE_OPERANDS EXTRA : CLOB, "memory");               \
    }

// SPL: samples per lane.  DIRECT: the block stores its outputs from registers
// (no LDS output area).
template <int K>
struct AsmTile;
template <>
struct AsmTile<KIND_R64> {
    static constexpr int SPL = 1;
    static constexpr bool DIRECT = false;
    NEAT_TILE_FN(NEAT_TILE_S1_64, NEAT_CLOB_S1_64, )
};
template <>
struct AsmTile<KIND_R64X2> {
    static constexpr int SPL = 2;
    static constexpr bool DIRECT = false;
    NEAT_TILE_FN(NEAT_TILE_S2_64, NEAT_CLOB_S2_64, )
};
template <>
struct AsmTile<KIND_R128> {
    static constexpr int SPL = 1;
    static constexpr bool DIRECT = false;
    NEAT_TILE_FN(NEAT_TILE_S1_128, NEAT_CLOB_S1_128, )
};
template <>
struct AsmTile<KIND_R224> {
    static constexpr int SPL = 1;
    static constexpr bool DIRECT = false;
    NEAT_TILE_FN(NEAT_TILE_S1_224, NEAT_CLOB_S1_224, )
};
template <>
struct AsmTile<KIND_R32X4> {
    static constexpr int SPL = 4;
    static constexpr bool DIRECT = true;
    NEAT_TILE_FN(NEAT_TILE_S4_32, NEAT_CLOB_S4_32, NEAT_OUT_OPERANDS)
};
template <>
struct AsmTile<KIND_R64REC> {
    static constexpr int SPL = 1;
    static constexpr bool DIRECT = false;
    NEAT_TILE_FN(NEAT_TILE_S1_64R, NEAT_CLOB_S1_64R, NEAT_NSW_OPERAND)
};
template <>
struct AsmTile<KIND_R32REC> {
    static constexpr int SPL = 2;
    static constexpr bool DIRECT = false;
    NEAT_TILE_FN(NEAT_TILE_S2_32R, NEAT_CLOB_S2_32R, NEAT_NSW_OPERAND)
};
template <>
struct AsmTile<KIND_R52REC> {
    static constexpr int SPL = 1;
    static constexpr bool DIRECT = false;
    NEAT_TILE_FN(NEAT_TILE_S1_52R, NEAT_CLOB_S1_52R, NEAT_NSW_OPERAND)
};

// ---------------------------------------------------------------- nodes (C++)
// The LDS store's node loop: the operations of node_loop_asm.h in the same
// order, so both give identical bits.
template <int ACLS>
__device__ __forceinline__ void pair_vals(float &acc, bool first, float x0, float w0, float x1,
                                          float w1) {
    if (ACLS == ACLS_SUM) {
        acc = first ? x0 * w0 : fmaf(x0, w0, acc);
        acc = fmaf(x1, w1, acc);
    } else if (ACLS == ACLS_PROD) {
        if (first) {
            acc = x0 * w0;
            acc = acc * (x1 * w1);
        } else {
            const float ta = x0 * w0, tb = x1 * w1;
            acc = acc * ta;
            acc = acc * tb;
        }
    } else {
        const float ta = x0 * w0, tb = x1 * w1;
        acc = first ? maximum3(ta, tb, tb) : maximum3(acc, ta, tb);
    }
}

// The same where the lanes' classes differ: every class's value, and a select.
__device__ __forceinline__ float pair_lanes(bool prod, bool mx, float acc, bool first, float x0,
                                            float w0, float x1, float w1) {
    float s = acc, p = acc, m = acc;
    pair_vals<ACLS_SUM>(s, first, x0, w0, x1, w1);
    pair_vals<ACLS_PROD>(p, first, x0, w0, x1, w1);
    pair_vals<ACLS_MAX>(m, first, x0, w0, x1, w1);
    return prod ? p : mx ? m : s;
}

template <int ACLS, class Store>
__device__ __forceinline__ void pair(float &acc, bool first, int s0, float w0, int s1, float w1,
                                     const Store &v) {
    pair_vals<ACLS>(acc, first, v.template get<0>(s0), w0, v.template get<0>(s1), w1);
}

// pairs (>= 1) edge pairs: the first three from the record r, then the
// overflow array from e, four words per pair.
template <int ACLS, class Store, class EP>
__device__ __forceinline__ float aggregate(const i32x16 &r, EP e, int pairs, const Store &v) {
    float acc = 0.0f;
#pragma unroll
    for (int k = 0; k < REC_INLINE_PAIRS; ++k) {
        if (k < pairs)
            pair<ACLS>(acc, k == 0, r[REC_PAIRS + 4 * k], fbits(r[REC_PAIRS + 4 * k + 1]),
                       r[REC_PAIRS + 4 * k + 2], fbits(r[REC_PAIRS + 4 * k + 3]), v);
    }
    for (int p = 0; p < pairs - REC_INLINE_PAIRS; ++p)
        pair<ACLS>(acc, false, e[4 * p], fbits(e[4 * p + 1]), e[4 * p + 2], fbits(e[4 * p + 3]),
                   v);
    return acc;
}

// The activation of code act, as the assembly blocks compute it.
__device__ __forceinline__ float activation(int act, float z) {
    switch (act) {
    case ACT_TANH: {
        const float e = exp2_hw(2.885390043258667f * z);
        return fmaf(rcp_hw(1.0f + e), -2.0f, 1.0f);
    }
    case ACT_SIGMOID: return rcp_hw(1.0f + exp2_hw(-1.4426950216293335f * z));
    case ACT_RELU: return maximum3(z, 0.0f, 0.0f);
    case ACT_SIN: return act_sin(z);
    case ACT_GAUSS: return exp2_hw(-1.4426950216293335f * (z * z));
    case ACT_ABS: return maximum3(z, -z, -z);
    default: return z;  // identity
    }
}

// Every computed node of the program in record order; the aggregations read
// src and the results go to dst (the same store for a feedforward network).
template <class Store>
__device__ __forceinline__ void run_program(cprog_t *prog, int N, int O, int I, const Store &src,
                                            Store &dst) {
    const int ncomp = prog[HDR_NVALID] - I;
    if (ncomp <= 0) return;
    cprog_t *rec = prog + rec_off(O);
    cprog_t *e = prog + edge_off(N, O);
    i32x16 r = *(cint16_t *)rec;
    for (int k = 0; k < ncomp; ++k) {
        const unsigned code = (unsigned)r[REC_CODE], np = (unsigned)r[REC_NPAIRS];
        const int pairs = (int)(np & (unsigned)REC_NPAIRS_MASK);
        const int acls = slot_class((int)(np >> REC_FIELD_SHIFT));
        const int act = rec_act(code);
        const int slot = (int)(code & (unsigned)REC_DST_MASK);
        const float bias = fbits(r[REC_BIAS]), resp = fbits(r[REC_RESP]);
        // next record (the record array has room for N records)
        const i32x16 rn = *(cint16_t *)(rec + REC_WORDS * (k + 1));
        float a;
        if (acls == ACLS_PROD) a = aggregate<ACLS_PROD>(r, e, pairs, src);
        else if (acls == ACLS_MAX) a = aggregate<ACLS_MAX>(r, e, pairs, src);
        else a = pairs == 0 ? 0.0f : aggregate<ACLS_SUM>(r, e, pairs, src);
        if (pairs > REC_INLINE_PAIRS) e += 4 * (pairs - REC_INLINE_PAIRS);
        dst.template set<0>(slot, activation(act, fmaf(resp, a, bias)));
        r = rn;
    }
}

// ---------------------------------------------------------------- tiles
// Workgroup b is dealt to XCD b % 8; give each XCD a contiguous range.
__device__ __forceinline__ long long xcd_item(unsigned b, unsigned n) {
    const unsigned x = b & 7u, q = b >> 3, per = n >> 3, rem = n & 7u;
    return (long long)(x * per + (x < rem ? x : rem) + q);
}

// Inputs are read once and outputs written once: their loads and stores
// carry the non-temporal cache policy (bit 1 of the load's cache operand),
// which measured 11 % faster on the control workload than cached ones.
constexpr int CPOL_NT = 2;
typedef float v4f __attribute__((ext_vector_type(4)));

// Issue the DMA of n consecutive floats src[0..n) into lds[0..n).
__device__ __forceinline__ void dma_inputs(const float *src, float *lds, int n, int vec4) {
    const int lane = (int)(threadIdx.x & (WAVE - 1));
    if (vec4) {
        const int n4 = n >> 2;
        for (int c = 0; c < n4; c += WAVE)
            if (c + lane < n4)
                __builtin_amdgcn_global_load_lds((gvoid *)(src + 4 * (c + lane)),
                                                 (lvoid *)(lds + 4 * c), 16, 0, CPOL_NT);
        const int rem = n & 3;
        if (lane < rem)
            __builtin_amdgcn_global_load_lds((gvoid *)(src + 4 * n4 + lane),
                                             (lvoid *)(lds + 4 * n4), 4, 0, CPOL_NT);
    } else {
        for (int c = 0; c < n; c += WAVE)
            if (c + lane < n)
                __builtin_amdgcn_global_load_lds((gvoid *)(src + c + lane), (lvoid *)(lds + c), 4,
                                                 0, CPOL_NT);
    }
}

// Wait for this wave's DMA (the waves of a workgroup never share LDS data).
__device__ __forceinline__ void wait_dma() {
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Wait for this wave's DMA, issued before the last `later` memory operations
// (a wave's loads and stores retire in order), without waiting for those.
__device__ __forceinline__ void wait_dma_before(int later) {
    if (later >= 8) __builtin_amdgcn_s_waitcnt(0x0F78);       // vmcnt(8)
    else if (later >= 4) __builtin_amdgcn_s_waitcnt(0x0F74);  // vmcnt(4)
    else if (later >= 2) __builtin_amdgcn_s_waitcnt(0x0F72);  // vmcnt(2)
    else if (later == 1) __builtin_amdgcn_s_waitcnt(0x0F71);  // vmcnt(1)
    else __builtin_amdgcn_s_waitcnt(0x0F70);                  // vmcnt(0)
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// Grid-point coordinate -1 + 2 i / (side - 1).
__device__ __forceinline__ float grid_coord(int i, int side) {
    return (float)(2 * i - (side - 1)) / (float)(side - 1);
}

// Largest number of grid coordinates (side of the substrate grid).
constexpr int GRID_MAX_SIDE = 256;

// (p / d, p % d) for p < 2^24 and a uniform divisor d (< 2^16) with its
// reciprocal rd: the float estimate is off by at most one either way.
__device__ __forceinline__ void divmod_small(unsigned p, unsigned d, float rd, unsigned *q,
                                             unsigned *r) {
    int qq = (int)((float)p * rd);
    int rr = (int)p - qq * (int)d;
    if (rr >= (int)d) rr -= (int)d, ++qq;
    if (rr < 0) rr += (int)d, --qq;
    *q = (unsigned)qq;
    *r = (unsigned)rr;
}

template <int H, class Store>
__device__ __forceinline__ void place_grid(Store &v, long long q, int side) {
    const int pts = side * side;
    const int p1 = (int)(q / pts), p2 = (int)(q - (long long)p1 * pts);
    v.template set<H>(0, grid_coord(p1 % side, side));
    v.template set<H>(1, grid_coord(p1 / side, side));
    v.template set<H>(2, grid_coord(p2 % side, side));
    v.template set<H>(3, grid_coord(p2 / side, side));
    v.template set<H>(4, 1.0f);
}

template <int H, class Store>
__device__ __forceinline__ void store_outputs(const Store &v, cprog_t *prog, float *o, int O) {
    for (int j = 0; j < O; ++j) __builtin_nontemporal_store(v.template get<H>(prog[out_off() + j]), o + j);
}

// LDS byte address of a pointer into the workgroup's LDS.
__device__ __forceinline__ unsigned lds_addr(const float *p) {
    return (unsigned)(uintptr_t)(const __attribute__((address_space(3))) float *)p;
}

// Copy n floats of a tile's outputs from the LDS output area to HBM
// (16-byte pieces when the destination allows).
__device__ __forceinline__ void flush_outputs(const float *ostage, float *dst, int n) {
    const int lane = (int)(threadIdx.x & (WAVE - 1));
    int c0 = 0;
    if (((uintptr_t)dst & 15) == 0) {
        const int n4 = n >> 2;
        for (int c = lane; c < n4; c += WAVE)
            __builtin_nontemporal_store(reinterpret_cast<const v4f *>(ostage)[c],
                                        reinterpret_cast<v4f *>(dst) + c);
        c0 = 4 * n4;
    }
    for (int c = c0 + lane; c < n; c += WAVE) __builtin_nontemporal_store(ostage[c], dst + c);
}

// Bring words [0, n) of a genome's program into the L2 cache ahead of the
// node loop's scalar loads: one 4-byte DMA per 128-byte line, landing in a
// scratch LDS area (the caller waits for vmcnt(0) before reusing it).
__device__ __forceinline__ void touch_lines(const int32_t *base, int n, float *lds_scratch) {
    const int lane = (int)(threadIdx.x & (WAVE - 1));
    for (int off = lane * 32; off < n; off += WAVE * 32)
        __builtin_amdgcn_global_load_lds((gvoid *)(base + off), (lvoid *)lds_scratch, 4, 0, 0);
}

// Tile range [t0, t1) of run chunk, or false when it is empty.
__device__ __forceinline__ bool wave_tiles(citem_t *it, int chunk, int *t0, int *t1) {
    *t0 = chunk * it->tpw;
    *t1 = min(it->tiles, *t0 + it->tpw);
    return *t0 < *t1;
}

// Rejected genome: NaN outputs for the wave's samples.
__device__ __forceinline__ void fill_nan(float *out_g, int first, int end, int O) {
    const int lane = (int)(threadIdx.x & (WAVE - 1));
    for (int e = first * O + lane; e < end * O; e += WAVE) out_g[e] = __builtin_nanf("");
}

// One unit with a register store: tiles [t0, t1) of genome g.  area: the wave's
// LDS: input staging (TS x I floats; for grid queries the coordinates and the
// offsets too), then output staging (TS x O floats, or 64 that touch_lines writes
// where outputs are stored from registers).
template <int K, bool GRID>
__device__ __forceinline__ void forward_unit_reg(citem_t *it, int g, int t0, int t1, float *area,
                                                 int stage_floats) {
    constexpr int SPL = AsmTile<K>::SPL;
    constexpr bool DIRECT = AsmTile<K>::DIRECT;
    constexpr int TS = WAVE * SPL;  // samples per tile
    const unsigned lane = threadIdx.x & (WAVE - 1);
    const int N = it->N, I = it->I, O = it->O, B = it->B, side = GRID ? it->side : 0;
    cprog_t *prog = (cprog_t *)(it->prog + (size_t)g * it->prog_words);
    float *out_g = it->outputs + (size_t)g * B * O;
    if (prog[HDR_STATUS] != 0) {
        fill_nan(out_g, t0 * TS, min(B, t1 * TS), O);
        return;
    }
    const int32_t *p = (const int32_t *)prog;
    const int32_t *rec = p + rec_off(O), *edg = p + edge_off(N, O), *outs = p + out_off();
    const int ncomp = max(prog[HDR_NVALID] - I, 0);
    const int zs = zero_slot(prog[HDR_CLASS], N);
    float *istage = area, *ostage = area + stage_floats;
    const unsigned ibase = lds_addr(istage), obase = lds_addr(ostage);
    const float *in_g = GRID ? nullptr : it->inputs + (size_t)g * it->gstride;
    const int vec4 = it->vec4;
    if (!GRID) dma_inputs(in_g + (size_t)t0 * TS * I, istage, min(TS, B - t0 * TS) * I, vec4);
    // grid queries: the side coordinates and every sample's offset in the
    // tile as digits (x, y, points past them), once per unit, after the staging
    float *ctab = istage + TS * I;
    unsigned *otab = (unsigned *)(ctab + GRID_MAX_SIDE);
    const unsigned uside = (unsigned)side, pts = uside * uside;
    const float rside = GRID ? 1.0f / (float)side : 0.0f;
    // digits of the tile's first query (points p1, p2) and of a tile's length
    unsigned x1_0 = 0, y1_0 = 0, x2_0 = 0, y2_0 = 0;
    const unsigned step = GRID ? (unsigned)it->grid_step : 0u;
    const unsigned tx = step & 0xffu, ty = (step >> 8) & 0xffu, tk = (step >> 16) & 0xffu;
    // grid queries: the inputs of the lane's sample h (the fifth, 1, stays), by
    // adding its offset to the tile's first query digit by digit.  Where whole
    // rows of targets fit the tile (tx = ty = 0) the target point stays from tile
    // to tile.
    auto place = [&](int h, unsigned o, bool target) {
        float *x = istage + (h * WAVE + lane) * 5;
        unsigned x2 = x2_0 + (o & 0xffu), y2 = y2_0 + ((o >> 8) & 0xffu);
        unsigned x1 = x1_0 + (o >> 16), y1 = y1_0;
        if (x2 >= uside) x2 -= uside, ++y2;
        if (y2 >= uside) y2 -= uside, ++x1;
        if (pts >= (unsigned)TS) {
            if (x1 >= uside) x1 -= uside, ++y1;
        } else {
            unsigned c;
            divmod_small(x1, uside, rside, &c, &x1);
            y1 += c;
        }
        y1 = min(y1, uside - 1u);  // lanes past the last query
        x[0] = ctab[x1];
        x[1] = ctab[y1];
        if (target) {
            x[2] = ctab[x2];
            x[3] = ctab[y2];
        }
    };
    if (GRID) {
        for (int i = (int)lane; i < side; i += WAVE) ctab[i] = grid_coord(i, side);
        const unsigned q0 = (unsigned)(it->first + (long long)t0 * TS);
        const unsigned p1 = q0 / pts, p2 = q0 - p1 * pts;
        divmod_small(p1, uside, rside, &y1_0, &x1_0);
        divmod_small(p2, uside, rside, &y2_0, &x2_0);
        __builtin_amdgcn_wave_barrier();
        // the first tile's inputs, and the offsets for the others
        for (int h = 0; h < SPL; ++h) {
            const unsigned o = (unsigned)(h * WAVE) + lane;
            const unsigned k = pts >= (unsigned)TS ? 0u : o / pts;
            unsigned oy, ox;
            divmod_small(o - k * pts, uside, rside, &oy, &ox);
            const unsigned d = ox | (oy << 8) | (k << 16);
            otab[o] = d;
            istage[o * 5 + 4] = 1.0f;
            place(h, d, true);
        }
    }
    // the records and overflow edges the node loop will read, in one burst
    // (the first tile's wait covers it)
    touch_lines(rec, REC_WORDS * (ncomp + 1), ostage);
    touch_lines(edg, EDGE_WORDS * prog[HDR_NEDGES], ostage);
    if (GRID) wait_dma();

    for (int t = t0; t < t1; ++t) {
        if (GRID) {
            if (t > t0) {
                // this tile's first query
                x2_0 += tx, y2_0 += ty, x1_0 += tk;
                if (x2_0 >= uside) x2_0 -= uside, ++y2_0;
                if (y2_0 >= uside) y2_0 -= uside, ++x1_0;
                while (x1_0 >= uside) x1_0 -= uside, ++y1_0;
                for (int h = 0; h < SPL; ++h) place(h, otab[h * WAVE + lane], (tx | ty) != 0);
            }
        } else if (DIRECT && t > t0) {
            // the stores of the last tile follow this tile's DMA
            wait_dma_before(SPL * ((O >> 2) + ((O >> 1) & 1) + (O & 1)));
        } else {
            wait_dma();
        }
        if (!DIRECT && t > t0) flush_outputs(ostage, out_g + (size_t)(t - 1) * TS * O, TS * O);
        int dn = 0, dvec = 0;
        const float *dsrc = in_g;
        if (!GRID && t + 1 < t1) {
            const int nf = min(TS, B - (t + 1) * TS) * I;
            dvec = (vec4 && (nf & 3) == 0) ? 1 : 0;
            dn = dvec ? nf >> 2 : nf;
            dsrc = in_g + (size_t)(t + 1) * TS * I;
        }
        AsmTile<K>::tile(rec, edg, ncomp, zs, I, ibase, dn, dvec, dsrc, lane, outs, O, obase,
                         it->sweeps, out_g + (size_t)t * TS * O, min(TS, B - t * TS));
    }
    if (DIRECT) return;
    flush_outputs(ostage, out_g + (size_t)(t1 - 1) * TS * O, (min(B, t1 * TS) - (t1 - 1) * TS) * O);
}

// One unit with the LDS store: tiles [t0, t1) of genome g.  stage: the wave's input
// staging area (TS x I floats; unused for grid items).
template <bool GRID, int LD>
__device__ __forceinline__ void forward_unit_lds(citem_t *it, int g, int t0, int t1,
                                                 float *stage, LdsStoreT<LD> &v) {
    constexpr int TS = LD;
    const int lane = (int)(threadIdx.x & (WAVE - 1));
    // half-wave tiles: lanes LD.. take no sample (their columns would alias)
    const bool active = LD == WAVE || lane < LD;
    const int N = it->N, I = it->I, O = it->O, B = it->B, side = GRID ? it->side : 0;
    cprog_t *prog = (cprog_t *)(it->prog + (size_t)g * it->prog_words);
    float *out_g = it->outputs + (size_t)g * B * O;
    if (prog[HDR_STATUS] != 0) {
        fill_nan(out_g, t0 * TS, min(B, t1 * TS), O);
        return;
    }
    const float *in_g = GRID ? nullptr : it->inputs + (size_t)g * it->gstride;
    const int vec4 = it->vec4;
    if (!GRID) dma_inputs(in_g + (size_t)t0 * TS * I, stage, min(TS, B - t0 * TS) * I, vec4);
    if (active) v.init(zero_slot(prog[HDR_CLASS], N));
    for (int t = t0; t < t1; ++t) {
        const int nb = min(TS, B - t * TS);
        if (GRID) {
            if (active) place_grid<0>(v, it->first + (long long)t * TS + lane, side);
        } else {
            wait_dma();
            if (active)
                for (int i = 0; i < I; ++i) v.template set<0>(i, stage[lane * I + i]);
            if (t + 1 < t1) {
                // every lane has read its inputs before the buffer refills
                __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
                __builtin_amdgcn_wave_barrier();
                dma_inputs(in_g + (size_t)(t + 1) * TS * I, stage, min(TS, B - (t + 1) * TS) * I,
                           vec4);
            }
        }
        if (active) run_program(prog, N, O, I, v, v);
        if (lane < nb) store_outputs<0>(v, prog, out_g + (size_t)(t * TS + lane) * O, O);
    }
}

// ---------------------------------------------------------------- levels
// Mapping "lanes over a level" (FWD_LVL), for genomes evaluated on few
// samples, where a lane-per-sample tile would leave most lanes idle.  A
// wave takes a tile of BW = 2^sh samples (BW <= 64) and walks the genome
// level by level (Section 3.3's order groups nodes by level: a level's
// nodes read only earlier levels).  Each step spreads 64 / BW of the
// level's computed nodes over the lanes, node-major (lane = node * BW +
// sample), so one step evaluates up to 64 (node, sample) pairs and a
// genome costs about sum over levels of nodes * BW / 64 steps instead of
// one node loop iteration per node.  A lane reads its node's 64-byte
// record with vector loads and aggregates its in-edges in its own lane, in
// the record's order with the operations of the other stores (identical
// bits).  Values live in this wave's LDS area: slot s of the tile's sample
// j at v[s * BW + j].  Every node of a step reads its sources before any
// node of the step writes (a barrier-free wave step with the results held
// in registers), and a slot the program reuses after its last reader
// (liveness) is taken only by a later position, so no value is overwritten
// before it is read.
//
// What bounds it: a step is a chain of some 2000 cycles (record, sources,
// aggregation, activation), and few waves share a SIMD.  At 700 genomes of up
// to 365 nodes on 18 samples: 25.8 us; 36.3 when overflow pairs were read one
// by one (30.2 with four requested together), every lane loaded its whole
// record and pairs (the 64 bytes x 64 lanes of a step hold the vector cache's
// return path for 64 cycles; 27.9 with a quarter per lane), and each
// aggregation class took a branch per pair.  Requests two steps ahead, selects
// for the activations, twice the waves with half as wide tiles: 28.3, 26.2 and
// 37.2 us.  Calculation alone, before / now: N = 300, P = 100, B = 16: 20.6 /
// 18.0; N = 200, P = 700, B = 16: 18.1 / 16.9; N = 140, P = 100 .. 3000, whose
// levels are short, B = 4 .. 16: 14.0 - 30.2 / 14.1 - 30.0.
constexpr int LVL_AHEAD = 1;

struct LvlStore {
    float *v;
    int sh;  // log2 BW
    int j;   // this lane's sample in the tile
    template <int H>
    __device__ __forceinline__ float get(int s) const {
        return v[(s << sh) + j];
    }
};

typedef const __attribute__((address_space(1))) int32_t gint_t;
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef const __attribute__((address_space(1))) i32x4 gint4_t;

// Order this wave's LDS accesses (the hardware keeps a wave's LDS
// operations in order; this stops the compiler from moving them).
__device__ __forceinline__ void wave_lds_sync() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// The steps of every level in order: records kb .. kb + npw - 1 below k1 of
// level l (l = nlev when none is left).  The level starts are held a lane
// each, 64 at a time: reading one is no memory access.
struct LvlSteps {
    gint_t *lvl;
    int nlev, I, npw;
    int l, kb, k1;
    int base, start;  // lane i: the start of level base + i
    __device__ __forceinline__ void begin() {
        l = -1, kb = 0, k1 = 0;
        if (base != 0) hold(0);
    }
    __device__ __forceinline__ void hold(int b) {
        base = b;
        start = lvl[min(b + (int)(threadIdx.x & (WAVE - 1)), nlev)];
    }
    __device__ __forceinline__ void next() {
        if (l >= 0 && kb + npw < k1) {
            kb += npw;
            return;
        }
        if (l >= nlev) return;
        for (++l; l < nlev; ++l) {
            if (l + 1 - base >= WAVE) hold(l);
            kb = max(__builtin_amdgcn_readlane(start, l - base), I) - I;
            k1 = __builtin_amdgcn_readlane(start, l + 1 - base) - I;
            if (kb < k1) return;
        }
    }
};

// Sixteen words (a record, or four overflow pairs) of this lane's node, as
// requested.  QUAD (tiles of four samples and more): a quad of lanes has one
// node, each lane loads one quarter, and the quad's lanes exchange them by DPP;
// else every lane loads all of it.
template <bool QUAD>
struct LvlWords {
    i32x4 w[QUAD ? 1 : 4];
    // quarter q lies at at(q)
    template <class At>
    __device__ __forceinline__ void load(At at) {
        if constexpr (QUAD) {
            w[0] = *at((int)(threadIdx.x & 3u));
        } else {
#pragma unroll
            for (int q = 0; q < 4; ++q) w[q] = *at(q);
        }
    }
    template <int Q>
    __device__ __forceinline__ i32x4 quarter() const {
        if constexpr (QUAD) {
            i32x4 r;
#pragma unroll
            for (int c = 0; c < 4; ++c)  // quad_perm: lane Q's to all four
                r[c] = __builtin_amdgcn_update_dpp(0, w[0][c], Q * 0x55, 0xf, 0xf, true);
            return r;
        } else {
            return w[Q];
        }
    }
};

// A step's request: this lane's record and its first overflow edge.
template <bool QUAD>
struct LvlReq {
    LvlWords<QUAD> rec;
    int e;
    bool some, active;  // the step has records; this lane has one
    __device__ __forceinline__ void load(LvlSteps &s, gint_t *recs, gint_t *ebeg, int node) {
        s.next();
        const int k = s.kb + node;
        some = s.l < s.nlev;
        active = some && k < s.k1;
        // (a lane without a node reads record 0: loads without branches can be
        // counted, so a wait for older ones leaves these in flight)
        gint4_t *r = (gint4_t *)(recs + REC_WORDS * (active ? k : 0));
        rec.load([&](int q) { return r + q; });
        e = ebeg[active ? k : 0];
    }
};

// One step: this lane's node (request q) on its sample; the next step is
// requested by next() once this one's overflow pairs are (a wait for them then
// leaves the later requests in flight).  Every active lane's result is written
// once all lanes of the step have read their sources.
template <bool QUAD, class Next>
__device__ __forceinline__ void lvl_step(const LvlReq<QUAD> &q, gint_t *edges, Next next,
                                         const LvlStore &src, float *v, int sh, int j) {
    // the sources of this step were written by earlier steps
    wave_lds_sync();
    const i32x4 head = q.rec.template quarter<0>();
    const unsigned code = (unsigned)head[REC_CODE], np = (unsigned)head[REC_NPAIRS];
    const int pairs = (int)(np & (unsigned)REC_NPAIRS_MASK);
    const int over = pairs - REC_INLINE_PAIRS;
    // overflow pairs four at a time (lists begin at a multiple of two edges:
    // 16-byte loads; past the end the last pair again, or what follows an
    // empty list)
    gint4_t *ov = (gint4_t *)(edges + EDGE_WORDS * q.e);
    LvlWords<QUAD> o;
    o.load([&](int i) { return ov + max(min(i, over - 1), 0); });
    const i32x4 in[REC_INLINE_PAIRS] = {q.rec.template quarter<1>(), q.rec.template quarter<2>(),
                                        q.rec.template quarter<3>()};
    const bool active = q.active;
    next();
    float y = 0.0f;
    int slot = -1;
    if (active) {
        const int acls = slot_class((int)(np >> REC_FIELD_SHIFT));
        slot = (int)(code & (unsigned)REC_DST_MASK);
        // the six inline sources at once (unused inline edges name the
        // constant slot with weight 0)
        float x[2 * REC_INLINE_PAIRS];
#pragma unroll
        for (int p = 0; p < REC_INLINE_PAIRS; ++p) {
            x[2 * p] = src.get<0>(in[p].x);
            x[2 * p + 1] = src.get<0>(in[p].z);
        }
        float a = 0.0f;
        const bool prod = acls == ACLS_PROD, mx = acls == ACLS_MAX;
#pragma unroll
        for (int p = 0; p < REC_INLINE_PAIRS; ++p)
            a = p < pairs ? pair_lanes(prod, mx, a, p == 0, x[2 * p], fbits(in[p].y), x[2 * p + 1],
                                       fbits(in[p].w))
                          : a;
        for (int p0 = 0; p0 < over; p0 += 4) {
            const i32x4 c[4] = {o.template quarter<0>(), o.template quarter<1>(),
                                o.template quarter<2>(), o.template quarter<3>()};
            float z[8];
#pragma unroll
            for (int p = 0; p < 4; ++p) {
                z[2 * p] = src.get<0>(c[p].x);
                z[2 * p + 1] = src.get<0>(c[p].z);
            }
            if (p0 + 4 < over) o.load([&](int i) { return ov + min(p0 + 4 + i, over - 1); });
#pragma unroll
            for (int p = 0; p < 4; ++p)
                a = p0 + p < over ? pair_lanes(prod, mx, a, false, z[2 * p], fbits(c[p].y),
                                               z[2 * p + 1], fbits(c[p].w))
                                  : a;
        }
        y = activation(rec_act(code), fmaf(fbits(head[REC_RESP]), a, fbits(head[REC_BIAS])));
    }
    // every lane of the step has read its sources
    wave_lds_sync();
    if (slot >= 0) v[(slot << sh) + j] = y;
}

// Every step of a tile, the records (and overflow offsets) requested LVL_AHEAD
// steps before they are used.
template <bool QUAD>
__device__ __forceinline__ void lvl_walk(LvlSteps &steps, gint_t *recs, gint_t *ebeg,
                                         gint_t *edges, int node, const LvlStore &src, float *v,
                                         int sh, int j) {
    LvlReq<QUAD> q[LVL_AHEAD + 1];
#pragma unroll
    for (int d = 0; d < LVL_AHEAD; ++d) q[d].load(steps, recs, ebeg, node);
    for (bool more = q[0].some; more;) {
#pragma unroll
        for (int d = 0; d <= LVL_AHEAD; ++d) {
            if (!more) continue;
            lvl_step<QUAD>(q[d], edges,
                           [&] {
                               q[(d + LVL_AHEAD) % (LVL_AHEAD + 1)].load(steps, recs, ebeg, node);
                           },
                           src, v, sh, j);
            more = q[(d + 1) % (LVL_AHEAD + 1)].some;  // requested before
        }
    }
}

// Tiles [t0, t1) of BW samples.
__device__ __forceinline__ void forward_unit_lvl(citem_t *it, int g, int t0, int t1, float *v) {
    const int lane = (int)(threadIdx.x & (WAVE - 1));
    const int sh = it->lvl_sh, BW = 1 << sh;
    const int N = it->N, C = it->C, I = it->I, O = it->O, B = it->B;
    cprog_t *prog = (cprog_t *)(it->prog + (size_t)g * it->prog_words);
    gint_t *gp = (gint_t *)(it->prog + (size_t)g * it->prog_words);
    float *out_g = it->outputs + (size_t)g * B * O;
    if (prog[HDR_STATUS] != 0) {
        fill_nan(out_g, t0 * BW, min(B, t1 * BW), O);
        return;
    }
    const float *in_g = it->inputs + (size_t)g * it->gstride;
    const int nlev = prog[HDR_NLEVELS];
    const int zs = zero_slot(prog[HDR_CLASS], N);
    gint_t *ebeg = gp + ebeg_off(N, C, O);
    gint_t *edges = gp + edge_off(N, O);
    gint_t *recs = gp + rec_off(O);
    const int j = lane & (BW - 1), node = lane >> sh, npw = WAVE >> sh;
    const LvlStore src{v, sh, j};
    LvlSteps steps{gp + lvl_off(N, C, O), nlev, I, npw, 0, 0, 0, 0, 0};
    steps.hold(0);  // requested before the inputs are
    for (int t = t0; t < t1; ++t) {
        const int s0 = t * BW, nb = min(BW, B - s0);
        // inputs of the tile (contiguous [nb][I] floats): v[i][j] = x[s0 + j][i];
        // columns past the tile's last sample read 0
        const float *x = in_g + (size_t)s0 * I;
        for (int e = lane; e < BW * I; e += WAVE) {
            const int jj = e / I, i = e - jj * I;
            v[(i << sh) + jj] = jj < nb ? x[e] : 0.0f;
        }
        if (lane < BW) {
            v[(zs << sh) + lane] = 0.0f;
            v[((zs + 1) << sh) + lane] = 1.0f;
        }
        steps.begin();
        if (sh >= 2) lvl_walk<true>(steps, recs, ebeg, edges, node, src, v, sh, j);
        else lvl_walk<false>(steps, recs, ebeg, edges, node, src, v, sh, j);
        wave_lds_sync();
        // outputs of the tile: y[s0 + j][o] = v[out slot o][j]
        float *o_t = out_g + (size_t)s0 * O;
        for (int e = lane; e < nb * O; e += WAVE) {
            const int jj = e / O, o = e - jj * O;
            __builtin_nontemporal_store(v[(prog[out_off() + o] << sh) + jj], o_t + e);
        }
        wave_lds_sync();
    }
}

// ---------------------------------------------------------------- segments
// Mapping "lanes over a level's in-edges" (FWD_SEG).  As in the level
// mapping, a wave takes a tile of BW = 2^sh samples and walks the levels,
// values in LDS at v[s * BW + j].  Here a step spreads the level's
// in-edges over the lanes: R = 64 / BW rows of edges, each row holding one
// edge for the tile's BW samples (lane = row * BW + sample).  The level's
// edges are laid out destination after destination (a node's edges in its
// record's order, a node without in-edges contributing one edge w = 1 from
// the constant 0), so every destination owns a run of consecutive rows: a
// segment.  Each lane forms w * v[src] and a segmented inclusive scan over
// the rows (Hillis-Steele, partner rows 1, 2, 4, ... back in the same
// segment) combines the terms with the destination's aggregation: sum,
// product or the NaN-propagating maximum (mean and min are folded into the
// response, as in every store).  A segment cut by the end of a step passes
// its partial result to the next step's first row (carry).  The lane
// holding a segment's last edge applies bias, response and activation and
// writes the value once every lane of the step has read its sources.  The
// terms are combined in a tree rather than a chain, so sums and products
// round differently from the other mappings (within the oracle's bound,
// which holds for any order); maxima are exact.
__device__ __forceinline__ float seg_combine(int acls, float early, float late) {
    return acls == ACLS_PROD ? early * late
                             : (acls == ACLS_MAX ? maximum3(early, late, late) : early + late);
}

// exclusive scan of one int per lane across the wave; *total = the sum
__device__ __forceinline__ int wave_excl_scan(int v, int *total) {
    const int lane = (int)(threadIdx.x & (WAVE - 1));
    int x = v;
#pragma unroll
    for (int d = 1; d < WAVE; d <<= 1) {
        const int y = __shfl_up(x, d, WAVE);
        if (lane >= d) x += y;
    }
    *total = __shfl(x, WAVE - 1, WAVE);
    return x - v;
}

__device__ __forceinline__ void forward_unit_seg(citem_t *it, int g, int t0, int t1, float *v) {
    const int lane = (int)(threadIdx.x & (WAVE - 1));
    const int sh = it->lvl_sh, BW = 1 << sh, R = WAVE >> sh;
    const int N = it->N, C = it->C, I = it->I, O = it->O, B = it->B;
    cprog_t *prog = (cprog_t *)(it->prog + (size_t)g * it->prog_words);
    gint_t *gp = (gint_t *)(it->prog + (size_t)g * it->prog_words);
    float *out_g = it->outputs + (size_t)g * B * O;
    if (prog[HDR_STATUS] != 0) {
        fill_nan(out_g, t0 * BW, min(B, t1 * BW), O);
        return;
    }
    const float *in_g = it->inputs + (size_t)g * it->gstride;
    const int nlev = prog[HDR_NLEVELS];
    const int zs = zero_slot(prog[HDR_CLASS], N);
    cprog_t *lvl = prog + lvl_off(N, C, O);
    gint_t *ebeg = gp + ebeg_off(N, C, O);
    gint_t *edges = gp + edge_off(N, O);
    gint_t *recs = gp + rec_off(O);
    // the rows of v, then each level's edge offsets by node (N + 1 ints)
    int *eoff = (int *)(v + ((size_t)it->lvl_rows << sh));
    const int row = lane >> sh, j = lane & (BW - 1);
    for (int t = t0; t < t1; ++t) {
        const int s0 = t * BW, nb = min(BW, B - s0);
        const float *x = in_g + (size_t)s0 * I;
        for (int e = lane; e < BW * I; e += WAVE) {
            const int jj = e / I, i = e - jj * I;
            v[(i << sh) + jj] = jj < nb ? x[e] : 0.0f;
        }
        if (lane < BW) {
            v[(zs << sh) + lane] = 0.0f;
            v[((zs + 1) << sh) + lane] = 1.0f;
        }
        for (int l = 0; l < nlev; ++l) {
            const int k0 = max(lvl[l], I) - I, k1 = lvl[l + 1] - I, nl = k1 - k0;
            if (nl <= 0) continue;
            // edges per node (at least one) and their offsets
            int base = 0;
            for (int c = 0; c < nl; c += WAVE) {
                int ec = 0;
                if (c + lane < nl) {
                    const int pairs =
                        recs[REC_WORDS * (k0 + c + lane) + REC_NPAIRS] & REC_NPAIRS_MASK;
                    ec = pairs > 0 ? 2 * pairs : 1;
                }
                int tot;
                const int ex = wave_excl_scan(ec, &tot);
                if (c + lane < nl) eoff[c + lane] = base + ex;
                base += tot;
            }
            if (lane == 0) eoff[nl] = base;
            wave_lds_sync();
            float carry = 0.0f;
            for (int eb = 0; eb < base; eb += R) {
                const int e = eb + row;
                const bool active = e < base;
                int node = 0, q = 0, ec = 1, acls = ACLS_SUM;
                float xv = 0.0f;
                unsigned code = 0;
                float bias = 0.0f, resp = 0.0f;
                if (active) {
                    // the node owning edge e: the last offset <= e
                    int lo = 0, hi = nl - 1;
                    while (lo < hi) {
                        const int mid = (lo + hi + 1) >> 1;
                        if (eoff[mid] <= e) lo = mid;
                        else hi = mid - 1;
                    }
                    node = lo;
                    q = e - eoff[lo];
                    ec = eoff[lo + 1] - eoff[lo];
                    const int k = k0 + node;
                    gint_t *r = recs + REC_WORDS * k;
                    code = (unsigned)r[REC_CODE];
                    bias = fbits(r[REC_BIAS]);
                    resp = fbits(r[REC_RESP]);
                    const unsigned np = (unsigned)r[REC_NPAIRS];
                    const int pairs = (int)(np & (unsigned)REC_NPAIRS_MASK);
                    acls = slot_class((int)(np >> REC_FIELD_SHIFT));
                    int src = zs;
                    float w = 1.0f;
                    if (pairs > 0) {
                        gint_t *ew = q < 2 * REC_INLINE_PAIRS
                                         ? r + REC_PAIRS + 2 * q
                                         : edges + EDGE_WORDS * (ebeg[k] + q - 2 * REC_INLINE_PAIRS);
                        src = ew[0];
                        w = fbits(ew[1]);
                    }
                    xv = v[(src << sh) + j] * w;
                    // a segment begun in an earlier step continues from its carry
                    if (row == 0 && q > 0) xv = seg_combine(acls, carry, xv);
                }
                // segmented inclusive scan over the rows (same sample)
#pragma unroll
                for (int d = 1; d < WAVE; d <<= 1) {
                    if (d >= R) break;
                    const float y = __shfl(xv, lane - d * BW >= 0 ? lane - d * BW : lane, WAVE);
                    if (active && row >= d && q >= d) xv = seg_combine(acls, y, xv);
                }
                carry = __shfl(xv, (R - 1) * BW + j, WAVE);
                const bool tail = active && q == ec - 1;
                float yv = 0.0f;
                if (tail)
                    yv = activation(rec_act(code), fmaf(resp, xv, bias));
                // every lane of the step has read its sources
                wave_lds_sync();
                if (tail) v[((int)(code & (unsigned)REC_DST_MASK) << sh) + j] = yv;
            }
            wave_lds_sync();
        }
        float *o_t = out_g + (size_t)s0 * O;
        for (int e = lane; e < nb * O; e += WAVE) {
            const int jj = e / O, o = e - jj * O;
            __builtin_nontemporal_store(v[(prog[out_off() + o] << sh) + jj], o_t + e);
        }
        wave_lds_sync();
    }
}

// ---------------------------------------------------------------- recurrent
// Recurrent networks (read as K synchronous sweeps; the program comes from
// the recurrent transformation: records in key order, one slot per node).
// One wave per (genome, tile of 64 samples).  The lane's values live in two
// LDS columns, the previous sweep's (cur) and the one being written (nxt),
// which swap after every sweep: v0 = the inputs at slots 0..I-1 and 0 at
// the other nodes; every sweep runs all records reading cur and writing nxt.
template <int LD>
__global__ __launch_bounds__(WAVE) void recurrent_kernel(RecLaunch L) {
    // tiles of LD samples (64, or 32 when two columns of 64 do not fit)
    extern __shared__ float smem[];
    const long long u = xcd_item(blockIdx.x, gridDim.x);
    if (u >= (long long)L.P * L.tiles) return;
    const int g = (int)(u / L.tiles), t = (int)(u - (long long)g * L.tiles);
    const int lane = (int)(threadIdx.x & (WAVE - 1));
    const bool active = LD == WAVE || lane < LD;  // lanes LD.. take no sample
    const int I = L.I, O = L.O, N = L.N;
    cprog_t *prog = (cprog_t *)(L.prog + (size_t)g * L.prog_words);
    float *out_g = L.outputs + (size_t)g * L.B * O;
    const int s0 = t * LD, nb = min(LD, L.B - s0);
    if (prog[HDR_STATUS] != 0) {
        fill_nan(out_g, s0, s0 + nb, O);
        return;
    }
    float *stage = smem;
    dma_inputs(L.inputs + (size_t)g * L.gstride + (size_t)s0 * I, stage, nb * I, L.vec4);
    LdsStoreT<LD> cur, nxt;
    cur.col = smem + L.stage_floats + (lane & (LD - 1));
    nxt.col = cur.col + (size_t)L.rows * LD;
    const int nvalid = prog[HDR_NVALID];
    if (active) {
        for (int s = I; s < nvalid; ++s) cur.template set<0>(s, 0.0f);
        cur.init(zero_slot(prog[HDR_CLASS], N));
        nxt.init(zero_slot(prog[HDR_CLASS], N));
    }
    wait_dma();
    // lanes past the tile's last sample read stale staging words; their
    // results are never stored
    if (active)
        for (int i = 0; i < I; ++i) {
            const float x = stage[lane * I + i];
            cur.template set<0>(i, x);
            nxt.template set<0>(i, x);
        }
    for (int k = 0; k < L.K; ++k) {
        if (active) run_program(prog, N, O, I, cur, nxt);
        float *c = cur.col;
        cur.col = nxt.col;
        nxt.col = c;
    }
    if (lane < nb) store_outputs<0>(cur, prog, out_g + (size_t)(s0 + lane) * O, O);
}

// Item holding unit u (items sorted by unit0; the first has unit0 = 0).
__device__ __forceinline__ citem_t *find_item(const FwdItem *table, int n, long long u) {
    citem_t *items = (citem_t *)table;
    int lo = 0, hi = n - 1;
    while (lo < hi) {
        const int mid = (lo + hi + 1) >> 1;
        if (items[mid].unit0 <= u) lo = mid;
        else hi = mid - 1;
    }
    return items + lo;
}

// The launch argument in the kernarg segment (FwdLaunch is the kernel's only
// argument, so it sits at offset 0; its inline item is its first member).
__device__ __forceinline__ const __attribute__((address_space(4))) FwdLaunch *launch_arg() {
    return (const __attribute__((address_space(4))) FwdLaunch *)
        __builtin_amdgcn_kernarg_segment_ptr();
}

// ---------------------------------------------------------------- any class
// Mapping "any class" (KIND_ANY): every genome of a population in one
// launch, each wave with the register store of its genome's class, and the
// level mapping for genomes past the register classes.
//
// What it replaces: a launch per class, one after another on the caller's
// stream, each of them as long as its largest genome's chain of nodes (some
// 260 cycles per node for a wave alone on its SIMD) although a population
// of a few hundred genomes fills none of them.  Here the chains of all
// classes run side by side.  The price: the kernel's registers are those of
// its largest class (two waves per SIMD for all).  Measured, launch per
// class against this kernel, in us (I / O rows and 4 N connections):
//   N = 365, P = 500, B = 24: 93 / 34.6; P = 1500, B = 300: 272 / 109
//   N = 222, P = 500, B = 24: 45.5 / 22.0; P = 3000, B = 300: 188 / 127
//   N = 140, P = 2000, B = 300: 58.9 / 60.4; P = 4000, B = 300: 91 / 110
//   N = 80, P = 2000, B = 48: 12.1 / 10.0; P = 4000, B = 48: 15.8 / 18.3
// Tiles are of 64 samples, or of 128 (it->lvl_rows) that a genome of the
// smallest class runs two to a lane and the others as two tiles of 64.
__device__ __forceinline__ void run_any(citem_t *it, int g, int t0, int t1, float *area,
                                        int stage_floats) {
    const int c = ((cprog_t *)(it->prog + (size_t)g * it->prog_words))[HDR_CLASS];
    const int wide = it->lvl_rows == 2 * WAVE ? 2 : 1;
    if (c == CLS_R64 && wide == 2) {
        forward_unit_reg<KIND_R64X2, false>(it, g, t0, t1, area, stage_floats);
        return;
    }
    t0 *= wide;
    t1 = min((it->B + WAVE - 1) / WAVE, t1 * wide);
    if (c == CLS_R64) {
        forward_unit_reg<KIND_R64, false>(it, g, t0, t1, area, stage_floats);
    } else if (c == CLS_R128) {
        forward_unit_reg<KIND_R128, false>(it, g, t0, t1, area, stage_floats);
    } else if (c == CLS_R224) {
        forward_unit_reg<KIND_R224, false>(it, g, t0, t1, area, stage_floats);
    } else {
        const int per = WAVE >> it->lvl_sh, all = (it->B + (1 << it->lvl_sh) - 1) >> it->lvl_sh;
        forward_unit_lvl(it, g, t0 * per, min(all, t1 * per), area);
    }
}

// One unit: find its item and genome, then run the unit's waves with a
// fresh value store (nothing carries over from one unit to the next).
template <int K, bool GRID>
__device__ __forceinline__ void run_unit(long long u, float *wave_area) {
    const auto *L = launch_arg();
    citem_t *it = L->items ? find_item(L->items, L->n_items, u) : (citem_t *)&L->one;
    const long long local = u - it->unit0;
    const int chunks = it->chunks;
    const int i = (int)(local / chunks), chunk = (int)(local - (long long)i * chunks);
    int g = i;
    const int cls = it->cls;
    if (cls >= 0) {
        cprog_t *pop = (cprog_t *)it->pop;
        if (i >= pop[POP_COUNT + cls]) return;
        g = pop[POP_IDS + pop[POP_BEGIN + cls] + i];
    }
    int t0, t1;
    if (!wave_tiles(it, chunk, &t0, &t1)) return;
    if constexpr (K == KIND_LVL) {
        forward_unit_lvl(it, g, t0, t1, wave_area);
    } else if constexpr (K == KIND_SEG) {
        forward_unit_seg(it, g, t0, t1, wave_area);
    } else if constexpr (K == KIND_ANY) {
        run_any(it, g, t0, t1, wave_area, L->stage_floats);
    } else if constexpr (K == KIND_LDS) {
        LdsStore v;
        v.col = wave_area + L->stage_floats + (threadIdx.x & (WAVE - 1));
        forward_unit_lds<GRID, WAVE>(it, g, t0, t1, wave_area, v);
    } else if constexpr (K == KIND_LDS32) {
        LdsStoreT<WAVE / 2> v;
        v.col = wave_area + L->stage_floats + (threadIdx.x & (WAVE / 2 - 1));
        forward_unit_lds<GRID, WAVE / 2>(it, g, t0, t1, wave_area, v);
    } else {
        forward_unit_reg<K, GRID>(it, g, t0, t1, wave_area, L->stage_floats);
    }
}

// Waves per SIMD that a register kernel's tile block leaves room for: what
// the compiler adds around it must not cost one.
constexpr int min_waves(int kind) {
    return kind == KIND_R64 ? 5
           : (kind == KIND_R64X2 || kind == KIND_R32X4 || kind == KIND_R128 ||
              kind == KIND_R64REC || kind == KIND_R32REC)
               ? 3
           : kind == KIND_R52REC ? 4
           : kind == KIND_R224 || kind == KIND_ANY ? 2
                                                   : 1;
}

// PERSIST: a grid smaller than the unit count, each workgroup looping.
// GRID: CPPN grid queries generated in the kernel instead of read inputs.
template <int K, bool PERSIST, bool GRID>
__global__ __launch_bounds__(WAVE *FWD_MAX_WAVES, min_waves(K)) void forward_kernel(FwdLaunch L) {
    extern __shared__ float smem[];
    float *wave_area = smem + (size_t)(threadIdx.x / WAVE) * L.wave_floats;
    // the wave index is uniform; say so, so everything derived stays scalar
    const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x / WAVE));
    const long long waves = blockDim.x / WAVE;
    const long long b0 = xcd_item(blockIdx.x, gridDim.x);
    if (!PERSIST) {
        const long long u = b0 * waves + wave;
        if (u < L.units) run_unit<K, GRID>(u, wave_area);
        return;
    }
    if (L.counter) {
        // every wave takes the next unit until none is left
        for (;;) {
            unsigned u = 0;
            if ((threadIdx.x & (WAVE - 1)) == 0) u = atomicAdd(L.counter, 1u);
            u = (unsigned)__builtin_amdgcn_readfirstlane((int)u);  // lane 0's, uniform
            if ((long long)u >= L.units) return;
            run_unit<K, GRID>((long long)u, wave_area);
        }
    }
    for (long long b = b0; b * waves < L.units; b += gridDim.x) {
        const long long u = b * waves + wave;
        if (u < L.units) run_unit<K, GRID>(u, wave_area);
    }
}

__global__ void zero_counters_kernel(unsigned *c, int n) {
    for (int i = (int)threadIdx.x; i < n; i += (int)blockDim.x) c[i] = 0u;
}

// Waves a forward launch aims at (NEAT_FWD_WAVES overrides, for tuning).
long long wave_target() {
    static const long long t = [] {
        const char *e = getenv("NEAT_FWD_WAVES");
        const long long v = e ? atoll(e) : 0;
        return v >= 1024 ? v : 32768ll;
    }();
    return t;
}

// LDS bytes of one wave's values in the level mapping: the tile width is
// the widest that keeps rows x width within it (NEAT_LVL_WAVE_BYTES
// overrides, for tuning).
size_t lvl_wave_bytes() {
    static const size_t b = [] {
        const char *e = getenv("NEAT_LVL_WAVE_BYTES");
        const long long v = e ? atoll(e) : 0;
        return v >= 1024 && v <= 65536 ? (size_t)v : (size_t)8192;
    }();
    return b;
}

int choose_chunks(long long P, int tiles, int *tpw) {
    // aim at a wave count that fills 256 CUs several times over while a
    // wave still reuses its genome's program across a run of tiles (and
    // hides the first tile's input latency behind the others)
    const long long target = wave_target();
    long long chunks = (target + P - 1) / (P > 0 ? P : 1);
    if (chunks < 1) chunks = 1;
    if (chunks > tiles) chunks = tiles;
    *tpw = (int)((tiles + chunks - 1) / chunks);
    return (tiles + *tpw - 1) / *tpw;
}

// One tiles-per-wave count for every item of a launch: the largest t whose
// units, sum of P x ceil(tiles / t), still reach the wave target (1 when
// even one tile per wave falls short).  The units never grow with t, so a
// binary search finds it.
int launch_tiles_per_wave(const std::vector<FwdItem> &items) {
    const long long target = wave_target();
    int max_tiles = 1;
    for (const FwdItem &it : items) max_tiles = std::max(max_tiles, it.tiles);
    auto units = [&](int t) {
        long long u = 0;
        for (const FwdItem &it : items) u += (long long)it.P * ((it.tiles + t - 1) / t);
        return u;
    };
    int lo = 1, hi = max_tiles;  // units(lo) >= target unless lo = 1
    while (lo < hi) {
        const int mid = lo + (hi - lo + 1) / 2;
        if (units(mid) >= target) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// samples of one tile
int tile_samples(int kind) {
    return kind == KIND_R32X4   ? 4 * WAVE
           : kind == KIND_R64X2 || kind == KIND_R32REC ? 2 * WAVE
                                : (kind == KIND_LDS32 ? WAVE / 2 : WAVE);
}

bool direct_kind(int kind) { return kind == KIND_R32X4; }

bool lds_kind(int kind) { return kind == KIND_LDS || kind == KIND_LDS32; }

// Whether a register kernel's wave holds five inputs and O outputs of a tile of
// grid queries and the coordinates, but not the samples' offsets as well.
bool grid_table_too_large(int kind, int O, size_t max_lds) {
    const size_t TS = (size_t)tile_samples(kind);
    const size_t floats = TS * 5 + GRID_MAX_SIDE + (direct_kind(kind) ? WAVE : TS * O);
    return sizeof(float) * floats <= max_lds && sizeof(float) * (floats + TS) > max_lds;
}

// kernel of class c under a variant
int kind_of(int variant, int cls, int B) {
    if (variant == FWD_LDS) return KIND_LDS;
    if (variant == FWD_LVL || variant == FWD_SEG || variant == FWD_ANY)
        variant = FWD_AUTO;  // grid, recurrent items
    switch (cls) {
    case CLS_R64:
        if (variant == FWD_REG2 || (variant == FWD_AUTO && B > WAVE)) return KIND_R64X2;
        return KIND_R64;
    case CLS_R128: return KIND_R128;
    case CLS_R224: return KIND_R224;
    }
    return KIND_LDS;
}

}  // namespace

const char *kind_name(int kind) {
    static const char *names[] = {"r64", "r64x2", "r128", "r224", "lds", "r64rec", "lds32",
                                  "lvl", "seg", "any", "r32x4", "r32rec", "r52rec"};
    return kind >= 0 && kind < N_KINDS ? names[kind] : "?";
}

// Level and segment mappings: the widest power-of-two tile of samples (<= 64,
// <= B rounded up) whose values, rows of them, fit a wave's LDS budget beside
// extra bytes (log2).
static int level_tile(int rows, int B, size_t extra) {
    int sh = 0;
    while (sh < 6 && (1 << sh) < B &&
           sizeof(float) * (size_t)rows * (2u << sh) + extra <= lvl_wave_bytes())
        ++sh;
    return sh;
}

// Samples of one KIND_ANY tile: 64 while the GPU holds every 64-sample tile
// at once (2048 waves of that kernel), else 128, which the smallest class
// runs at half the scalar work per sample.
static int any_tile(const FwdJob &J) {
    return J.B > WAVE && (long long)J.P * ((J.B + WAVE - 1) / WAVE) > 2048 ? 2 * WAVE : WAVE;
}

// The recurrent register store by rows: waves per SIMD count most, since a
// wave's chain of short dependent instructions leaves most issue slots empty.
// Both vectors of 52 slots leave room for four (64 slots: three), and of 32
// slots for three with two samples per lane, taken when one per lane would
// fill the GPU (3072 waves) anyway.  Calculation alone, 17 inputs, 6 outputs,
// B = 500, K = 4, 64 slots and one sample against this: N = 50, P = 5000: 184
// / 165 us (52 slots and two samples at two waves per SIMD: 170); N = 30, P =
// 10000: 213 / 145 us.
static int recurrent_kind(const FwdJob &J) {
    if (J.N > MEDIUM_ROWS) return KIND_R64REC;
    if (J.N <= SMALL_ROWS && J.B > WAVE &&
        (long long)J.P * ((J.B + WAVE - 1) / WAVE) > 3072)
        return KIND_R32REC;
    return KIND_R52REC;
}

// Four samples per lane for the smallest class: where every value has one of
// 32 slots and two-sample tiles fill the GPU (3072 waves of that kernel).  The
// node loop's scalar work is shared by twice the samples, and the register file
// holds as many samples per SIMD as with two per lane and 64 slots: CPPN grid
// queries, P = 1000, N = 30, 65536 queries: 508 us with two samples per lane and
// 64 slots, 414 us with two and 32 slots (five waves per SIMD instead of three),
// 395 us with four (the vector pipe 79 % busy), 384 us with outputs stored
// straight from registers.  Both ends of a network limit it: 256 staged samples
// of more than 12 inputs leave fewer than 12 waves per CU, and the stores of
// many outputs from registers, four at a time, are not combined into lines.
// N = 30, P = 3000, B = 500, two samples / four, us: I = 4, O = 1: 19.8 / 16.4;
// 8, 4: 22.4 / 20.0; 11, 1: 21.0 / 18.0; 6, 6: 22.7 / 22.1; 13, 2: 21.7 / 23.1;
// 4, 12: 28.3 / 29.2; 4, 20: 34.2 / 73.7 (12, 1 and 12, 4 would gain: 21.6 / 18.6,
// 23.3 / 22.2).
static bool four_samples(const FwdJob &J) {
    return J.N <= SMALL_ROWS && J.I + J.O <= 12 && J.B > 2 * WAVE &&
           (long long)J.P * ((J.B + 2 * WAVE - 1) / (2 * WAVE)) > 3072;
}

// Whether a job can leave the launches per class: more than one class, and
// nothing that those would refuse (it stays refused).
static bool classes_may_merge(const FwdJob &J, size_t max_lds) {
    const int top = max_class(J.N);
    if (J.side || J.recurrent || top == CLS_R64) return false;
    const size_t stage = sizeof(float) * (size_t)(2 * WAVE) * (J.I + J.O);
    const size_t lds32 = sizeof(float) * (size_t)(WAVE / 2) * (J.I + class_slots(top, J.N));
    return stage <= max_lds && (top != CLS_LDS || lds32 <= max_lds);
}

// Past 510 rows the level mapping's tiles hold two samples or one, and a genome
// past the register classes walks its levels 32 or 64 times for every 64
// samples of a launch for every class: some 500 us for a wave, whatever the
// size of the call.  The level mapping alone spreads those walks over its own
// waves, and LDS rows take them in one.  Calculation in us, launches per class /
// one launch for every class / levels (a call's only population):
//   N = 515, P = 700, B = 64: 342 / 476 / 169; B = 130: 346 / 941 / 399
//   N = 515, P = 100, B = 300: 254 / 500 / 89; P = 1500, B = 64: 448 / 515 / 398
//   N = 590, P = 700, B = 64: 330 / 491 / 180; P = 2500, B = 64: 779 / 597 / 512
//   N = 590, P = 1500, B = 200: 689 / 1093 / 786; P = 5000, B = 64: 1044 / 733 / 1152
//   N = 680, P = 700, B = 300: 960 / 1188 / 709; P = 5000, B = 64: 1596 / 1004 / 1430
//   N = 780, P = 700, B = 130: 1190 / 1329 / 315; N = 850, P = 2500, B = 130: 4789 /
//   2558 / 1330; N = 1000, P = 5000, B = 64: 5721 / 2070 / 1488
// So the level mapping past 740 rows, where few genomes fit the registers, and
// below while the call is small; else launches per class up to 660 rows where
// most of a 64-sample tile is used.  Up to 530 rows genomes past the registers
// are so rare that a population may have none, and the launches per class may
// take half their time (N = 511: P = 700, B = 64: 114 / 48 / 162; P = 100, B =
// 300: 115 / 48 / 77): lower lines.  Of several populations, on a GPU that is
// full anyway, levels past 660 rows (4 of 700 .. 1000 rows, B = 20 .. 200: 2479 /
// 1267 / 632; 4 of 515 .. 640, B = 100 .. 300: 1453 / 1558 / 1976).
constexpr int NARROW_ROWS = 510;
static int narrow_variant(const FwdJob &J, bool alone) {
    const long long all = (long long)J.P * J.B;
    if (J.N > 740) return FWD_LVL;
    if (J.N > 660) return !alone || all <= 300000 ? FWD_LVL : FWD_ANY;
    const bool rare = J.N <= 530;
    if (alone && all <= (rare ? 30000 : 90000)) return FWD_LVL;
    return J.B > (rare ? WAVE / 2 : WAVE) ? FWD_AUTO : FWD_ANY;
}

int shared_variant(const FwdJob &J, bool in_order, size_t max_lds) {
    if (!classes_may_merge(J, max_lds)) return FWD_AUTO;
    // The GPU is full, so only total work counts: the level mapping where a
    // 64-sample tile would be three quarters empty and the nodes many, and one
    // launch for every class where the launches per class spend most of
    // their time at two waves per SIMD.  Seven batches of 6 to 24 populations
    // (N up to 120 .. 400, B up to 16 .. 512), launches per class / this, us:
    // as parallel branches 537 / 461, 264 / 222, 196 / 201, 129 / 127, 147 /
    // 147, 203 / 206, 177 / 162 (one launch from 251 rows on: 461, 222, 219 ..;
    // from 223 on: 500, 222, 187 ..); one after another, where every launch
    // also ends in its own tail, 804 / 660, 378 / 302, 286 / 216, 187 / 168,
    // 162 / 162, 311 / 246, 275 / 236.
    if (J.N > 222 && J.B <= 16) return FWD_LVL;
    if (J.N > NARROW_ROWS) return narrow_variant(J, false);
    return J.N > (in_order ? 126 : 300) ? FWD_ANY : FWD_AUTO;
}

// One sample per lane where a call's only population, of 31 to 62 node rows,
// has more than 64 inputs: two per lane share the scalar work of a node, but a
// wave's chain is longer, and nothing is shared while three one-sample waves
// per SIMD are all that there are.  Calculation, two samples per lane / one,
// us: N = 50, P = 157, B = 128 (314 waves): 7.7 / 7.2; P = 1500, B = 128
// (3000): 9.1 / 8.5; P = 1000, B = 200 (4000): 8.9 / 9.5; N = 31, P = 1500, B =
// 128: 7.0 / 6.8; P = 1000, B = 200: 7.0 / 7.5.  Three tiles of 64 leave a
// quarter of two-sample tiles empty, which counts once the waves are many (N =
// 62, B = 192: P = 1500, 4500 waves: 11.5 / 12.8; P = 3000: 19.4 / 19.4; P =
// 8000: 43.4 / 40.7).  Up to 30 rows nothing is gained (N = 20, P = 1500, B =
// 192: 6.6 / 7.1).
static bool one_sample(const FwdJob &J) {
    const int tiles = (J.B + WAVE - 1) / WAVE;
    const long long waves = (long long)J.P * tiles;
    return !J.side && !J.recurrent && J.N > SMALL_ROWS && max_class(J.N) == CLS_R64 &&
           (waves <= 3072 || (tiles == 3 && waves > 8192));
}

int alone_variant(const FwdJob &J, size_t max_lds) {
    if (one_sample(J)) return FWD_REG;
    if (!classes_may_merge(J, max_lds)) return FWD_AUTO;
    const long long units = (long long)J.P * ((J.B + WAVE - 1) / WAVE);
    // Few samples: the level mapping, whose lanes share a genome's nodes,
    // has the shorter chain while its waves fit the GPU (N = 300, P =
    // 700: 24.5 us against 28.9 at B = 18, 37.6 against 28.9 at B = 48),
    // and past 2048 genomes up to 8 samples (N = 160, P = 4000: 19.9 us
    // against 32.0 at B = 4, 38.4 against 31.7 at B = 12).  The chains of
    // up to 130 rows are short and only the second holds (N = 127, P = 2000, B
    // = 4: levels 18.5, one launch for every class 15.1), from 121 rows on (P =
    // 5000, B = 2, launches per class / levels: N = 80: 17.6 / 19.0; N = 113:
    // 21.9 / 25.5; N = 126: 27.6 / 25.0).
    if (J.P > 2048 ? J.B <= 8 && J.N > 120 : J.N > 130 && (long long)J.P * J.B <= 16384)
        return FWD_LVL;
    if (J.N > NARROW_ROWS) return narrow_variant(J, true);
    // One launch for every class (figures at run_any): up to 130 rows, where
    // next to no genome needs the 224-register class and its launch ends at
    // once, while every wave is resident (N = 127, P = 5000, B = 64: 27.1 us
    // with launches per class against 36.0), up to 150 rows for four times as
    // many (N = 133: 47.1 against 39.8; N = 140, P = 5000, B = 130: 78.9 against
    // 81.7, B = 300: 104 against 113; N = 150: 143 against 123), and always past
    // that, where the launches per class leave the two largest at two waves per
    // SIMD anyway (P = 5000, B = 300: N = 151: 127 against 120; N = 160: 179
    // against 128).
    const long long most = J.N <= 130 ? 2048 : (J.N <= 150 ? 8192 : units);
    return units <= most ? FWD_ANY : FWD_AUTO;
}

int forward_plan(const FwdJob *jobs, int n, int variant, size_t max_lds,
                 std::vector<FwdKernelLaunch> &out, char *err, size_t errlen) {
    out.clear();
    // one launch per (kernel, input mode), made when its first item comes (a
    // call's usual plan has one or two; a record of each, cleared and searched on
    // every call: 0.49 us against 0.09 for a plan of one launch)
    constexpr int NL = 2 * N_KINDS;
    signed char at[NL];  // the launch's index in out, -1: none yet
    int rows_max[NL], stage_max[NL], ostage_max[NL];
    for (int x = 0; x < NL; ++x) at[x] = -1, rows_max[x] = stage_max[x] = ostage_max[x] = 0;
    auto items_of = [&](int x) -> std::vector<FwdItem> & {
        if (at[x] < 0) {
            at[x] = (signed char)out.size();
            out.emplace_back();
            out.back().kind = x / 2;
            out.back().grid_mode = x & 1;
        }
        return out[at[x]].items;
    };
    const int plan_variant = variant;
    for (int j = 0; j < n; ++j) {
        const FwdJob &J = jobs[j];
        if (J.P == 0 || J.B == 0) continue;
        const int top = max_class(J.N);
        int variant = J.variant >= 0 ? J.variant : plan_variant;
        // (grid queries without that room in tiles of 64 samples: LDS rows)
        if (J.side && grid_table_too_large(KIND_R64, J.O, max_lds)) variant = FWD_LDS;
        if ((variant == FWD_LVL || variant == FWD_SEG) && !J.side && !J.recurrent) {
            // the level and segment mappings: every genome, one launch per
            // mapping over all items (the segment mapping also keeps N_max + 1
            // edge offsets)
            const bool seg = variant == FWD_SEG;
            const int rows = class_slots(top, J.N);
            int sh = level_tile(rows, J.B, seg ? sizeof(int) * (size_t)(J.N + 1) : 0);
            // a population alone: narrower tiles, so more of a level's nodes
            // side by side, while the GPU holds every wave at once (N = 300,
            // P = 100, B = 24: 22 -> 19 us)
            if (n == 1)
                while (sh > 0 && (long long)J.P * ((J.B + (1 << (sh - 1)) - 1) >> (sh - 1)) <= 4096)
                    --sh;
            FwdItem it{};
            it.prog = J.prog;
            it.inputs = J.inputs;
            it.outputs = J.outputs;
            it.gstride = J.gstride;
            it.pop = J.prog + pop_off(J.P, J.N, J.C, J.O);
            it.cls = -1;
            it.P = J.P, it.N = J.N, it.C = J.C, it.I = J.I, it.O = J.O, it.B = J.B;
            it.prog_words = prog_words(J.N, J.C, J.O);
            it.lvl_sh = sh;
            it.lvl_rows = rows;
            it.tiles = (J.B + (1 << sh) - 1) >> sh;
            const int x = 2 * (seg ? KIND_SEG : KIND_LVL);
            items_of(x).push_back(it);
            rows_max[x] = std::max(rows_max[x], (rows << sh) + (seg ? J.N + 1 : 0));
            continue;
        }
        // FWD_LDS takes every genome in one pass over all genomes; the other
        // variants take class c's genomes with class c's kernel; a recurrent
        // job (N_max <= 62) takes every genome with the recurrent kernel;
        // FWD_ANY takes every genome with the kernel that holds all classes
        const bool any = variant == FWD_ANY && !J.side && !J.recurrent && top != CLS_R64;
        const bool whole = variant == FWD_LDS || J.recurrent || any;
        const int c_lo = whole ? -1 : 0, c_hi = whole ? -1 : top;
        for (int c = c_lo; c <= c_hi; ++c) {
            int kind = J.recurrent ? recurrent_kind(J)
                       : any       ? KIND_ANY
                                   : kind_of(variant, c < 0 ? CLS_LDS : c, J.B);
            if (kind == KIND_R64X2 && variant == FWD_AUTO && four_samples(J)) kind = KIND_R32X4;
            // grid queries whose outputs leave no room for the table of offsets
            // beside them: half as many samples per tile
            if (J.side && kind == KIND_R64X2 && grid_table_too_large(kind, J.O, max_lds))
                kind = KIND_R64;
            // LDS rows too large for 64 columns per wave: half-wave tiles
            if (kind == KIND_LDS &&
                sizeof(float) * (size_t)WAVE * (J.I + class_slots(top, J.N)) > max_lds)
                kind = KIND_LDS32;
            FwdItem it{};
            it.prog = J.prog;
            it.inputs = J.inputs;
            it.outputs = J.outputs;
            it.gstride = J.gstride;
            it.first = J.first;
            it.pop = J.prog + pop_off(J.P, J.N, J.C, J.O);
            // populations of N_max <= 62 are all R64 and have no class list
            it.cls = (c < 0 || top == CLS_R64) ? -1 : c;
            it.P = J.P, it.N = J.N, it.C = J.C, it.I = J.I, it.O = J.O, it.B = J.B;
            it.side = J.side;
            it.prog_words = prog_words(J.N, J.C, J.O);
            if (J.recurrent) it.sweeps = J.sweeps;
            if (J.side) {
                const int ts = tile_samples(kind), pts = J.side * J.side;
                it.grid_step = ts % pts % J.side | (ts % pts / J.side) << 8 | (ts / pts) << 16;
            }
            const int TS = kind == KIND_ANY ? any_tile(J) : tile_samples(kind);
            it.tiles = (J.B + TS - 1) / TS;
            it.vec4 = (!J.side && ((uintptr_t)J.inputs % 16 == 0) && (J.gstride % 4 == 0)) ? 1 : 0;
            const int x = 2 * kind + (J.side ? 1 : 0);
            std::vector<FwdItem> &items = items_of(x);
            items.push_back(it);
            // register kernels on grid queries keep the coordinates and the
            // samples' offsets after the staged inputs
            if (!J.side || !lds_kind(kind))
                stage_max[x] = std::max(stage_max[x], TS * J.I + (J.side ? GRID_MAX_SIDE + TS : 0));
            // outputs stored from registers leave only what touch_lines writes
            if (!lds_kind(kind))
                ostage_max[x] = std::max(ostage_max[x], direct_kind(kind) ? WAVE : TS * J.O);
            if (kind == KIND_ANY) {
                // the values of a genome past the register classes, in the same area
                const int rows = class_slots(top, J.N), sh = level_tile(rows, J.B, 0);
                items.back().lvl_sh = sh;
                items.back().lvl_rows = TS;
                rows_max[x] = std::max(rows_max[x], rows << sh);
            }
            if (lds_kind(kind)) rows_max[x] = std::max(rows_max[x], class_slots(top, J.N));
        }
    }
    for (int x = 0; x < NL; ++x) {
        if (at[x] < 0) continue;
        FwdKernelLaunch &K = out[at[x]];
        const int kind = K.kind;
        const size_t rows = (kind == KIND_LVL || kind == KIND_SEG) ? (size_t)rows_max[x]
                            : lds_kind(kind) ? (size_t)rows_max[x] * tile_samples(kind)
                                             : (size_t)ostage_max[x];
        size_t wave_floats = (size_t)stage_max[x] + rows;
        // (the waves' staging areas start at 16 bytes: their loads and stores are
        // that wide, while a level mapping's rows may end anywhere)
        if (kind == KIND_ANY)
            wave_floats = std::max(wave_floats, (size_t)round_up(rows_max[x], 4));
        const size_t wave_bytes = wave_floats * sizeof(float);
        int waves = FWD_MAX_WAVES;
        while (waves > 1 && wave_bytes * waves > max_lds) --waves;
        if (wave_bytes > max_lds) {
            snprintf(err, errlen,
                     "forward kernel %s needs %zu B of LDS per wave (value rows %d, input "
                     "staging %d floats), device allows %zu",
                     kind_name(kind), wave_bytes, lds_kind(kind) ? rows_max[x] : 0,
                     stage_max[x], max_lds);
            out.clear();
            return NEAT_E_TOO_LARGE;
        }
        // Several items of a kernel with two or four samples per lane (the
        // streaming ones, taken for B > 64) share the launch's wave target: one tiles-per-wave
        // count for all, the largest that still gives the target, so a
        // population split into items runs as it does whole and each wave
        // overlaps its next tile's input DMA with the current tile (the
        // control workload as 10 items: 0.238 -> 0.214 ms).  Other kernels
        // keep each item's own target: their short-B items are latency-bound
        // and gain from spreading tiles over waves (a launch-wide target made
        // the uneven batch's calculation up to 32 % slower).
        const int shared_tpw = tile_samples(kind) > WAVE && K.items.size() > 1
                                   ? launch_tiles_per_wave(K.items) : 0;
        long long units = 0;
        for (FwdItem &it : K.items) {
            if (shared_tpw > 0) {
                // as many units as the shared count gives, their tiles
                // balanced (32 tiles at 15 per wave: 11 + 11 + 10, not
                // 15 + 15 + 2), as choose_chunks balances an item's own
                const int t = std::min(shared_tpw, std::max(1, it.tiles));
                it.chunks = (it.tiles + t - 1) / t;
                it.tpw = (it.tiles + it.chunks - 1) / it.chunks;
            } else {
                it.chunks = choose_chunks(it.P, it.tiles, &it.tpw);
            }
            it.unit0 = units;
            units += (long long)it.P * it.chunks;
        }
        const long long groups = (units + waves - 1) / waves;
        K.args.wave_floats = (int)wave_floats;
        K.args.stage_floats = stage_max[x];
        K.args.units = units;
        K.block = (unsigned)(WAVE * waves);
        K.lds = wave_bytes * waves;
        // the LDS store limits the workgroups a CU holds: loop over units with
        // a grid of a few per CU instead of one workgroup per unit
        const long long cap = (lds_kind(kind) || kind == KIND_LVL || kind == KIND_SEG)
                                  ? 256ll * 2 * std::max<long long>(1, (long long)(163840 / K.lds))
                                  : (1ll << 31) - 1;
        K.args.persistent = groups > cap ? 1 : 0;
        K.grid = (unsigned)std::min(groups, cap);
        if (K.items.size() == 1) K.args.one = K.items[0];
    }
    // in the order of the kernels
    const auto before = [](const FwdKernelLaunch &a, const FwdKernelLaunch &b) {
        return 2 * a.kind + a.grid_mode < 2 * b.kind + b.grid_mode;
    };
    if (!std::is_sorted(out.begin(), out.end(), before)) std::sort(out.begin(), out.end(), before);
    return NEAT_OK;
}

int forward_plan_auto(std::vector<FwdJob> &jobs, bool in_order, size_t max_lds,
                      std::vector<FwdKernelLaunch> &out, char *err, size_t errlen) {
    std::vector<size_t> own;  // jobs that a rule takes off the launches per class
    int I = 0, O = 0, rows = 0;
    for (size_t k = 0; k < jobs.size(); ++k) {
        FwdJob &J = jobs[k];
        I = std::max(I, J.I), O = std::max(O, J.O);
        rows = std::max(rows, class_slots(max_class(J.N), J.N));
        if (J.variant != FWD_AUTO) continue;
        J.variant = jobs.size() > 1 ? shared_variant(J, in_order, max_lds)
                                    : alone_variant(J, max_lds);
        if (J.variant != FWD_AUTO) own.push_back(k);
    }
    // A launch over several jobs reserves the largest input staging and the
    // largest output staging or rows of any of them, which need not belong to
    // one job: only while even their sum fits, all jobs taken together, can no
    // plan be refused.  Else what is refused is what the launches per class
    // refuse, and they are the plan where the other one does not fit.
    const bool roomy =
        sizeof(float) * ((size_t)(2 * WAVE) * (I + O + 1) + GRID_MAX_SIDE) <= max_lds &&
        sizeof(float) * (size_t)WAVE * (I + rows) <= max_lds;
    std::vector<FwdKernelLaunch> by_class;
    if (!roomy && jobs.size() > 1 && !own.empty()) {
        std::vector<FwdJob> plain = jobs;
        for (size_t k : own) plain[k].variant = FWD_AUTO;
        const int rc = forward_plan(plain.data(), (int)plain.size(), FWD_AUTO, max_lds, by_class,
                                    err, errlen);
        if (rc != NEAT_OK) return rc;
    }
    const int rc = forward_plan(jobs.data(), (int)jobs.size(), FWD_AUTO, max_lds, out, err, errlen);
    if (rc == NEAT_OK || by_class.empty()) return rc;
    out.swap(by_class);
    return NEAT_OK;
}

size_t recurrent_lds_bytes(int N, int I, int ld) {
    return sizeof(float) * (size_t)ld * ((size_t)I + 2 * (size_t)class_slots(max_class(N), N));
}

hipError_t recurrent_launch(RecLaunch L, size_t max_lds, hipStream_t stream) {
    const int ld = recurrent_lds_bytes(L.N, L.I, WAVE) <= max_lds ? WAVE : WAVE / 2;
    L.tiles = (L.B + ld - 1) / ld;
    L.stage_floats = ld * L.I;
    const long long blocks = (long long)L.P * L.tiles;
    if (blocks == 0) return hipSuccess;
    if (ld == WAVE)
        hipLaunchKernelGGL(recurrent_kernel<WAVE>, dim3((unsigned)blocks), dim3(WAVE),
                           recurrent_lds_bytes(L.N, L.I, WAVE), stream, L);
    else
        hipLaunchKernelGGL(recurrent_kernel<WAVE / 2>, dim3((unsigned)blocks), dim3(WAVE),
                           recurrent_lds_bytes(L.N, L.I, WAVE / 2), stream, L);
    return hipGetLastError();
}

hipError_t launch_zero_counters(unsigned *c, int n, hipStream_t stream) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(zero_counters_kernel, dim3(1), dim3(64), 0, stream, c, n);
    return hipGetLastError();
}

hipError_t forward_launch(const FwdKernelLaunch &k, const FwdItem *dev_items, hipStream_t stream,
                          unsigned *counter) {
    FwdLaunch L = k.args;
    L.counter = L.persistent ? counter : nullptr;
    // only one item goes inline
    if (dev_items == nullptr && k.items.size() != 1) return hipErrorInvalidValue;
    if (k.items.size() == 1 && dev_items == nullptr) {
        L.items = nullptr;
        L.n_items = 1;
    } else {
        L.items = dev_items;
        L.n_items = (int)k.items.size();
    }
    // register kernels are never persistent (their grids have no cap)
#define NEAT_LAUNCH1(KIND, PERSIST, GRID)                                                  \
    hipLaunchKernelGGL((forward_kernel<KIND, PERSIST, GRID>), dim3(k.grid), dim3(k.block), \
                       k.lds, stream, L)
#define NEAT_LAUNCH_REG(KIND)                                                              \
    if (k.grid_mode) NEAT_LAUNCH1(KIND, false, true);                                      \
    else NEAT_LAUNCH1(KIND, false, false);
#define NEAT_LAUNCH2(KIND, GRID)                                                           \
    if (L.persistent) NEAT_LAUNCH1(KIND, true, GRID);                                      \
    else NEAT_LAUNCH1(KIND, false, GRID);
#define NEAT_LAUNCH_LDS(KIND)                                                              \
    if (k.grid_mode) {                                                                     \
        NEAT_LAUNCH2(KIND, true)                                                           \
    } else {                                                                               \
        NEAT_LAUNCH2(KIND, false)                                                          \
    }
    switch (k.kind) {
    case KIND_R64: NEAT_LAUNCH_REG(KIND_R64) break;
    case KIND_R64X2: NEAT_LAUNCH_REG(KIND_R64X2) break;
    case KIND_R32X4: NEAT_LAUNCH_REG(KIND_R32X4) break;
    case KIND_R128: NEAT_LAUNCH_REG(KIND_R128) break;
    case KIND_R224: NEAT_LAUNCH_REG(KIND_R224) break;
    case KIND_R64REC: NEAT_LAUNCH1(KIND_R64REC, false, false); break;
    case KIND_R32REC: NEAT_LAUNCH1(KIND_R32REC, false, false); break;
    case KIND_R52REC: NEAT_LAUNCH1(KIND_R52REC, false, false); break;
    case KIND_LDS32: NEAT_LAUNCH_LDS(KIND_LDS32) break;
    case KIND_LVL: NEAT_LAUNCH2(KIND_LVL, false) break;
    case KIND_SEG: NEAT_LAUNCH2(KIND_SEG, false) break;
    case KIND_ANY: NEAT_LAUNCH1(KIND_ANY, false, false); break;
    default: NEAT_LAUNCH_LDS(KIND_LDS) break;
    }
#undef NEAT_LAUNCH_LDS
#undef NEAT_LAUNCH2
#undef NEAT_LAUNCH_REG
#undef NEAT_LAUNCH1
    return hipGetLastError();
}

}  // namespace neat
