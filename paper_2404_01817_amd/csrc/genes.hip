// genes.hip -- gene-level population operators: NEAT's compatibility
// distance and crossover.
//
// Compatibility distance of every genome of a population to every species
// representative (speciation divides the
// population by distances between networks: the NEAT algorithm of the
// paper's appendix; Appendix A names the disjoint and homologous
// coefficients).  Per pair (genome A, representative B):
//   genes: node rows with a key, connection rows with an in key;
//   an A gene is homologous when B has a gene with the same key (nodes) or
//   the same (in, out) keys (connections), its partner being the first
//   such B row; node distance |bias - bias'| + |resp - resp'| + [act !=
//   act'] + [agg != agg'], connection distance |w - w'| + [enabled !=
//   enabled'];
//   per kind (cd (|A| + |B| - 2 h) + ch sum) / max(|A|, |B|), 0 when both
//   are empty; the distance is the node part plus the connection part.
//
// Two kernels: distance_dict_kernel (a dictionary of the keys of up to 16
// representatives in LDS, one lookup per gene for all of them), and
// distance_kernel (a table per representative) where not even one
// representative's dictionary fits.  Keys are compared as floats: -0 is
// folded into +0 before hashing, and a connection whose out key is NaN
// never matches.
#include <hip/hip_runtime.h>

#include <algorithm>

#include "genes.h"

namespace neat {
namespace {

constexpr int WAVE = 64;
constexpr unsigned long long EMPTY64 = ~0ull;

__device__ __forceinline__ unsigned key_bits(float k) {
    return __float_as_uint(k == 0.0f ? 0.0f : k);  // -0 -> +0
}

__device__ __forceinline__ unsigned mix(unsigned long long x, int H) {
    x ^= x >> 29;
    x *= 0xbf58476d1ce4e5b9ull;
    x ^= x >> 32;
    return (unsigned)x & (unsigned)(H - 1);
}

__device__ __forceinline__ int wave_sum(int v) {
    for (int o = WAVE / 2; o > 0; o >>= 1) v += __shfl_xor(v, o);
    return v;
}

// Wave sums on the DPP lane network (register-to-register, no LDS round
// trips): lanes pair up within rows of 16 (swap neighbours, swap pairs,
// mirror each half row, mirror the row), after which every lane of a row
// holds the row's sum; the four row sums are read out into scalars.  Called
// with the whole wave active.
constexpr int DPP_SWAP1 = 0xB1;      // quad_perm [1, 0, 3, 2]
constexpr int DPP_SWAP2 = 0x4E;      // quad_perm [2, 3, 0, 1]
constexpr int DPP_HALF_MIRROR = 0x141;
constexpr int DPP_MIRROR = 0x140;

__device__ __forceinline__ int row_sums(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, DPP_SWAP1, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, DPP_SWAP2, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, DPP_HALF_MIRROR, 0xF, 0xF, false);
    v += __builtin_amdgcn_update_dpp(0, v, DPP_MIRROR, 0xF, 0xF, false);
    return v;
}
__device__ __forceinline__ float row_sums(float v) {
#define NEAT_DPP_ADD(CTRL) \
    v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xF, 0xF, false))
    NEAT_DPP_ADD(DPP_SWAP1);
    NEAT_DPP_ADD(DPP_SWAP2);
    NEAT_DPP_ADD(DPP_HALF_MIRROR);
    NEAT_DPP_ADD(DPP_MIRROR);
#undef NEAT_DPP_ADD
    return v;
}
__device__ __forceinline__ int wave_total(int v) {
    v = row_sums(v);
    return __builtin_amdgcn_readlane(v, 0) + __builtin_amdgcn_readlane(v, 16) +
           __builtin_amdgcn_readlane(v, 32) + __builtin_amdgcn_readlane(v, 48);
}
__device__ __forceinline__ float wave_total(float v) {
    v = row_sums(v);
    const float r0 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 0));
    const float r1 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 16));
    const float r2 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 32));
    const float r3 = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(v), 48));
    return (r0 + r1) + (r2 + r3);
}

// insert key -> row (keeping the smallest row for a key)
__device__ __forceinline__ void insert(unsigned long long *hk, int *hr, int H,
                                       unsigned long long key, int row) {
    unsigned s = mix(key, H);
    for (;;) {
        const unsigned long long prev = atomicCAS(hk + s, EMPTY64, key);
        if (prev == EMPTY64 || prev == key) {
            atomicMin(hr + s, row);
            return;
        }
        s = (s + 1) & (unsigned)(H - 1);
    }
}

__device__ __forceinline__ int lookup(const unsigned long long *hk, const int *hr, int H,
                                      unsigned long long key) {
    unsigned s = mix(key, H);
    for (;;) {
        const unsigned long long k = hk[s];
        if (k == key) return hr[s];
        if (k == EMPTY64) return -1;
        s = (s + 1) & (unsigned)(H - 1);
    }
}

// ---- distance by dictionary.
//
// A workgroup takes up to R representatives and a run of genomes.  Every
// distinct key of its representatives gets one entry in an LDS hash table
// that holds, beside the key, the row each representative has the gene at
// (16 bytes: R row numbers of W bytes, all ones where it has none); the
// representatives' attributes are copied into LDS by row.  A wave then takes
// a genome at a time: each lane looks its genes up once (one node row and
// four connection rows per round) and, representative by representative,
// reads the partner's attributes directly.  Counts of homologous genes are
// ballots; the 2 R sums of attribute distances are folded over the lanes
// together (each step halves the values a lane holds), so lane l ends with
// one of them.
//
// What bounds it: vector issue (74 instructions per pair of a genome and a
// representative at N = 50, C = 200; the vector pipe 68 % busy).  The table
// lookups, whose probe loops run as long as the longest chain of any lane,
// are paid once per genome and group of representatives instead of once per
// pair, and the tables are built once per workgroup instead of once per
// eight genomes.  Measured against a table per representative: P = 10000,
// N = 50, C = 200, Q = 64: 465 -> 104 us; Q = 1: 21.8 -> 16.1 us; P = 1250,
// N = 400, C = 1600, Q = 64: 3460 -> 445 us.
// R: representatives of a group (at most 16 / W), RB: those that one test of
// the group's size covers.
template <int W, int R_, int RB_>
struct DictShape {
    static constexpr int R = R_, RB = RB_;
    static constexpr unsigned NONE = W == 1 ? 0xffu : 0xffffu;
    static constexpr int LN = WAVE / (2 * R);    // lanes per folded sum
    // the attribute row to read for row number j: one-byte numbers are read
    // as they are (the attributes are followed by 256 rows of LDS), the
    // result of an absent gene is dropped
    static __device__ __forceinline__ int index(unsigned j, bool hit) {
        return W == 1 || hit ? (int)j : 0;
    }
};
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ unsigned dict_slot(unsigned a, unsigned b, int shift) {
    unsigned h = (a ^ (a >> 13)) * 0x9e3779b1u + (b ^ (b >> 11)) * 0x85ebca77u;
    h ^= h >> 15;
    h *= 0x2c1b3c6du;
    return h >> shift;
}

// Row number of representative r in an entry's 16 bytes.
template <int W>
__device__ __forceinline__ unsigned dict_row(const u32x4 &e, int r) {
    return (e[r * W / 4] >> (8 * (r * W % 4))) & (W == 1 ? 0xffu : 0xffffu);
}

// Put row into representative r's place of entry s; true when the
// representative had the key already (the place then needs the repair).
template <int W>
__device__ __forceinline__ bool dict_put(unsigned *rows, unsigned s, int r, int row) {
    const int sh = 8 * (r * W % 4);
    const unsigned none = W == 1 ? 0xffu : 0xffffu;
    const unsigned old =
        atomicAnd(rows + 4 * s + r * W / 4, ~(none << sh) | ((unsigned)row << sh));
    return ((old >> sh) & none) != none;
}
template <int W>
__device__ __forceinline__ void dict_set(unsigned *rows, unsigned s, int r, int row) {
    if constexpr (W == 1) ((unsigned char *)(rows + 4 * s))[r] = (unsigned char)row;
    else ((unsigned short *)(rows + 4 * s))[r] = (unsigned short)row;
}

// One connection row (four floats) of a tensor that need not be 16-byte
// aligned.
__device__ __forceinline__ float4 conn_row(const float *p, bool vec) {
    if (vec) return *reinterpret_cast<const float4 *>(p);
    return make_float4(p[0], p[1], p[2], p[3]);
}

// a's and b's sums over the lanes that differ in one lane bit, a's in the
// lanes where the bit is 0 and b's where it is 1.
__device__ __forceinline__ float fold32(float a, float b) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
__device__ __forceinline__ float fold16(float a, float b) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(a), __float_as_uint(b), false,
                                                    false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}
// x is needed as loaded (a select on a fresh load would become a branch
// around it, and the loads one wait each)
__device__ __forceinline__ void keep(float &x) { asm volatile("" : "+v"(x)); }

template <int CTRL>
__device__ __forceinline__ float dpp_sum(float a) {
    return a + __int_as_float(
                   __builtin_amdgcn_update_dpp(0, __float_as_int(a), CTRL, 0xF, 0xF, false));
}
template <int CTRL>
__device__ __forceinline__ float fold_dpp(float a, float b, bool hi) {
    const float x = dpp_sum<CTRL>(a), y = dpp_sum<CTRL>(b);
    return hi ? y : x;
}
constexpr int DPP_ROR8 = 0x128;

template <int W, int R, int RB>
__global__ __launch_bounds__(1024) void distance_dict_kernel(DistLaunch L) {
    using D = DictShape<W, R, RB>;
    extern __shared__ __align__(16) unsigned char dict_lds[];
    const int N = L.N, C = L.C, HN = L.hn, HC = L.hc, rq = L.rq;
    const int ra = (rq + RB - 1) / RB * RB;  // attribute rows of whole guards
    unsigned *crow = (unsigned *)dict_lds;                       // [HC][4] rows by representative
    unsigned *nrow = crow + 4 * (size_t)HC;                      // [HN][4]
    float4 *nattr = (float4 *)(nrow + 4 * (size_t)HN);           // [ra][N] bias, resp, act, agg
    unsigned long long *ckey = (unsigned long long *)(nattr + (size_t)ra * N);  // [HC] in, out
    float2 *cattr = (float2 *)(ckey + HC);                       // [ra][C] enabled, weight
    unsigned *nkey = (unsigned *)(cattr + (size_t)ra * C);       // [HN]
    int *cnt = (int *)(nkey + HN);                               // [3][R] nodes, connections, repeats
    const int t = (int)threadIdx.x, T = (int)blockDim.x;
    const int lane = t & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane(t / WAVE), waves = T / WAVE;
    const int in_launch = (int)(blockIdx.x / (unsigned)L.blocks_per_group);
    const int part = (int)(blockIdx.x - (unsigned)in_launch * (unsigned)L.blocks_per_group);
    const int q0 = L.q_first + in_launch * rq, nq = min(rq, L.Q - q0);
    const int sn = 32 - L.hn_log2, sc = 32 - L.hc_log2;  // hash shifts
    const bool vec = L.vec != 0;

    // ---- the dictionary of representatives q0 .. q0 + nq - 1
    for (int s = t; s < HC; s += T) {
        ckey[s] = EMPTY64;
        ((u32x4 *)crow)[s] = u32x4{~0u, ~0u, ~0u, ~0u};
    }
    for (int s = t; s < HN; s += T) {
        nkey[s] = ~0u;
        ((u32x4 *)nrow)[s] = u32x4{~0u, ~0u, ~0u, ~0u};
    }
    if (t < 3 * R) cnt[t] = 0;
    __syncthreads();
    for (int i = t; i < nq * N; i += T) {
        const int r = i / N, row = i - r * N;
        const float *y = L.rnodes + (size_t)(q0 + r) * N * 5 + (size_t)row * 5;
        const float key = y[0];
        nattr[i] = make_float4(y[1], y[2], y[3], y[4]);
        if (isnan(key)) continue;
        atomicAdd(&cnt[r], 1);
        const unsigned k = key_bits(key);
        unsigned s = dict_slot(k, 0u, sn);
        for (;;) {
            const unsigned prev = atomicCAS(nkey + s, ~0u, k);
            if (prev == ~0u || prev == k) break;
            s = (s + 1) & (unsigned)(HN - 1);
        }
        if (dict_put<W>(nrow, s, r, row)) cnt[2 * R + r] = 1;
    }
    for (int i = t; i < nq * C; i += T) {
        const int r = i / C, row = i - r * C;
        const float4 y = conn_row(L.rconns + (size_t)(q0 + r) * C * 4 + (size_t)row * 4, vec);
        cattr[i] = make_float2(y.z, y.w);
        if (isnan(y.x)) continue;
        atomicAdd(&cnt[R + r], 1);
        if (isnan(y.y)) continue;  // can never match
        const unsigned a = key_bits(y.x), b = key_bits(y.y);
        const unsigned long long k = ((unsigned long long)a << 32) | b;
        unsigned s = dict_slot(a, b, sc);
        for (;;) {
            const unsigned long long prev = atomicCAS(ckey + s, EMPTY64, k);
            if (prev == EMPTY64 || prev == k) break;
            s = (s + 1) & (unsigned)(HC - 1);
        }
        if (dict_put<W>(crow, s, r, row)) cnt[2 * R + r] = 1;
    }
    __syncthreads();
    // a representative with a repeated key: one lane sets its rows again from
    // the last to the first, so that the first one stays
    bool repeats = false;
    for (int r = 0; r < nq; ++r) repeats |= cnt[2 * R + r] != 0;
    if (repeats) {  // uniform
        for (int r = wave; r < nq; r += waves) {
            if (cnt[2 * R + r] == 0 || lane != 0) continue;
            for (int row = N - 1; row >= 0; --row) {
                const float key = L.rnodes[(size_t)(q0 + r) * N * 5 + (size_t)row * 5];
                if (isnan(key)) continue;
                const unsigned k = key_bits(key);
                unsigned s = dict_slot(k, 0u, sn);
                while (nkey[s] != k) s = (s + 1) & (unsigned)(HN - 1);
                dict_set<W>(nrow, s, r, row);
            }
            for (int row = C - 1; row >= 0; --row) {
                const float *y = L.rconns + (size_t)(q0 + r) * C * 4 + (size_t)row * 4;
                if (isnan(y[0]) || isnan(y[1])) continue;
                const unsigned a = key_bits(y[0]), b = key_bits(y[1]);
                const unsigned long long k = ((unsigned long long)a << 32) | b;
                unsigned s = dict_slot(a, b, sc);
                while (ckey[s] != k) s = (s + 1) & (unsigned)(HC - 1);
                dict_set<W>(crow, s, r, row);
            }
        }
        __syncthreads();
    }
    // this lane's folded sum: its representative, kind and gene count
    const int my_r = (lane & 31) / D::LN;
    const bool conn_half = lane >= 32;
    const int my_b = cnt[(conn_half ? R : 0) + my_r];

    // ---- genomes, one per wave
    const unsigned g0 = (unsigned)part * (unsigned)L.per_block;
    const unsigned g1 = min((unsigned)L.P, g0 + (unsigned)L.per_block);
    for (unsigned g = g0 + (unsigned)wave; g < g1; g += (unsigned)waves) {
        const float *An = L.nodes + (size_t)g * N * 5;
        const float *Ac = L.conns + (size_t)g * C * 4;
        int na = 0, ca = 0;
        unsigned hun[R], huc[R];  // homologous genes and, 16 bits up, their unlike codes
        // opaque copies: what is derived from them for each representative is
        // computed where it is used (kept across genomes, it would spill)
        int Ns = N, Cs = C, lane_now = lane;
        asm volatile("" : "+s"(Ns), "+s"(Cs), "+v"(lane_now));
        float v[2 * R];  // attribute distances: nodes, connections
#pragma unroll
        for (int r = 0; r < R; ++r) hun[r] = huc[r] = 0u, v[r] = v[R + r] = 0.0f;
        for (int n0 = 0; n0 < N; n0 += WAVE) {
            const int row = n0 + lane;
            float x[5];
#pragma unroll
            for (int f = 0; f < 5; ++f)
                x[f] = row < N ? An[(size_t)row * 5 + f] : __builtin_nanf("");
            const bool have = !isnan(x[0]);
            na += __popcll(__ballot(have));
            u32x4 e = {~0u, ~0u, ~0u, ~0u};
            if (have) {
                const unsigned k = key_bits(x[0]);
                for (unsigned s = dict_slot(k, 0u, sn);; s = (s + 1) & (unsigned)(HN - 1)) {
                    const unsigned kk = nkey[s];
                    if (kk == k) {
                        e = ((const u32x4 *)nrow)[s];
                        break;
                    }
                    if (kk == ~0u) break;
                }
            }
#pragma unroll
            for (int r0 = 0; r0 < R; r0 += RB) {
                if (r0 >= nq) continue;  // uniform; places past nq are empty
#pragma unroll
                for (int r = r0; r < r0 + RB; ++r) {
                    const unsigned j = dict_row<W>(e, r);
                    const bool hit = j != D::NONE;
                    const unsigned long long hm = __ballot(hit);
                    float4 y = nattr[r * Ns + D::index(j, hit)];
                    keep(y.x), keep(y.y);
                    hun[r] += __popcll(hm) + ((__popcll(hm & __ballot(x[3] != y.z)) +
                                               __popcll(hm & __ballot(x[4] != y.w))) << 16);
                    const float d = fabsf(x[1] - y.x) + fabsf(x[2] - y.y);
                    v[r] += hit ? d : 0.0f;
                }
            }
        }
        constexpr int CR = 4;  // connection rows of a lane in one round
        for (int c0 = 0; c0 < C; c0 += CR * WAVE) {
            float en[CR], w[CR];
            unsigned k0[CR], k1[CR], s[CR];
            unsigned long long kk[CR];
            bool go[CR];
            u32x4 e[CR];
#pragma unroll
            for (int m = 0; m < CR; ++m) {
                const int row = c0 + m * WAVE + lane;
                const float nan = __builtin_nanf("");
                float4 x = make_float4(nan, nan, nan, nan);
                if (row < C) x = conn_row(Ac + (size_t)row * 4, vec);
                ca += __popcll(__ballot(!isnan(x.x)));
                en[m] = x.z, w[m] = x.w;
                go[m] = !isnan(x.x) && !isnan(x.y);
                k0[m] = key_bits(x.x), k1[m] = key_bits(x.y);
                s[m] = dict_slot(k0[m], k1[m], sc);
            }
            // first probes together, then the further ones row by row
#pragma unroll
            for (int m = 0; m < CR; ++m) kk[m] = ckey[s[m]];
#pragma unroll
            for (int m = 0; m < CR; ++m) {
                const unsigned long long k = ((unsigned long long)k0[m] << 32) | k1[m];
                while (go[m] && kk[m] != k && kk[m] != EMPTY64) {
                    s[m] = (s[m] + 1) & (unsigned)(HC - 1);
                    kk[m] = ckey[s[m]];
                }
                e[m] = u32x4{~0u, ~0u, ~0u, ~0u};
                if (go[m] && kk[m] == k) e[m] = ((const u32x4 *)crow)[s[m]];
            }
#pragma unroll
            for (int r0 = 0; r0 < R; r0 += RB) {
                if (r0 >= nq) continue;
#pragma unroll
                for (int r = r0; r < r0 + RB; ++r) {
                    const float2 *attr = cattr + r * Cs;
                    float2 y[CR];
                    bool hit[CR];
                    unsigned like = 0, unlike = 0;
#pragma unroll
                    for (int m = 0; m < CR; ++m) {
                        const unsigned j = dict_row<W>(e[m], r);
                        hit[m] = j != D::NONE;
                        like += __popcll(__ballot(hit[m]));
                        y[m] = attr[D::index(j, hit[m])];
                    }
#pragma unroll
                    for (int m = 0; m < CR; ++m) {
                        keep(y[m].y);
                        unlike += __popcll(__ballot(hit[m]) & __ballot(en[m] != y[m].x));
                        v[R + r] += hit[m] ? fabsf(w[m] - y[m].y) : 0.0f;
                    }
                    huc[r] += like + (unlike << 16);
                }
            }
        }
        // fold the 2 R sums over the lanes: value i ends in lanes LN i ..
#pragma unroll
        for (int i = 0; i < R; ++i) v[i] = fold32(v[i], v[i + R]);
#pragma unroll
        for (int i = 0; i < R / 2; ++i) v[i] = fold16(v[i], v[i + R / 2]);
#pragma unroll
        for (int i = 0; i < R / 4; ++i) v[i] = fold_dpp<DPP_ROR8>(v[i], v[i + R / 4], lane & 8);
        float sum = v[0];
        if constexpr (R >= 8) {
#pragma unroll
            for (int i = 0; i < R / 8; ++i)
                v[i] = fold_dpp<DPP_HALF_MIRROR>(v[i], v[i + R / 8], lane & 4);
            sum = R == 16 ? fold_dpp<DPP_SWAP2>(v[0], v[1], lane & 2) : dpp_sum<DPP_SWAP2>(v[0]);
        } else {
            sum = dpp_sum<DPP_SWAP2>(dpp_sum<DPP_HALF_MIRROR>(sum));
        }
        sum = dpp_sum<DPP_SWAP1>(sum);
        // the counts of this lane's sum
        unsigned hu = 0;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            hu = lane_now / D::LN == r ? hun[r] : hu;
            hu = lane_now / D::LN == R + r ? huc[r] : hu;
        }
        const int h = (int)(hu & 0xffffu);
        sum += (float)(hu >> 16);
        const int a = conn_half ? ca : na, m = max(a, my_b);
        const float d =
            m ? (L.cd * (float)(a + my_b - 2 * h) + L.ch * sum) / (float)m : 0.0f;
        const float other = __shfl_xor(d, 32);
        if (!conn_half && (lane & (D::LN - 1)) == 0 && my_r < nq)
            L.out[(size_t)g * L.Q + q0 + my_r] = d + other;
    }
}

// ---- distance by a table per representative, for shapes whose dictionary
// does not fit in LDS.  DIST_WAVES waves per workgroup, DIST_PER_WAVE
// genomes per wave: a representative's tables are built once for
// DIST_WAVES * DIST_PER_WAVE genomes.
constexpr int DIST_WAVES = 4, DIST_PER_WAVE = 2;
constexpr int DIST_GENOMES = DIST_WAVES * DIST_PER_WAVE;

__global__ __launch_bounds__(WAVE *DIST_WAVES) void distance_kernel(DistLaunch L) {
    extern __shared__ unsigned long long dsm[];
    const int N = L.N, C = L.C, HN = L.hn, HC = L.hc;
    unsigned long long *nk = dsm;            // node table: keys [HN]
    unsigned long long *ck = nk + HN;        // connection table: keys [HC]
    int *nr = (int *)(ck + HC);              // rows [HN]
    int *cr = nr + HN;                       // rows [HC]
    int *bcount = cr + HC;                   // B's node and connection genes
    const int t = (int)threadIdx.x, lane = t & (WAVE - 1), wave = t / WAVE;
    const int T = WAVE * DIST_WAVES;

    // this wave's genomes and their gene counts (once)
    long long gs[DIST_PER_WAVE];
    int na[DIST_PER_WAVE], ca[DIST_PER_WAVE];
#pragma unroll
    for (int i = 0; i < DIST_PER_WAVE; ++i) {
        gs[i] = (long long)blockIdx.x * DIST_GENOMES + wave * DIST_PER_WAVE + i;
        int a = 0, c = 0;
        if (gs[i] < L.P) {
            const float *An = L.nodes + (size_t)gs[i] * N * 5;
            const float *Ac = L.conns + (size_t)gs[i] * C * 4;
            for (int r = lane; r < N; r += WAVE) a += !isnan(An[(size_t)r * 5]);
            for (int r = lane; r < C; r += WAVE) c += !isnan(Ac[(size_t)r * 4]);
        }
        na[i] = wave_sum(a);
        ca[i] = wave_sum(c);
    }

    for (int q = 0; q < L.Q; ++q) {
        const float *Bn = L.rnodes + (size_t)q * N * 5;
        const float *Bc = L.rconns + (size_t)q * C * 4;
        for (int s = t; s < HN; s += T) nk[s] = EMPTY64, nr[s] = 0x7fffffff;
        for (int s = t; s < HC; s += T) ck[s] = EMPTY64, cr[s] = 0x7fffffff;
        if (t < 2) bcount[t] = 0;
        __syncthreads();
        int nb = 0, cb = 0;
        for (int r = t; r < N; r += T) {
            const float k = Bn[(size_t)r * 5];
            if (isnan(k)) continue;
            ++nb;
            insert(nk, nr, HN, key_bits(k), r);
        }
        for (int r = t; r < C; r += T) {
            const float ki = Bc[(size_t)r * 4], ko = Bc[(size_t)r * 4 + 1];
            if (isnan(ki)) continue;
            ++cb;
            if (isnan(ko)) continue;  // can never match
            insert(ck, cr, HC, ((unsigned long long)key_bits(ki) << 32) | key_bits(ko), r);
        }
        nb = wave_sum(nb);
        cb = wave_sum(cb);
        if (lane == 0) {
            atomicAdd(bcount, nb);
            atomicAdd(bcount + 1, cb);
        }
        __syncthreads();
        nb = bcount[0];
        cb = bcount[1];
#pragma unroll
        for (int i = 0; i < DIST_PER_WAVE; ++i) {
            if (gs[i] >= L.P) continue;  // uniform across the wave
            const float *An = L.nodes + (size_t)gs[i] * N * 5;
            const float *Ac = L.conns + (size_t)gs[i] * C * 4;
            int hn = 0, hc = 0;
            float sn = 0.0f, sc = 0.0f;
            for (int r = lane; r < N; r += WAVE) {
                const float *x = An + (size_t)r * 5;
                if (isnan(x[0])) continue;
                const int j = lookup(nk, nr, HN, key_bits(x[0]));
                if (j < 0) continue;
                const float *y = Bn + (size_t)j * 5;
                ++hn;
                sn += fabsf(x[1] - y[1]) + fabsf(x[2] - y[2]) + (float)(x[3] != y[3]) +
                      (float)(x[4] != y[4]);
            }
            for (int r = lane; r < C; r += WAVE) {
                const float *x = Ac + (size_t)r * 4;
                if (isnan(x[0]) || isnan(x[1])) continue;
                const int j = lookup(ck, cr, HC,
                                     ((unsigned long long)key_bits(x[0]) << 32) | key_bits(x[1]));
                if (j < 0) continue;
                const float *y = Bc + (size_t)j * 4;
                ++hc;
                sc += fabsf(x[3] - y[3]) + (float)(x[2] != y[2]);
            }
            hn = wave_total(hn);
            hc = wave_total(hc);
            sn = wave_total(sn);
            sc = wave_total(sc);
            if (lane == 0) {
                const int mn = max(na[i], nb), mc = max(ca[i], cb);
                const float dn =
                    mn ? (L.cd * (float)(na[i] + nb - 2 * hn) + L.ch * sn) / (float)mn : 0.0f;
                const float dc =
                    mc ? (L.cd * (float)(ca[i] + cb - 2 * hc) + L.ch * sc) / (float)mc : 0.0f;
                L.out[(size_t)gs[i] * L.Q + q] = dn + dc;
            }
        }
        __syncthreads();  // the tables are cleared for the next representative
    }
}

// Crossover (Section 3.2: the genetic operators become row and attribute
// writes of the tensors; the gene alignment is NEAT's): the child of
// (p1, p2) keeps p1's rows; a p1 gene homologous in p2 (same node key, or
// same (in, out) keys; partner = p2's first such row) takes the partner's
// non-key columns when its uniform number is below 0.5.  One wave per
// child, four children per workgroup while their tables fit in 64 KB of LDS
// (else one): p2's genes go into the wave's own LDS hash tables, every lane
// writes its p1 rows (connection rows as 16-byte loads and stores when the
// tensor is 16-byte aligned).
constexpr int CROSS_WAVES = 4;

__global__ __launch_bounds__(WAVE *CROSS_WAVES) void crossover_kernel(CrossLaunch L) {
    extern __shared__ unsigned long long dsm[];
    const int N = L.N, C = L.C, HN = L.hn, HC = L.hc;
    const int lane = (int)threadIdx.x & (WAVE - 1), wave = (int)threadIdx.x / WAVE;
    const int waves = (int)blockDim.x / WAVE;
    unsigned long long *nk = dsm + (size_t)wave * L.words;  // this wave's tables
    unsigned long long *ck = nk + HN;
    int *nr = (int *)(ck + HC);
    int *cr = nr + HN;
    const long long k = (long long)blockIdx.x * waves + wave;
    const bool live = k < L.Pc;
    int a = 0, b = 0;
    if (live) a = L.pairs[2 * k], b = L.pairs[2 * k + 1];
    // uniform across the wave; every wave reaches both barriers
    const bool ok = live && a >= 0 && a < L.P && b >= 0 && b < L.P;
    if (live && !ok) {
        for (int e = lane; e < N * 5; e += WAVE) L.cn[(size_t)k * N * 5 + e] = __builtin_nanf("");
        for (int e = lane; e < C * 4; e += WAVE) L.cc[(size_t)k * C * 4 + e] = __builtin_nanf("");
    }
    if (!ok) a = b = 0;
    const float *An = L.nodes + (size_t)a * N * 5, *Ac = L.conns + (size_t)a * C * 4;
    const float *Bn = L.nodes + (size_t)b * N * 5, *Bc = L.conns + (size_t)b * C * 4;
    if (ok) {
        for (int s = lane; s < HN; s += WAVE) nk[s] = EMPTY64, nr[s] = 0x7fffffff;
        for (int s = lane; s < HC; s += WAVE) ck[s] = EMPTY64, cr[s] = 0x7fffffff;
    }
    __syncthreads();
    if (ok) {
        for (int r = lane; r < N; r += WAVE) {
            const float key = Bn[(size_t)r * 5];
            if (!isnan(key)) insert(nk, nr, HN, key_bits(key), r);
        }
        for (int r = lane; r < C; r += WAVE) {
            const float ki = Bc[(size_t)r * 4], ko = Bc[(size_t)r * 4 + 1];
            if (!isnan(ki) && !isnan(ko))
                insert(ck, cr, HC, ((unsigned long long)key_bits(ki) << 32) | key_bits(ko), r);
        }
    }
    __syncthreads();
    if (!ok) return;
    float *On = L.cn + (size_t)k * N * 5, *Oc = L.cc + (size_t)k * C * 4;
    for (int r = lane; r < N; r += WAVE) {
        const float *x = An + (size_t)r * 5;
        const float *src = x;
        if (!isnan(x[0]) && L.rn[(size_t)k * N + r] < 0.5f) {
            const int j = lookup(nk, nr, HN, key_bits(x[0]));
            if (j >= 0) src = Bn + (size_t)j * 5;
        }
        float *o = On + (size_t)r * 5;
        o[0] = x[0];
#pragma unroll
        for (int c = 1; c < 5; ++c) o[c] = src[c];
    }
    for (int r = lane; r < C; r += WAVE) {
        const float *x = Ac + (size_t)r * 4;
        float4 v;
        if (L.vec) v = *reinterpret_cast<const float4 *>(x);
        else v = make_float4(x[0], x[1], x[2], x[3]);
        if (!isnan(v.x) && !isnan(v.y) && L.rc[(size_t)k * C + r] < 0.5f) {
            const int j = lookup(ck, cr, HC,
                                 ((unsigned long long)key_bits(v.x) << 32) | key_bits(v.y));
            if (j >= 0) {
                const float *y = Bc + (size_t)j * 4;
                if (L.vec) {
                    const float2 w = *reinterpret_cast<const float2 *>(y + 2);
                    v.z = w.x, v.w = w.y;
                } else {
                    v.z = y[2], v.w = y[3];
                }
            }
        }
        *reinterpret_cast<float4 *>(Oc + (size_t)r * 4) = v;
    }
}

// Tensorized edits (Section 3.2): additions at the first NaN row, NaN
// removals, attribute writes; a genome's edits in their order, genomes in
// parallel, one wave per genome.  The wave keeps one bit per row of its genome
// (the key is NaN), so an addition finds its row without touching memory.
// The rows that the edits write are found first, by scalar steps for the
// additions and removals; eight edits then go out per store, one after another
// where two of the wave's edits write one row.
//
// What bounds it: the latency of the wave's loads, so they are few and
// independent: the list is sorted by genome, and the probes that lead a search to
// where evenly spread edits would put the genome's run and the next one's, the 64
// whole records there and the rows' keys are requested together.  Every entry of
// `applied` is written in one pass.  The begins that the searches find never fall
// from one genome to the next, whatever the order of the list (a probe that is
// below one genome is below the next), so they cut it into one part per genome: a
// wave applies the records of its genome at its part's front and writes 0 for the
// rest (none when the list is sorted).  Records of genomes out of range, and
// others before the first part or past the last, belong to the wave whose share of
// the positions they lie in.
// Measured at 10,000 genomes of 50 node and 200 connection rows, 80,000 edits:
// 18.9 us, before 25.2 us and 4.8 us for clearing `applied` (one genome per
// workgroup, keys staged in LDS, edits one by one); of the 18.9 us, 6 are the
// records and the launch, 5.5 the 50 MB of key lines, the rest the edits.  One
// genome per workgroup: 23.8 against 22.9 with four, both with edits one by one.
// The same list shuffled: 23 us (15 ms while begins came from the windows, fell
// and rose with the list, and every record beside a run had its genome's run
// looked up).
constexpr int EDIT_WAVES = 4;      // genomes per workgroup
constexpr int EDIT_CHUNKS = 4;     // 64-row chunks of connection rows kept in registers

// The list as a binary tree down to blocks of 64 records: at a block of 2 x 64 x
// 2^k records a search goes right if the last record of the left half is below the
// key, and counts the records below the key in the block of 64 that it comes to.
// Every probe stays inside [0, n) whatever the order of the edits, and a larger key
// never gives a smaller index.
//
// The probes on the way to positions to[0] and to[1], one per lane, and the blocks
// of 64 there are requested before any of them is used: where evenly spread edits
// put this genome's run and the next one's, so both searches cost one latency and
// some twenty lines.  A search that leaves its way probes the 63 ends of six steps
// at once.  80,000 edits of 10,000 genomes behind a crossover: 53.7 us for both,
// 55.0 with steps of 64 parts (sixty-four lines each on the way).
struct EditTree {
    const EditRec *e;
    int n, height, lane;  // steps from the whole list to a block
    int to[2], block[2];  // genomes of the blocks there
    int probe;            // lane 32 w + k: the genome at step k (of 2^k blocks) of way w
    static __device__ __forceinline__ int start(int at) { return at & ~(WAVE - 1); }
    __device__ __forceinline__ int load(long long p) const {
        return p < n ? e[p].genome : 0x7fffffff;
    }
    __device__ __forceinline__ void request(int to0, int to1) {
        to[0] = to0, to[1] = to1;
        const long long t = lane < 32 ? to0 : to1;
        const int k = lane & 31;
        probe = 0x7fffffff;
        if (k < height) probe = load((t >> (7 + k) << (7 + k)) + (64ll << k) - 1);
    }
    // first index whose genome is >= key
    __device__ __forceinline__ int search(int w, int key) const {
        const unsigned right = (unsigned)(__ballot(probe < key) >> (32 * w));
        const unsigned off = right ^ (unsigned)(to[w] / WAVE);
        if (!off) return start(to[w]) + __popcll(__ballot(block[w] < key));
        int k = 31 - __clz((int)off);
        long long lo = (long long)to[w] >> (7 + k) << (7 + k);
        lo += (long long)((right >> k) & 1u) << (6 + k);
        while (k > 0) {
            const int steps = min(k, 6);
            k -= steps;
            const unsigned long long below =
                __ballot(lane + 1 < 1 << steps &&
                         load(lo + ((long long)(lane + 1) << (6 + k)) - 1) < key);
            int s = 0;
            for (int b = steps - 1; b >= 0; --b)
                s += (int)((below >> (s + (1 << b) - 1)) & 1ull) << b;
            lo += (long long)s << (6 + k);
        }
        return (int)lo + __popcll(__ballot(load(lo + lane) < key));
    }
};

__device__ __forceinline__ int lane_int(int v, int i) { return __builtin_amdgcn_readlane(v, i); }
// One bit per row of a tensor whose key is NaN, 64 rows per chunk: in scalar
// registers (CH chunks), or in LDS (CH = 0).
template <int CH>
struct NanRows {
    unsigned long long m[CH > 0 ? CH : 1] = {};
    unsigned long long *lds = nullptr;
    int chunks = 0;
    __device__ __forceinline__ void load(const float *t, int w, int rows, int lane) {
        chunks = (rows + WAVE - 1) / WAVE;
        if constexpr (CH > 0) {
#pragma unroll
            for (int k = 0; k < CH; ++k) {
                const int r = k * WAVE + lane;
                m[k] = __ballot(r < rows && isnan(t[(size_t)min(r, rows - 1) * w]));
            }
        } else {
            for (int k = 0; k < chunks; ++k) {
                const int r = k * WAVE + lane;
                const unsigned long long b = __ballot(r < rows && isnan(t[(size_t)min(r, rows - 1) * w]));
                if (lane == 0) lds[k] = b;
            }
            sync();
        }
    }
    // lane 0's LDS writes before the other lanes' reads
    static __device__ __forceinline__ void sync() {
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
        __builtin_amdgcn_wave_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
    }
    // first row with the bit, or -1
    __device__ __forceinline__ int first() const {
        if constexpr (CH > 0) {
            int row = -1;
#pragma unroll
            for (int k = CH - 1; k >= 0; --k)
                if (m[k]) row = k * WAVE + __ffsll((long long)m[k]) - 1;
            return row;
        } else {
            for (int k = 0; k < chunks; ++k) {
                const unsigned long long b = lds[k];
                if (b) return k * WAVE + __ffsll((long long)b) - 1;
            }
            return -1;
        }
    }
    __device__ __forceinline__ void set(int row, bool nan, int lane) {
        const unsigned long long bit = 1ull << (row & (WAVE - 1));
        if constexpr (CH > 0) {
#pragma unroll
            for (int k = 0; k < CH; ++k) {  // selects, not an indexed array
                const unsigned long long s = row / WAVE == k ? bit : 0ull;
                m[k] = nan ? m[k] | s : m[k] & ~s;
            }
        } else {
            const unsigned long long b = lds[row / WAVE];
            if (lane == 0) lds[row / WAVE] = nan ? b | bit : b & ~bit;
            sync();
        }
    }
};

// A record in the lanes (lane l: one record's words).
struct EditLanes {
    int genome, op, row, column;
    float v[5];
    __device__ __forceinline__ void load(const EditRec *e, int at, int n, int lane) {
        genome = -1;
        if (at + lane < n) {
            const EditRec r = e[at + lane];
            genome = r.genome, op = r.op, row = r.row, column = r.column;
#pragma unroll
            for (int f = 0; f < 5; ++f) v[f] = r.v[f];
        }
    }
};

// CN, CC: chunks of node and connection rows in registers (0: in LDS)
template <int CN, int CC>
__global__ __launch_bounds__(WAVE *EDIT_WAVES) void edit_kernel(EditLaunch L) {
    extern __shared__ unsigned long long edit_lds[];
    const int lane = (int)threadIdx.x & (WAVE - 1);
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x / WAVE);
    const int g = (int)blockIdx.x * EDIT_WAVES + wave;
    if (g >= L.P) return;
    const int N = L.N, C = L.C, n = L.n;
    float *gn = L.nodes + (size_t)g * N * 5, *gc = L.conns + (size_t)g * C * 4;
    NanRows<CN> nn;
    NanRows<CC> nc;
    nn.lds = edit_lds + (size_t)wave * L.mask_words;
    nc.lds = nn.lds + (N + WAVE - 1) / WAVE;
    EditTree tree;
    tree.e = L.edits, tree.n = n, tree.height = L.height, tree.lane = lane;
    EditLanes rec;
    int at = -WAVE;  // the position of lane 0's record
    const int front = L.edits[0].genome, back = L.edits[n - 1].genome;
    // records and the rows' keys, requested beside the search where most
    // genomes have edits
    tree.request((int)((long long)g * n / L.P), min((int)((long long)(g + 1) * n / L.P), n - 1));
    const int here = EditTree::start(tree.to[0]), next = EditTree::start(tree.to[1]);
    if (L.prefetch) {
        at = here;
        rec.load(L.edits, at, n, lane);
        tree.block[0] = at + lane < n ? rec.genome : 0x7fffffff;
        tree.block[1] = next == here ? tree.block[0] : tree.load((long long)next + lane);
        nn.load(gn, 5, N, lane);
        if (C > 0) nc.load(gc, 4, C, lane);
    } else {
        tree.block[0] = tree.load((long long)here + lane);
        tree.block[1] = next == here ? tree.block[0] : tree.load((long long)next + lane);
    }
    // this genome's part [lo, lo1) of the list, and all genomes' [lo0, loP): whole
    // unless its ends are out of range
    int lo = tree.search(0, g), lo1 = tree.search(1, g + 1), lo0 = 0, loP = n;
    if (front < 0) lo0 = tree.search(0, 0);
    if (back >= L.P) loP = tree.search(1, L.P);
    if (g == 0) lo = lo0;
    if (g == L.P - 1) lo1 = loP;
    int e = lo;  // the genome's run continues at e
    bool masks = L.prefetch != 0;
    for (;;) {
        if (e >= lo1) break;
        if (e < at || e >= at + WAVE) {
            at = e;
            rec.load(L.edits, at, n, lane);
        }
        // records e .. e + cnt - 1, in lanes i0 ..
        const int i0 = e - at;
        const unsigned long long same = __ballot(at + lane < n && rec.genome == g) >> i0;
        const int run = ~same ? __ffsll((long long)~same) - 1 : WAVE;
        const int cnt = min(run, lo1 - e);
        if (cnt == 0) break;
        if (!masks) {
            nn.load(gn, 5, N, lane);
            if (C > 0) nc.load(gc, 4, C, lane);
            masks = true;
        }
        // which rows the edits write, -1 where one does not apply: one lane
        // per edit, then the additions and removals in their order
        const bool mine = lane >= i0 && lane < i0 + cnt;
        const bool add = mine && (rec.op == 0 || rec.op == 2);
        const bool rem = mine && (rec.op == 1 || rec.op == 3);
        const bool attr = mine && (rec.op == 4 || rec.op == 5);
        const bool node = rec.op == 0 || rec.op == 1 || rec.op == 4;
        const bool there = rec.row >= 0 && rec.row < (node ? N : C);
        const bool column = node ? rec.column >= 1 && rec.column <= 4
                                 : rec.column >= 2 && rec.column <= 3;
        int row = there && (rem || (attr && column)) ? rec.row : -1;
        const unsigned long long adds = __ballot(add), nodes = __ballot(node);
        const unsigned long long nan_after = __ballot(rem || isnan(rec.v[0]));
        unsigned long long todo = adds | __ballot(rem && there);
        while (todo) {
            const int i = __ffsll((long long)todo) - 1;
            todo &= todo - 1;
            const bool nd = (nodes >> i) & 1ull, nan = (nan_after >> i) & 1ull;
            int r = lane_int(row, i);
            if ((adds >> i) & 1ull) {
                r = nd ? nn.first() : nc.first();
                if (r < 0) continue;
                row = lane == i ? r : row;
            }
            if (nd) nn.set(r, nan, lane);
            else nc.set(r, nan, lane);
        }
        if (mine) L.applied[at + lane] = row >= 0;
        // do two of them write one row
        const int id = node ? row : N + row;
        const unsigned long long live = __ballot(row >= 0);
        unsigned long long twice = 0;
        for (unsigned long long m = live; m; m &= m - 1) {
            const unsigned long long eq = __ballot(id == lane_int(id, __ffsll((long long)m) - 1));
            twice |= eq & m & (m - 1);
        }
        // eight edits per store, eight lanes each: together where their rows
        // differ, else one after another
        for (int k = i0; k < i0 + cnt; k += 8) {
            const int j = (k + lane / 8) & (WAVE - 1), col = lane % 8;
            const int rj = __shfl(row, j), what = __shfl(add ? 0 : rem ? 1 : 2 + rec.column, j);
            float v = __shfl(rec.v[0], j);
            const float v1 = __shfl(rec.v[1], j), v2 = __shfl(rec.v[2], j);
            const float v3 = __shfl(rec.v[3], j), v4 = __shfl(rec.v[4], j);
            const bool nd = (nodes >> j) & 1ull;
            const int w = nd ? 5 : 4;
            if (what == 0) v = col == 0 ? v : col == 1 ? v1 : col == 2 ? v2 : col == 3 ? v3 : v4;
            if (what == 1) v = __builtin_nanf("");
            const bool put = k + lane / 8 < i0 + cnt && rj >= 0 && col < w && (what < 2 || col == what - 2);
            float *o = (nd ? gn : gc) + (size_t)max(rj, 0) * w + col;
            if (!twice) {
                if (put) *o = v;
            } else {
                for (int s = 0; s < 8; ++s) {
                    if (put && lane / 8 == s) *o = v;
                    nn.sync();
                }
            }
        }
        e += cnt;
        if (e < at + WAVE) break;  // the run ended inside the lanes
    }
    // what is left of its part, and its share of the positions before the first
    // part and past the last
    for (int i = e + lane; i < lo1; i += WAVE) L.applied[i] = 0;
    if (lo0 > 0 || loP < n) {
        const int s0 = (int)((long long)g * n / L.P), s1 = (int)((long long)(g + 1) * n / L.P);
        for (int i = s0 + lane; i < s1; i += WAVE)
            if (i < lo0 || i >= loP) L.applied[i] = 0;
    }
}

// No genomes: nothing can apply.
__global__ __launch_bounds__(256) void edit_clear_kernel(int32_t *applied, int n) {
    const long long i = (long long)blockIdx.x * 256 + threadIdx.x;
    if (i < n) applied[i] = 0;
}

int pow2_at_least(int x) {
    int h = 64;
    while (h < x) h <<= 1;
    return h;
}

}  // namespace

// the two hash tables and two counters
size_t gene_tables_lds_bytes(int N, int C) {
    const int hn = pow2_at_least(2 * N), hc = pow2_at_least(2 * C);
    return (size_t)(hn + hc) * (sizeof(unsigned long long) + sizeof(int)) + 2 * sizeof(int);
}

hipError_t crossover_launch(CrossLaunch L, hipStream_t stream) {
    L.hn = pow2_at_least(2 * L.N);
    L.hc = pow2_at_least(2 * L.C);
    L.words = L.hn + L.hc + (L.hn + L.hc) / 2;  // keys, then rows (hn + hc even)
    L.vec = ((uintptr_t)L.conns % 16) == 0;
    if (L.Pc == 0) return hipSuccess;
    // four children per workgroup while their tables stay small (≤ 64 KB)
    const size_t wave_bytes = sizeof(unsigned long long) * (size_t)L.words;
    const int waves = 4 * wave_bytes <= 65536 ? CROSS_WAVES : 1;
    hipLaunchKernelGGL(crossover_kernel, dim3((unsigned)((L.Pc + waves - 1) / waves)),
                       dim3(WAVE * waves), waves * wave_bytes, stream, L);
    return hipGetLastError();
}

hipError_t edit_launch(EditLaunch L, hipStream_t stream) {
    if (L.n == 0) return hipSuccess;
    if (L.P == 0) {
        hipLaunchKernelGGL(edit_clear_kernel, dim3((unsigned)(((long long)L.n + 255) / 256)),
                           dim3(256), 0, stream, L.applied, L.n);
        return hipGetLastError();
    }
    L.prefetch = L.n >= L.P;
    L.height = 0;
    while ((long long)L.n > (long long)WAVE << L.height) ++L.height;
    const dim3 grid((unsigned)(((long long)L.P + EDIT_WAVES - 1) / EDIT_WAVES));
    const dim3 block(WAVE * EDIT_WAVES);
    if (L.N <= WAVE && L.C <= WAVE * EDIT_CHUNKS) {
        hipLaunchKernelGGL((edit_kernel<1, EDIT_CHUNKS>), grid, block, 0, stream, L);
    } else {
        L.mask_words = (L.N + WAVE - 1) / WAVE + (L.C + WAVE - 1) / WAVE;
        hipLaunchKernelGGL((edit_kernel<0, 0>), grid, block,
                           sizeof(unsigned long long) * EDIT_WAVES * (size_t)L.mask_words, stream,
                           L);
    }
    return hipGetLastError();
}

// The dictionary's shape for groups of rq representatives, and its LDS
// bytes: tables a quarter larger than the keys they can have to hold (rows
// that are absent and keys that representatives share leave them emptier).
static size_t dict_shape(int N, int C, int rq, int row_bytes, int *hn, int *hc) {
    const int rb = rq <= 4 ? 1 : 4, ra = (rq + rb - 1) / rb * rb;
    *hn = pow2_at_least((5 * rq * N + 3) / 4);
    *hc = pow2_at_least((5 * rq * C + 3) / 4);
    return (size_t)*hc * 24 + (size_t)*hn * 20 + (size_t)ra * ((size_t)16 * N + (size_t)8 * C) +
           3 * sizeof(int) * (16 / row_bytes) + (row_bytes == 1 ? 256 * sizeof(float4) : 0);
}

static int log2_of(int x) {
    int l = 0;
    while ((1 << l) < x) ++l;
    return l;
}

hipError_t distance_launch(DistLaunch L, size_t max_lds, hipStream_t stream) {
    if (L.P == 0 || L.Q == 0) return hipSuccess;
    // Rows are numbered in one byte (16 representatives per group) while
    // every row number is below 255, else in two (8).  A group takes as many
    // representatives as their dictionary fits in LDS (none: the kernel with a
    // table per representative).  With few genomes it takes fewer, so that
    // the groups reach every CU (P = 100, Q = 64: 10.5 us in groups of 16,
    // 9.5 us in groups of 4).  Groups of up to 4 have a kernel that folds 8
    // sums instead of 32 (P = 10000, Q = 1: 24.5 us with 32, 16.1 us with 8).
    const int row_bytes = std::max(L.N, L.C) <= 255 ? 1 : 2;
    int rq = std::min(L.Q, 16 / row_bytes);
    while (rq > 0 && dict_shape(L.N, L.C, rq, row_bytes, &L.hn, &L.hc) > max_lds) --rq;
    if (rq == 0) {
        L.hn = pow2_at_least(2 * L.N);
        L.hc = pow2_at_least(2 * L.C);
        const dim3 grid((unsigned)(((long long)L.P + DIST_GENOMES - 1) / DIST_GENOMES));
        hipLaunchKernelGGL(distance_kernel, grid, dim3(WAVE * DIST_WAVES),
                           gene_tables_lds_bytes(L.N, L.C), stream, L);
        return hipGetLastError();
    }
    constexpr int CUS = 256;
    auto parts = [](long long x, int by) { return (x + by - 1) / by; };
    while (rq > 4 && parts(L.Q, rq) * parts(L.P, 16) < CUS) rq = (rq + 1) / 2;
    const int groups = (int)parts(L.Q, rq);
    L.rq = (int)parts(L.Q, groups);
    const size_t lds = dict_shape(L.N, L.C, L.rq, row_bytes, &L.hn, &L.hc);
    L.hn_log2 = log2_of(L.hn), L.hc_log2 = log2_of(L.hc);
    L.vec = ((uintptr_t)L.conns % 16) == 0 && ((uintptr_t)L.rconns % 16) == 0;
    // one workgroup of 16 waves per CU, or two of eight (four for the small
    // groups, whose kernels hold fewer registers)
    const bool small = L.rq <= 4;
    const int waves = 2 * lds > max_lds ? 16 : 8;
    const int per_cu = waves == 16 ? 1 : (int)std::min<size_t>(small ? 4 : 2, max_lds / lds);
    const int target = std::max(1, CUS * per_cu / groups);  // workgroups per group
    const long long least = ((long long)L.P + target - 1) / target;
    L.per_block = (int)std::min<long long>((least + waves - 1) / waves * waves, 1 << 30);
    L.blocks_per_group = (int)(((long long)L.P + L.per_block - 1) / L.per_block);
    // a launch holds fewer than 2^32 threads
    const int most = (int)std::min<long long>(groups, 0xffffffffll / (WAVE * waves) / L.blocks_per_group);
    for (int first = 0; first < groups; first += most) {
        L.q_first = first * L.rq;
        const dim3 grid((unsigned)std::min(most, groups - first) * (unsigned)L.blocks_per_group);
        const dim3 block((unsigned)(WAVE * waves));
#define NEAT_DICT(W, R, RB)                                                                 \
    hipLaunchKernelGGL((distance_dict_kernel<W, R, RB>), grid, block, lds, stream, L)
        if (row_bytes == 1) {
            if (small) NEAT_DICT(1, 4, 1);
            else NEAT_DICT(1, 16, 4);
        } else {
            if (small) NEAT_DICT(2, 4, 1);
            else NEAT_DICT(2, 8, 4);
        }
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
#undef NEAT_DICT
    return hipSuccess;
}

}  // namespace neat
