// Block-sparse flash attention on the matrix cores of gfx950 (grouped, dense, joint), bf16 or half,
// head_dim 128 or 64.  The kernel template; its instantiations are compiled in attn_mfma_*.hip.
//
// Computes Sec. 3.1 Eq. 1 restricted to the attendable KV groups of Sec. 3.2.  Because all
// queries of a group share one KV list, every (query tile, KV tile) product is a full dense
// tile: no masking inside tiles, only a list walk around them.
//
// Work split: one workgroup = NWAVES wavefronts = 32*NWAVES queries of ONE group; each wave
// owns 32 queries.  K/V of the listed groups are gathered from row-major token order (a group's
// rows are runs of g_last contiguous tokens) straight into LDS with global_load_lds_dwordx4,
// in tiles of 64 tokens, double buffered; no registers are staged and nothing is permuted in
// HBM.
//
// MFMA formulation (v_mfma_f32_32x32x16_bf16, 64-lane waves), "transposed" so that softmax
// statistics never cross lanes except once between the two halves of the wave:
//   S^T[key, query] = K_tile (A operand, rows = keys, from LDS) x Q^T (B operand, registers)
//       -> lane (query = lane % 32, half = lane / 32) holds 16 keys of that query per 32-key
//          block: key = 8*(r/4) + 4*half + r%4 for accumulator register r.
//   O^T[dim, query] += V^T_tile (A operand, rows = head dims) x P^T (B operand)
//       -> P^T is exactly the S^T accumulator layout if the contraction index of the second
//          product is enumerated in that same (r, half) order, so P never leaves the lane's
//          registers; the matching V^T fragments come out of the row-major V tile through the
//          LDS transpose read ds_read_b64_tr_b16.
// Softmax runs in base 2 with scale*log2(e) folded into one FMA per score; the reference
// maximum, the running sum and the O accumulator stay fp32; P is rounded to bf16 (RNE) for the
// second product; the row sum is taken over the unrounded fp32 weights with plain adds.
//
// Schedule: one barrier per KV tile, and between two barriers ONE instruction stream per wave in
// which the work is software-pipelined by 32-key blocks (half a tile): while the matrix pipe forms
// the scores of block h, the vector ALU turns the scores of block h-1 into weights and the matrix
// pipe adds block h-2 to O.  The three stages of a half step do not depend on each other, so every
// MFMA is followed by its share of the vector work: a 32x32x16 MFMA holds the matrix pipe for 32
// cycles but the issue port for 8, and 24 cycles of other vector instructions fit behind it.
// (Measured on this chip: v_dot2c_f32_bf16 is not among them - it waits for the matrix pipe and
// holds it for 16 cycles - which is why the row sum uses v_add_f32.)
#pragma once
#include <type_traits>

#include "grat_common.h"
#include "tile_order.h"

namespace grat {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) _Float16 f16x8;
typedef __attribute__((ext_vector_type(2))) _Float16 f16x2;
typedef __attribute__((ext_vector_type(8))) short frag8;   // 8 sixteen-bit elements of either type
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(16))) float f32x16;

#define LDS_PTR(T) __attribute__((address_space(3))) T*

// KV tokens per LDS tile (template argument BN of the kernel): 64, or 32 as an option for the 2-wave
// workgroups (64 queries) of small groups, whose four tiles then take 32 KiB so that four workgroups
// (two waves per SIMD) share a compute unit instead of two - worth it for short lists, where a
// workgroup's fixed cost weighs most; long lists run better on 64-key tiles (half as many barriers,
// tile look-ups and load instructions per key).
constexpr int kFragAhead = 2;         // an MFMA's LDS fragment is read this many MFMAs ahead of it

// LDS tiles are unpadded [64 rows][D / 8 chunks of 16 B]; the chunk index is XOR-swizzled per row so
// that the fragment reads are bank-conflict free.  K is read with ds_read_b128 by lanes holding
// consecutive rows: 16 of them have to fall on the 16 chunk positions of a 256-byte line (64 banks), which
// is one row of 128 head dims (spread rows over all 16 positions and keep the two dim-halves of a row
// apart) or two rows of 64.  V is read with the 8-byte transpose read by 4 rows x 4 chunks at a time:
// each of 4 consecutive rows goes to a different group of 4 chunks of the line.
template <int D>
__device__ __forceinline__ int k_swizzle(int row) { return D == 128 ? ((row & 7) << 1) | ((row >> 3) & 1) : (row >> 1) & 7; }
template <int D>
__device__ __forceinline__ int v_swizzle(int row) { return D == 128 ? (row & 3) << 2 : (row & 2) << 1; }

// What depends on the 16-bit element type (F16 = false: bfloat16, true: IEEE half).  Fragments
// travel as type-neutral frag8 and are reinterpreted at the MFMA.
template <bool F16>
struct Elem {
    // a lane's block row sum (16 weights) beyond this forces a new reference maximum: every single
    // weight then stays inside the type's range (half: 65504) with its full relative precision
    static constexpr float kSumLimit = F16 ? 0x1p+15f : 0x1p+40f;
    static __device__ __forceinline__ f32x16 mfma(frag8 a, frag8 b, f32x16 c) {
        if constexpr (F16)
            return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8, a), __builtin_bit_cast(f16x8, b), c, 0, 0, 0);
        else
            return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
    }
    // two fp32 values rounded to nearest-even and packed (lo in the low half)
    static __device__ __forceinline__ uint32_t pack(float lo, float hi) {
        const f32x2 v = {lo, hi};
        if constexpr (F16) return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, f16x2));
        else return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
    }
};

// Exchange between the two lanes that hold the same query (lane and lane ^ 32) with one
// v_permlane32_swap.  The two results are copied to scalars before they are reinterpreted:
// a bit cast applied directly to a vector element reads element 0 with this compiler.
__device__ __forceinline__ void swap_halves(float x, float& lower, float& upper) {
    const uint32_t a = __builtin_bit_cast(uint32_t, x);
    const auto r = __builtin_amdgcn_permlane32_swap(a, a, false, false);
    const uint32_t r0 = r[0], r1 = r[1];
    lower = __builtin_bit_cast(float, r0);   // value held by the lane with the same query, half 0
    upper = __builtin_bit_cast(float, r1);   // ... half 1
}
__device__ __forceinline__ float max_across_halves(float x) {
    float lo, hi;
    swap_halves(x, lo, hi);
    return fmaxf(lo, hi);
}
__device__ __forceinline__ float sum_across_halves(float x) {
    float lo, hi;
    swap_halves(x, lo, hi);
    return lo + hi;
}

// (MODE: see AttnMode in grat_common.h)

// Box coordinates of an intra-group token, packed for the border tests of kRagged: 12 + 10 + 10 bits.
__device__ __forceinline__ uint32_t pack_coord(int c0, int c1, int c2) {
    return (uint32_t)c0 << 20 | (uint32_t)c1 << 10 | (uint32_t)c2;
}
// every coordinate of c at most the matching one of lim (lim = largest coordinates inside the grid)
__device__ __forceinline__ bool coord_inside(uint32_t c, uint32_t lim) {
    return (c >> 20) <= (lim >> 20) && ((c >> 10) & 1023u) <= ((lim >> 10) & 1023u) && (c & 1023u) <= (lim & 1023u);
}

// D = head_dim, 128 or 64.
//
// One query tile: tile t_in_head of its kind in (batch, head) bh.  DENSE: it is a tile of consecutive
// query rows that walks the whole sequence (always in kDense, the prompt rows in kJoint), else a
// tile of one query group.  k_tiles / v_tiles: the workgroup's tile buffers in LDS, two for K and two for V of every
// team (of several teams: V's right behind K's).
//
// TEAMS > 1 (small launches): the workgroup is that many teams of NWAVES waves; every team owns all its queries
// and walks the KV tiles team, team + TEAMS, ... in buffers of its own, and the results are merged through LDS at
// the end.
template <int NWAVES, int BN, int MODE, bool F16, int D, bool DENSE, int TEAMS>
__device__ __forceinline__ void attn_tile(const AttnParams& p, const int bh, const int t_in_head,
                                          uint8_t (*k_tiles)[BN * D * 2], uint8_t (*v_tiles)[BN * D * 2],
                                          const int gamma_fixed = -1) {
    static_assert(TEAMS == 1 || MODE != kRagged, "tiles are dealt to teams by their number, boxes all of one size");
    static_assert(BN == 64 || (BN == 32 && NWAVES == 2), "64-key tiles, or 32-key tiles for 2-wave workgroups");
    constexpr int kBN = BN;
    constexpr int kRowBytes = D * 2;          // of a token
    constexpr int kRowChunks = kRowBytes / 16;
    constexpr int kTileBytes = kBN * kRowBytes;
    static_assert(D == 128 || D == 64, "head_dim 128 or 64");
    using E = Elem<F16>;
    constexpr int NT = NWAVES * TEAMS * 64;
    constexpr int BM = NWAVES * 32;
    constexpr int LPW = kTileBytes / (1024 * NWAVES);   // 1-KiB direct loads (4 or 8 token rows) per wave per tile
    constexpr bool dense = DENSE;

    extern __shared__ int32_t s_dyn[];   // [n_g] row offsets inside a group, then [max_kv] group origins (kRagged: and the two tables below)
    // Teams have one copy of the walk over a whole sequence, from its last tile to the first.  64-key tiles (two teams): a tile
    // cut short comes first, and only the first two steps look for it (head_dim 128, 8 heads, 2 049 tokens 31.1 -> 29.7 us).
    // 32-key tiles (four teams): every step looks, the order is of no use to it; what helps is that there is one copy, since two
    // spilled 27 registers (1 024 tokens 16.4 -> 13.8).  Undivided walks gain nothing or lose backwards where no tile is cut short
    // (head_dim 128: 8 191 tokens 660 | 664, 4 352 tokens 215.5 | 219.8; head_dim 64: 8 191 tokens 425 | 419, 8 192 tokens 415 | 418).
    constexpr bool kBackwards = DENSE && TEAMS > 1;
    constexpr bool kLists = MODE == kGrouped || MODE == kRagged;   // every KV tile comes from a listed group
    constexpr bool kLeadThenLists = MODE == kJoint && !DENSE;      // prompt tiles first, then the listed groups

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_in_wg = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int team = TEAMS == 1 ? 0 : wave_in_wg / NWAVES;
    const int wave = TEAMS == 1 ? wave_in_wg : wave_in_wg % NWAVES;   // in its team
    uint8_t (*const sK)[kTileBytes] = k_tiles + 2 * team;
    uint8_t (*const sV)[kTileBytes] = v_tiles + 2 * team;
    const int qcol = lane & 31;   // query within the wave's 32
    const int half = lane >> 5;

    const Geometry& geo = p.geo;
    // (index decompositions go through host-prepared multipliers: see fastdiv.h)
    const int b_idx = (int)fdiv((uint32_t)bh, p.fd_heads), h_idx = bh - b_idx * p.heads;
    const int64_t head_off = (int64_t)b_idx * p.stride_b + (int64_t)h_idx * p.stride_h;
    const uint16_t* Qh = (const uint16_t*)p.Q + head_off;
    const uint16_t* Kh = (const uint16_t*)p.K + head_off;
    const uint16_t* Vh = (const uint16_t*)p.V + head_off;
    uint16_t* Oh = (uint16_t*)p.O + (int64_t)b_idx * p.o_stride_b + (int64_t)h_idx * p.o_stride_h;
    const int stride_n = p.stride_n;

    // s_rowbytes[t]: byte offset (row * stride_n * 2) of intra-group token t relative to its group's
    // first token - a group spans less than 4 GiB; s_origin[i]: ROW of the first token of the i-th
    // listed KV group - wave-uniform, turned into a 64-bit address in scalar registers, so the
    // sequence itself may be as large as memory (packed [B][N][3][H][d] layouts of long sequences)
    uint32_t* s_rowbytes = (uint32_t*)s_dyn;
    // kRagged: s_coord[t] = box coordinates of intra-group token t (behind s_rowbytes, so that it
    // stays 16-byte aligned), s_limit[i] = largest box coordinates of listed group i that are still
    // inside the grid (both packed)
    uint32_t* s_coord = s_rowbytes + geo.group_tokens;
    uint32_t* s_origin = (uint32_t*)s_dyn + (MODE == kDense ? 0 : (MODE == kRagged ? 2 : 1) * geo.group_tokens);
    uint32_t* s_limit = s_origin + p.max_kv;
    uint32_t q_limit = 0;   // kRagged: the same limit for the query group
    // kRagged: index of the last token of a box that is inside the grid, and the tiles of the box up to it
    // (later ones would only add weights of 0: 90x160 tokens in 16x16 groups, half, 2 x 24 heads: 3 % of the time
    // for 2 of 64 tiles a column of groups)
    auto last_inside = [&](uint32_t lim) { return (int)(((lim >> 20) * geo.g[1] + ((lim >> 10) & 1023u)) * geo.g[2] + (lim & 1023u)); };
    auto box_tiles = [&](uint32_t lim) { return last_inside(lim) / kBN + 1; };
    const uint32_t row_pitch = (uint32_t)stride_n * 2u;   // bytes between consecutive tokens
    const uint32_t full_box = pack_coord(geo.g[0] - 1, geo.g[1] - 1, geo.g[2] - 1);
    bool clipped = false;   // kRagged: this workgroup's query group or one it attends is cut by the border
    bool active = true;     // kRagged: one of this wave's queries is inside the grid

    int n_tiles;        // KV tiles to walk
    int tiles_per_group = 1;
    int n_listed = 1;   // grouped tiles: entries in s_origin
    int n_lead = 0;     // grouped tile of a joint sequence: leading KV tiles that hold the prompt tokens
    int mask_tile = -1, mask_valid = kBN;   // the one KV tile with fewer than kBN valid keys, if any
    // query rows of this wave: row i of its 32 is row q_first + i of the dense rows, resp. token
    // q_first + i of its group, whose first token is row q_base of the head
    uint32_t q_base = 0;
    int q_first;
    frag8 qf[D / 16];   // Q^T fragments (B operand): this lane's query, dims 16*ks + 8*half .. +7
    if (dense) {
        n_tiles = (p.n_tokens + kBN - 1) / kBN;
        if (p.n_tokens % kBN) { mask_tile = kBackwards ? 0 : n_tiles - 1; mask_valid = p.n_tokens % kBN; }
        q_first = t_in_head * BM + wave * 32;
    } else {
        int qt, gamma;
        if (gamma_fixed >= 0) {   // the caller has picked the group: t_in_head is the tile inside it
            gamma = gamma_fixed;
            qt = t_in_head;
        } else {
            const uint32_t u_group = fdiv((uint32_t)t_in_head, p.fd_q_tiles);
            qt = t_in_head - (int)u_group * p.q_tiles;
            gamma = strip_order_group(u_group, geo.G[0] * geo.G[1], geo.G[2], p);
        }
        const int n_g = geo.group_tokens;
        const int T12 = geo.T[1] * geo.T[2];
        // row of the first token of group gid, relative to the first grid row
        auto group_origin = [&](uint32_t gid, int& p0, int& p1, int& p2) {
            uint32_t v, r2, q0, r1;
            fdivmod(gid, p.fd_G2, v, r2);
            fdivmod(v, p.fd_G1, q0, r1);
            p0 = (int)q0; p1 = (int)r1; p2 = (int)r2;
            return p0 * geo.g[0] * T12 + p1 * geo.g[1] * geo.T[2] + p2 * geo.g[2];
        };
        // box coordinates of token t of a group
        auto token_coord = [&](uint32_t t, int& c0, int& c1, int& c2) {
            uint32_t v, r2, q0, r1;
            fdivmod(t, p.fd_g2, v, r2);
            fdivmod(v, p.fd_g1, q0, r1);
            c0 = (int)q0; c1 = (int)r1; c2 = (int)r2;
        };
        const uint32_t grid_base = MODE == kJoint ? (uint32_t)p.grid_row0 : 0u;   // first grid row
        auto box_limit = [&](int gid) {   // largest box coordinates of group gid inside the grid
            int p0, p1, p2;
            group_origin((uint32_t)gid, p0, p1, p2);
            return pack_coord(min(geo.g[0], geo.T[0] - p0 * geo.g[0]) - 1, min(geo.g[1], geo.T[1] - p1 * geo.g[1]) - 1,
                              min(geo.g[2], geo.T[2] - p2 * geo.g[2]) - 1);
        };
        // The list's count and entries are asked for first (each thread one entry, without regard to the count: what
        // lies behind it is padding and not used), then the queries, with their row offset worked out in arithmetic
        // rather than read from the table below: they come from HBM (nobody has touched them before), loads return in
        // order, and the tables, the barrier and the first K tile's request do not wait for them that way.
        const int listed = p.kv_count[gamma], first_entry = p.kv_index[(int64_t)gamma * p.max_kv + min(tid, p.max_kv - 1)];
        asm volatile("" ::: "memory");   // (... in this order)
        {
            int gp0, gp1, gp2;
            const int q_origin = group_origin((uint32_t)gamma, gp0, gp1, gp2);
            q_base = grid_base + (uint32_t)q_origin;
            q_first = qt * BM + wave * 32;
            int c0, c1, c2;
            token_coord((uint32_t)(q_first + qcol), c0, c1, c2);
            uint32_t off = (uint32_t)(c0 * T12 + c1 * geo.T[2] + c2) * row_pitch;
            if (MODE == kRagged) {
                q_limit = box_limit(gamma);
                if (qt * BM > last_inside(q_limit)) return;   // no query of this workgroup is inside the grid
                active = q_first <= last_inside(q_limit);
                if (!coord_inside(pack_coord(c0, c1, c2), q_limit)) off = 0;   // a query outside the grid: any valid row will do
            }
            const uint8_t* src = (const uint8_t*)Qh + (uint64_t)q_base * row_pitch + off + 16 * half;
#pragma unroll
            for (int ks = 0; ks < D / 16; ++ks) qf[ks] = *(const frag8*)(src + 32 * ks);
        }
        for (int t = tid; t < n_g; t += NT) {
            int c0, c1, c2;
            token_coord((uint32_t)t, c0, c1, c2);
            s_rowbytes[t] = (uint32_t)(c0 * T12 + c1 * geo.T[2] + c2) * row_pitch;
            if (MODE == kRagged) s_coord[t] = pack_coord(c0, c1, c2);
        }
        // (a caller-made list is taken as it is, but its count and entries are forced into range: a
        // bad list then gives wrong numbers, never an access outside the tables or the tensors)
        const int cnt = min(max(__builtin_amdgcn_readfirstlane(listed), 0), p.max_kv);
        for (int i = tid; i < cnt; i += NT) {
            const int entry = i == tid ? first_entry : p.kv_index[(int64_t)gamma * p.max_kv + i];
            const int gid = min(max(entry, 0), geo.num_groups - 1);
            int p0, p1, p2;
            s_origin[i] = grid_base + (uint32_t)group_origin((uint32_t)gid, p0, p1, p2);
            if (MODE == kRagged) s_limit[i] = box_limit(gid);
        }
        // the tables stand (a barrier that waits for LDS only: __syncthreads() would wait for the queries)
        __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
        __builtin_amdgcn_s_barrier();
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
        tiles_per_group = n_g / kBN;
        if (MODE == kJoint) {
            n_lead = (p.n_global + kBN - 1) / kBN;
            if (p.n_global % kBN) { mask_tile = n_lead - 1; mask_valid = p.n_global % kBN; }
        }
        n_tiles = n_lead + cnt * tiles_per_group;
        if (MODE == kRagged) {
            bool cut = q_limit != full_box;
            for (int i = lane; i < cnt; i += 64) cut = cut || s_limit[i] != full_box;
            clipped = __builtin_amdgcn_ballot_w64(cut) != 0;
            if (clipped) {
                n_tiles = 0;
                for (int i = lane; i < cnt; i += 64) n_tiles += box_tiles(s_limit[i]);
#pragma unroll
                for (int m = 1; m < 64; m *= 2) n_tiles += __shfl_xor(n_tiles, m);
                n_tiles = __builtin_amdgcn_readfirstlane(n_tiles);
            }
        }
        n_listed = cnt;
    }
    if (n_tiles == 0) return;   // an empty list is outside the contract; never touch memory for it
    const int n_walk = n_tiles;                            // tiles of all teams
    const int n_longest = (n_tiles + TEAMS - 1) / TEAMS;   // tiles of the team with most
    if constexpr (TEAMS > 1) {   // from here on tiles are counted within the team
        if (mask_tile >= 0) mask_tile = mask_tile % TEAMS == team ? mask_tile / TEAMS : -1;
        n_tiles = (n_tiles - team + TEAMS - 1) / TEAMS;
    }
    // byte offset inside the head of row i of this wave's 32 query (= output) rows; the rows of a
    // dense tile past the last query re-read the last one and are never stored
    auto q_row_off = [&](int i) -> uint64_t {
        if (dense) return (uint64_t)(uint32_t)(p.dense_row0 + min(q_first + i, p.n_dense_rows - 1)) * row_pitch;
        return (uint64_t)q_base * row_pitch + s_rowbytes[q_first + i];
    };

    if (dense) {
        const uint8_t* src = (const uint8_t*)Qh + q_row_off(qcol) + 16 * half;
#pragma unroll
        for (int ks = 0; ks < D / 16; ++ks) qf[ks] = *(const frag8*)(src + 32 * ks);
    }

    f32x16 oacc[D / 32];                  // O^T accumulator: blocks of 32 head dims
    f32x16 S[2];                          // S^T of the two 32-key blocks in flight
    uint32_t pw[2][8];                    // their weights P^T as 16-bit pairs, in accumulator order
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) oacc[db][r] = 0.f;
#pragma unroll
    for (int kb = 0; kb < 2; ++kb) {
#pragma unroll
        for (int r = 0; r < 16; ++r) S[kb][r] = 0.f;
#pragma unroll
        for (int r = 0; r < 8; ++r) pw[kb][r] = 0u;
    }
    float m_ref = -INFINITY;   // reference maximum of raw scores the weights are taken against
    float l_run = 0.f;         // this lane's share of the running sum (its 16 keys per block)
    const float c = p.scale_log2;

    // ---- tile loads: LPW one-KiB pieces per wave; lane -> (row = rows per piece * piece + lane / chunks per row, chunk) ----
    // Address of a piece = head base + (wave-uniform) byte offset of the tile's first token, kept
    // in scalar registers, + a per-lane byte offset: row within the group (one table read) plus
    // the swizzled 16-byte chunk of the row.
    int load_row[LPW];
    uint32_t load_kcol[LPW], load_vcol[LPW];
#pragma unroll
    for (int k = 0; k < LPW; ++k) {
        const int row = 64 / kRowChunks * (wave * LPW + k) + lane / kRowChunks;
        load_row[k] = row;
        load_kcol[k] = (uint32_t)(((lane % kRowChunks) ^ k_swizzle<D>(row)) * 16);   // byte offset of the global chunk
        load_vcol[k] = (uint32_t)(((lane % kRowChunks) ^ v_swizzle<D>(row)) * 16);
    }
    struct TileAddr {
        uint32_t base;        // wave-uniform
        uint32_t off[LPW];    // per lane
    };
    int gi_k = 0, j_k = 0, gi_v = 0, j_v = 0;   // list entry / tile-in-group of the next K (dense walk: and V) tile
    TileAddr ka, va;
    // V(t) lies in the rows of K(t): where the rows come out of table reads, its address is taken
    // from K's with the other swizzle in the column part instead of being looked up again (+0.7 %;
    // the dense walk, whose addresses are arithmetic, measured 1 % slower that way and forms both)
    uint32_t k_to_vcol[LPW];
#pragma unroll
    for (int k = 0; k < LPW; ++k) k_to_vcol[k] = load_vcol[k] - load_kcol[k];
    auto v_from_k = [&](TileAddr& v, const TileAddr& kk) {
        v.base = kk.base;
#pragma unroll
        for (int k = 0; k < LPW; ++k) v.off[k] = kk.off[k] + k_to_vcol[k];
    };
    // Offsets of a tile are looked up one tile before it is fetched, so the table reads never sit
    // between a barrier and the loads that follow it.
    // (clip: the walk of a workgroup that has to do with a clipped group, see `walk`)
    auto tile_addr = [&](auto clip, TileAddr& a, const uint32_t* col, int t, int& gi, int& j) {
        constexpr bool kClip = MODE == kRagged && decltype(clip)::value;
        if constexpr (TEAMS > 1) {   // back to the number of the tile in the walk of all teams
            t = t * TEAMS + team;
            if (!dense) {
                const uint32_t u = (uint32_t)max(0, t - n_lead);
                gi = (int)fdiv(u, p.fd_group_tiles);
                j = (int)u - gi * tiles_per_group;
            }
        }
        if (dense) {
            // consecutive rows of the whole sequence; rows past the end re-read the last token (masked later)
            if constexpr (kBackwards) t = max(0, n_walk - 1 - t);
            a.base = (uint32_t)(t * kBN);
#pragma unroll
            for (int k = 0; k < LPW; ++k)   // (also asked for tiles past the end, never fetched: keep the offset small)
                a.off[k] = (uint32_t)max(0, min(load_row[k], p.n_tokens - 1 - t * kBN)) * row_pitch + col[k];
        } else if (kLeadThenLists) {
            // Both kinds of address are formed every time and one is selected, so that there is no
            // branch (and no block of table reads with waits of its own) inside a step.
            const bool lead = t < n_lead;
            const uint32_t base_list = __builtin_amdgcn_readfirstlane(s_origin[min(gi, n_listed - 1)]);
            a.base = lead ? (uint32_t)(p.global_row0 + t * kBN) : base_list;
#pragma unroll
            for (int k = 0; k < LPW; ++k) {
                const uint32_t o_list = s_rowbytes[j * kBN + load_row[k]];
                const uint32_t o_lead = (uint32_t)max(0, min(load_row[k], p.n_global - 1 - t * kBN)) * row_pitch;
                a.off[k] = (lead ? o_lead : o_list) + col[k];
            }
            if (!lead && ++j == tiles_per_group) { j = 0; ++gi; }
        } else {
            a.base = __builtin_amdgcn_readfirstlane(s_origin[min(gi, n_listed - 1)]);   // (may be asked past the end)
            int tiles_here = tiles_per_group;
            if (kClip) tiles_here = box_tiles(__builtin_amdgcn_readfirstlane(s_limit[min(gi, n_listed - 1)]));
            // kClip: rows of the box beyond the last token of the sequence are pulled back onto it
            const uint64_t to_end = (uint64_t)((uint32_t)geo.n_tokens - 1u - a.base) * row_pitch;
            const uint32_t max_off = to_end > 0xffffffffull ? 0xffffffffu : (uint32_t)to_end;
#pragma unroll
            for (int k = 0; k < LPW; ++k) {
                const uint32_t o = s_rowbytes[j * kBN + load_row[k]];
                a.off[k] = (kClip ? min(o, max_off) : o) + col[k];
            }
            if (++j == tiles_here) { j = 0; ++gi; }
        }
    };
    // The loads are written as inline assembly on purpose: the compiler's wait-count pass treats a
    // direct-to-LDS load it can see as a possible alias of every later LDS read and would drain
    // the prefetch before the first fragment read that follows.  Completion is waited for
    // explicitly (s_waitcnt vmcnt(0)) before the barrier that publishes the tile.
    auto issue_tile = [&](const uint16_t* head, uint8_t* dst_tile, const TileAddr& a) {
        // (made uniform again here: carried across iterations the offset may sit in a vector register)
        const uint8_t* base = (const uint8_t*)head + (uint64_t)__builtin_amdgcn_readfirstlane(a.base) * row_pitch;
#pragma unroll
        for (int k = 0; k < LPW; ++k) {
            // LDS destination of this wave's piece; the hardware adds lane * 16
            const uint32_t lds_dst = __builtin_amdgcn_readfirstlane(
                (uint32_t)(uintptr_t)(LDS_PTR(uint8_t))(dst_tile + (wave * LPW + k) * 1024));
            // (one wait state between the M0 write and the LDS-DMA instruction that reads it)
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2"
                         :: "s"(lds_dst), "v"(a.off[k]), "s"(base) : "memory", "m0");
        }
    };

    // ---- fragment addresses ----------------------------------------------------------------
    // K (A operand of S^T): row 32*kb + qcol, chunk (2*ks + half) ^ swizzle(row)
    const int k_lane_base = qcol * kRowBytes;
    const int k_x = k_swizzle<D>(qcol) ^ half;          // (2*ks + half) ^ sw == (2*ks) ^ (sw ^ half)
    // V (A operand of O^T) via transpose reads: 16-lane block -> (e = row in quad, cq = 4-dim column)
    const int tr_e = (lane & 15) >> 2, tr_cq = lane & 3, tr_dsel = (lane >> 4) & 1;
    const int v_lane_base = (4 * half + tr_e) * kRowBytes + 8 * (tr_cq & 1);
    // chunk = 4*db + 2*dsel + cq/2, swizzled with v_swizzle(row) = v_swizzle(e) = 4*v_x  ->  4*(db ^ v_x) + 2*dsel + cq/2
    const int v_x = v_swizzle<D>(tr_e) >> 2;
    const int v_chunk_lo = 2 * tr_dsel + (tr_cq >> 1);

    // ---- the software pipeline ---------------------------------------------------------------
    // Work is cut into 32-key blocks (half a K/V tile).  For block h the three stages run one half
    // step apart:  QK(h) -> S[h % 2]   |   weights(h-1): S[(h-1) % 2] -> pw[(h-1) % 2]   |
    // PV(h-2) with pw[h % 2].  Inside a half step the three streams are independent of each other,
    // so the vector work can be dealt out evenly between the MFMAs: a 32x32x16 MFMA occupies the
    // matrix pipe for 32 cycles but the issue port for only 8, and up to 24 cycles of other vector
    // instructions fit in its shadow.  (The packed dot product is not one of them: it runs on the
    // matrix pipe and waits for it, so the row sum is taken with plain adds.)
    // (the per-lane part of the K fragment addresses is formed once and pinned in registers: left to
    // itself the compiler re-adds the swizzled chunk offset in front of every read)
    uint32_t k_addr[D / 16];
#pragma unroll
    for (int ks = 0; ks < D / 16; ++ks) {
        k_addr[ks] = (uint32_t)(uintptr_t)(LDS_PTR(uint8_t))(&sK[0][0] + k_lane_base + (((2 * ks) ^ k_x) << 4));
        asm volatile("" : "+v"(k_addr[ks]));
    }
    auto k_frag = [&](int kbuf, int kb, int ks) -> frag8 {
        return *(LDS_PTR(const frag8))(uintptr_t)(k_addr[ks] + kbuf * kTileBytes + (kBN == 64 ? kb * 32 * kRowBytes : 0));
    };
    auto v_frag = [&](int vbuf, int kb, int s2, int db) -> frag8 {
        const uint8_t* src = sV[vbuf] + v_lane_base + ((kBN == 64 ? 32 * kb : 0) + 16 * s2) * kRowBytes + ((4 * (db ^ v_x) + v_chunk_lo) << 4);
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))src);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(src + 8 * kRowBytes));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    auto mask_tail = [&](int kb) {   // the ragged tile: keys past the end of their run get weight 0
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int key = (kBN == 64 ? 32 * kb : 0) + 8 * (r >> 2) + 4 * half + (r & 3);
            if (key >= mask_valid) S[kb][r] = -INFINITY;
        }
    };
    // kRagged: called once per 32-key block, in walk order.  Keys of a border group's box that lie
    // outside the grid get weight 0.  (The first block of every box holds its first token, which is
    // always inside, so the first block of a walk never ends up without a finite score.)
    int gi_m = 0, j_m = 0;   // list entry / tile-in-group of the tile whose scores are being weighted
    auto mask_outside = [&](int kb) {
        const uint32_t lim = __builtin_amdgcn_readfirstlane(s_limit[min(gi_m, n_listed - 1)]);
        if (lim != full_box) {
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                // accumulator registers 4*rq .. 4*rq+3 hold 4 consecutive keys
                const uint4 cc = *(const uint4*)&s_coord[j_m * kBN + (kBN == 64 ? 32 * kb : 0) + 8 * rq + 4 * half];
                if (!coord_inside(cc.x, lim)) S[kb][4 * rq] = -INFINITY;
                if (!coord_inside(cc.y, lim)) S[kb][4 * rq + 1] = -INFINITY;
                if (!coord_inside(cc.z, lim)) S[kb][4 * rq + 2] = -INFINITY;
                if (!coord_inside(cc.w, lim)) S[kb][4 * rq + 3] = -INFINITY;
            }
        }
        if ((kBN == 32 || kb == 1) && ++j_m == box_tiles(lim)) { j_m = 0; ++gi_m; }
    };
    // Weights are taken against a reference maximum m_ref that is only as fresh as it needs to be:
    // the common path computes exp2(c*s - c*m_ref) without looking at the block's own maximum and
    // checks afterwards that no row sum of the block left the safe range.  Only then (and on the
    // first block, whose maximum is taken up front) is the true maximum computed, O and the running
    // sum rescaled, and the block's weights recomputed.  Any reference gives the same quotient
    // O / l; this one keeps every weight below 2^40, which bf16 and the fp32 accumulators hold
    // without loss of relative accuracy.
    auto block_max = [&](int kb) {
        float mx = S[kb][0];
#pragma unroll
        for (int r = 1; r < 16; ++r) mx = fmaxf(mx, S[kb][r]);
        return max_across_halves(mx);
    };
    auto refresh_reference = [&](int kb, float& ls) {   // the rare path
        const float m_new = fmaxf(m_ref, block_max(kb));
        const float alpha = __builtin_amdgcn_exp2f((m_ref - m_new) * c);
        m_ref = m_new;
        l_run *= alpha;
#pragma unroll
        for (int db = 0; db < D / 32; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) oacc[db][r] *= alpha;
        const float mc = m_ref * c;
        ls = 0.f;
#pragma unroll
        for (int r = 0; r < 16; r += 2) {
            const float p0 = __builtin_amdgcn_exp2f(fmaf(S[kb][r], c, -mc));
            const float p1 = __builtin_amdgcn_exp2f(fmaf(S[kb][r + 1], c, -mc));
            pw[kb][r >> 1] = E::pack(p0, p1);
            ls += p0 + p1;
        }
    };

    // ---- prologue: K tile 0 -----------------------------------------------------------------
    TileAddr vb{};
    auto start = [&](auto clip) {
        tile_addr(clip, ka, load_kcol, 0, gi_k, j_k);
        issue_tile(Kh, sK[0], ka);
        if (dense) tile_addr(clip, va, load_vcol, 0, gi_v, j_v);
        else v_from_k(va, ka);
        vb = va;
        if (1 < n_tiles) tile_addr(clip, ka, load_kcol, 1, gi_k, j_k);
    };

    // swap_barrier(t) publishes K(t) and V(t-1), fetched during the previous tile, and frees the
    // buffers of K(t-1) and V(t-2), which are refilled with K(t+1) and V(t) right away.
    // next_addrs(t): looks up where K(t+2) and V(t+1) lie (one tile before they are fetched, so that
    // the table reads never sit between a barrier and the loads that follow it).
    // 32-key tiles (2-wave workgroups): a step is a single 32-key block, so PV trails QK by two tiles
    // and V(t) is only fetched at barrier t+1, into the buffer V(t-2) was read from during step t;
    // vb = where V(t-1) lies, one tile behind va.
    auto next_addrs = [&](auto clip, int t) {
        // (looked up unconditionally, also past the last tile, so that the table reads stay inside the
        // straight-line block around them instead of becoming a block of their own with its own waits)
        if (kBN == 32) vb = va;
        if (dense) tile_addr(clip, va, load_vcol, t + 1, gi_v, j_v);
        else v_from_k(va, ka);   // tile t + 1, whose K part has just been asked for
        tile_addr(clip, ka, load_kcol, t + 2, gi_k, j_k);
    };
    auto swap_barrier = [&](int t) {
        __builtin_amdgcn_s_waitcnt(0);   // this wave's direct-to-LDS loads have landed
        __syncthreads();                 // ... everyone's have, and all reads of the buffers to refill are done
        if (t + 1 < n_tiles) issue_tile(Kh, sK[(t + 1) & 1], ka);
        if (kBN == 64) {
            if (t < n_tiles) issue_tile(Vh, sV[t & 1], va);
        } else {
            if (t >= 1 && t - 1 < n_tiles) issue_tile(Vh, sV[(t - 1) & 1], vb);
        }
    };

    // One step = the two half steps between two barriers, as one instruction stream.  Half KB (0, 1)
    // works on keys 32*KB .. 32*KB+31 of its tiles.  Per half, QK: form S[KB] from the K tile in
    // sK[kbuf]; SM: weights of the block whose scores are in S[KB ^ 1] (0 none, 1 against the current
    // reference, 2 first block of the walk: the reference is its maximum); PV: O^T += V^T P^T for
    // half KB of the V tile in sV[vbuf], with the weights in pw[KB].  check: the walk contains a tile
    // with fewer than 64 valid keys (kRagged: has to do with a clipped group); t_sm0 / t_sm1 = tile index of the block weighted in each half.
    // The items (one MFMA each, with its fragment read kFragAhead items ahead) run in one rolling
    // sequence over both halves; the vector chunks of a half are dealt out over its items.
    auto step = [&](auto qk0_c, auto sm0_c, auto pv0_c, auto qk1_c, auto sm1_c, auto pv1_c, auto check, auto kbuf_c,
                    int vbuf, int t_sm0, int t_sm1) {
        constexpr int kbuf = decltype(kbuf_c)::value;
        constexpr int SMm[2] = {decltype(sm0_c)::value, decltype(sm1_c)::value};
        constexpr int NQ[2] = {decltype(qk0_c)::value ? D / 16 : 0, decltype(qk1_c)::value ? D / 16 : 0};
        constexpr int NP[2] = {decltype(pv0_c)::value ? 2 * (D / 32) : 0, decltype(pv1_c)::value ? 2 * (D / 32) : 0};
        constexpr int NI[2] = {NQ[0] + NP[0], NQ[1] + NP[1]};
        constexpr int NT = NI[0] + NI[1], AHEAD = kFragAhead;
        frag8 fr[NT > 0 ? NT : 1];
        auto fetch = [&](int i) {
            const int h = i < NI[0] ? 0 : 1, j = i - (h ? NI[0] : 0);
            if (j < NQ[h]) fr[i] = k_frag(kbuf, h, j);
            else fr[i] = v_frag(vbuf, h, (j - NQ[h]) / (D / 32), (j - NQ[h]) % (D / 32));
        };
        float mc = 0.f, ls0 = 0.f, ls1 = 0.f, t1[8], e0[8];
        auto sm_begin = [&](int h) {   // h: the half; the block being weighted is h ^ 1
            if (SMm[h] == 0) return;
            const int sb = h ^ 1;
            if constexpr (decltype(check)::value) {
                if constexpr (MODE == kRagged) mask_outside(sb);
                else if ((h ? t_sm1 : t_sm0) == mask_tile) mask_tail(sb);
            }
            if (SMm[h] == 2) {
                m_ref = block_max(sb);
                // (the first block of a team would be a later one of an undivided walk, where scores of -infinity only
                // weigh 0: any reference that later scores replace)
                if (TEAMS > 1 && m_ref == -INFINITY) m_ref = -1e38f / fmaxf(c, 1.f);
            }
            mc = m_ref * c;
        };
        // two vector chunks per pair of scores: {fma, fma, exp2} and {exp2, pack, add, add}
        auto sm_chunk = [&](int h, int ch) {
            const int g = ch >> 1, sb = h ^ 1;
            if ((ch & 1) == 0) {
                const float t0 = fmaf(S[sb][2 * g], c, -mc);
                t1[g] = fmaf(S[sb][2 * g + 1], c, -mc);
                e0[g] = __builtin_amdgcn_exp2f(t0);
            } else {
                const float e1 = __builtin_amdgcn_exp2f(t1[g]);
                pw[sb][g] = E::pack(e0[g], e1);
                asm volatile("" : "+v"(pw[sb][g]));   // (keeps the conversion here: its first use is a block later)
                ls0 = g == 0 ? e0[g] : ls0 + e0[g];
                ls1 = g == 0 ? e1 : ls1 + e1;
            }
        };
        auto sm_end = [&](int h) {
            if (SMm[h] == 0) return;
            float ls = ls0 + ls1;
            if (SMm[h] == 1) {
                if (__builtin_amdgcn_ballot_w64(!(ls < E::kSumLimit)) != 0) refresh_reference(h ^ 1, ls);
            }
            l_run += ls;
        };
        // first of the 16 chunks of half h that go with its item j
        auto chunk_lo = [&](int h, int j) { return SMm[h] ? j * 16 / NI[h] : 0; };
#pragma unroll
        for (int a = 0; a < AHEAD && a < NT; ++a) fetch(a);
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            sm_begin(h);
            if (NI[h] == 0) {
#pragma unroll
                for (int ch = 0; ch < (SMm[h] ? 16 : 0); ++ch) sm_chunk(h, ch);
            }
#pragma unroll
            for (int j = 0; j < NI[h]; ++j) {
                const int i = (h ? NI[0] : 0) + j;
                if (i + AHEAD < NT) fetch(i + AHEAD);
                if (j < NQ[h]) {
                    if (j == 0) {
                        f32x16 zero;
#pragma unroll
                        for (int r = 0; r < 16; ++r) zero[r] = 0.f;
                        S[h] = E::mfma(fr[i], qf[j], zero);
                    } else {
                        S[h] = E::mfma(fr[i], qf[j], S[h]);
                    }
                } else {
                    const int s2 = (j - NQ[h]) / (D / 32), db = (j - NQ[h]) % (D / 32);
                    const uint32_t* w = &pw[h][4 * s2];
                    const frag8 b = __builtin_bit_cast(frag8, make_uint4(w[0], w[1], w[2], w[3]));
                    oacc[db] = E::mfma(fr[i], b, oacc[db]);
                }
#pragma unroll
                for (int ch = chunk_lo(h, j); ch < chunk_lo(h, j + 1); ++ch) sm_chunk(h, ch);
                __builtin_amdgcn_sched_barrier(0);
            }
            sm_end(h);
        }
    };
    using std::integral_constant;
    constexpr integral_constant<int, 0> c0{};
    constexpr integral_constant<int, 1> c1{};
    constexpr integral_constant<int, 2> c2{};
    constexpr std::false_type no{};
    constexpr std::true_type yes{};

    // kRagged: a workgroup whose own group and listed groups are all whole takes the plain walk; in the others (clip) border
    // keys are masked, and waves without a query inside the grid only fetch (90x160 tokens, 16x16 groups, half, 2 x
    // 24 heads: two thirds of the workgroups take the plain walk; 760 -> 741 us, head_dim 64, 250x250 tokens 990 -> 950).
    // (A loop of their own for those waves: a branch around the steps of the others would end the straight-line code that
    // covers the table reads, 1.6 % at 97x70 tokens, head_dim 64.)
    // (Two copies of the walk cost the 32-key kernels 23 (head_dim 128) and 17 spilled registers, all outside of the steps.  One copy
    // that asks in every step whether anything is clipped spills none and is better only where a walk is short and all is over
    // in one round: one | two, 8x8 groups, 24 heads, 20x28 tokens 21.6 | 22.1 us, 60x60 44.2 | 44.5, 250x250 647 | 629; head_dim 64
    // 18.6 | 18.6, 26.9 | 27.0, 363 | 347.)
    auto fetch_only = [&]() {
        start(yes);
        for (int t = 0; t < n_tiles + (kBN == 64 ? 1 : 2); ++t) {   // as many barriers as the walks below have
            swap_barrier(t);
            next_addrs(yes, t);
        }
    };
    if constexpr (kBN == 64) {
        // tile 0: both QK products, and the weights of its first block against that block's maximum
        auto first_tile = [&](auto clip) {
            start(clip);
            swap_barrier(0);
            next_addrs(clip, 0);
            if (!kLists && mask_tile == 0) {
                step(yes, c0, no, no, c0, no, no, c0, 0, 0, 0);
                mask_tail(0);
                step(no, c0, no, yes, c2, no, no, c0, 0, 0, 0);
            } else {
                step(yes, c0, no, yes, c2, no, clip, c0, 0, 0, 0);
            }
        };
        // tile t >= 1, first half: QK(t, keys 0..31), weights of (t-1, keys 32..63), PV of (t-1, keys 0..31);
        // second half: QK(t, 32..63), weights of (t, 0..31), PV of (t-1, 32..63)
        auto tile_step = [&](auto check, auto kbuf, int t) {   // kbuf = t & 1, as a compile-time constant
            swap_barrier(t);
            next_addrs(check, t);
            step(yes, c1, yes, yes, c1, yes, check, kbuf, kbuf ^ 1, t - 1, t);
        };
        auto walk = [&](auto check) {
            int t = 1;   // (two steps per trip: the LDS buffers of every step are compile-time constants)
            for (; t + 1 < n_tiles; t += 2) {
                tile_step(check, c1, t);
                tile_step(check, c0, t + 1);
            }
            if (t < n_tiles) tile_step(check, c1, t);
            swap_barrier(n_tiles);
            step(no, c1, yes, no, c0, yes, check, c0, (n_tiles - 1) & 1, n_tiles - 1, n_tiles - 1);
        };
        auto walk_backwards = [&]() {   // (of a tile cut short the first step weights one half, the second step the other)
            if (n_tiles > 1) tile_step(yes, c1, 1);
            int t = 2;
            for (; t + 1 < n_tiles; t += 2) {
                tile_step(no, c0, t);
                tile_step(no, c1, t + 1);
            }
            if (t < n_tiles) tile_step(no, c0, t);
            swap_barrier(n_tiles);
            step(no, c1, yes, no, c0, yes, yes, c0, (n_tiles - 1) & 1, n_tiles - 1, n_tiles - 1);
        };
        if (TEAMS > 1 && n_tiles == 0) {
        } else if constexpr (kBackwards) {
            first_tile(no);
            walk_backwards();
        } else if constexpr (MODE == kRagged) {
            if (clipped && !active) {
                fetch_only();
            } else if (clipped) {
                first_tile(yes);
                walk(yes);
            } else {
                first_tile(no);
                walk(no);
            }
        } else {
            first_tile(no);
            if (!kLists && mask_tile >= 0) walk(yes);
            else walk(no);
        }
    } else {
        // 32-key tiles: the step behind barrier b forms the scores of tile b, weights tile b-1 and adds
        // tile b-2 to O^T, all in the half (of S, pw and of the K and V buffers) of its parity.
        auto block_step = [&](auto check, auto par, auto qk, auto sm, auto pv, int b) {
            swap_barrier(b);
            next_addrs(check, b);
            if constexpr (decltype(par)::value == 0) step(qk, sm, pv, no, c0, no, check, c0, 0, b - 1, 0);
            else step(no, c0, no, qk, sm, pv, check, c1, 1, 0, b - 1);
        };
        auto walk = [&](auto check) {
            start(check);
            block_step(check, c0, yes, c0, no, 0);
            if (n_tiles > 1) block_step(check, c1, yes, c2, no, 1);
            else block_step(check, c1, no, c2, no, 1);
            int b = 2;
            for (; b + 1 < n_tiles; b += 2) {
                block_step(check, c0, yes, c1, yes, b);
                block_step(check, c1, yes, c1, yes, b + 1);
            }
            if (b < n_tiles) { block_step(check, c0, yes, c1, yes, b); ++b; }
            // here b = max(n_tiles, 2); the last tile still has to be weighted (unless it was the first) and added
            if (n_tiles >= 2) {
                if (b & 1) block_step(check, c1, no, c1, yes, b);
                else block_step(check, c0, no, c1, yes, b);
                ++b;
            }
            if (b & 1) block_step(check, c1, no, c0, yes, b);
            else block_step(check, c0, no, c0, yes, b);
        };
        if (TEAMS > 1 && n_tiles == 0) {
        } else if (kBackwards) {
            walk(yes);
        } else if (MODE == kRagged && clipped && !active) {
            fetch_only();
        } else if (MODE == kRagged ? clipped : !kLists && mask_tile >= 0) {
            walk(yes);
        } else {
            walk(no);
        }
    }

    // ---- merge of the teams -------------------------------------------------------------------
    // Every team leaves its O (fp32, [query][16-byte chunks, the chunk number XORed with the query]), reference and
    // sum in LDS; a thread then adds up a share of one query's head dims.
    if constexpr (TEAMS > 1) {
        constexpr int kMore = BN == 64 ? 1 : 2;   // barriers of a walk beside its tiles
        for (int i = n_tiles == 0 ? 0 : n_tiles + kMore; i < n_longest + kMore; ++i) __syncthreads();
        __syncthreads();   // everyone has finished with the tile buffers
        static_assert(TEAMS * BM * D * 4 == 4 * TEAMS * kTileBytes, "the partial results fill the tile buffers");
        constexpr int kChunks = D / 4;
        __shared__ float s_m[TEAMS][BM], s_l[TEAMS][BM];
        float* const part = (float*)&k_tiles[0][0];
        {
            const int row = wave * 32 + qcol;
            float* const dst = part + (team * BM + row) * D;
#pragma unroll
            for (int db = 0; db < D / 32; ++db)
#pragma unroll
                for (int rq = 0; rq < 4; ++rq) {
                    const f32x16& o = oacc[db];
                    *(float4*)(dst + 4 * ((8 * db + 2 * rq + half) ^ (row % kChunks))) =
                        make_float4(o[4 * rq], o[4 * rq + 1], o[4 * rq + 2], o[4 * rq + 3]);
                }
            const float l = sum_across_halves(l_run);
            if (half == 0) {
                s_m[team][row] = m_ref;
                s_l[team][row] = l;
            }
        }
        __syncthreads();
        constexpr int TPR = NT / BM, kPieces = D / 8 / TPR;   // threads of a row; 16-byte pieces of the output row for each
        const int row = tid / TPR, sub = tid % TPR, q_tile = q_first - wave * 32;
        if (dense && q_tile + row >= p.n_dense_rows) return;
        float M = s_m[0][row], f[TEAMS], sum = 0.f;
#pragma unroll
        for (int w = 1; w < TEAMS; ++w) M = fmaxf(M, s_m[w][row]);
#pragma unroll
        for (int w = 0; w < TEAMS; ++w) {   // (a team without tiles: weight 0)
            f[w] = __builtin_amdgcn_exp2f((s_m[w][row] - M) * c);
            sum = fmaf(f[w], s_l[w][row], sum);
        }
        const float inv = 1.f / sum;
        const uint64_t out_row = dense ? (uint64_t)(uint32_t)(p.dense_row0 + q_tile + row)
                                       : (uint64_t)(q_base + s_rowbytes[q_tile + row] / row_pitch);
        uint8_t* const dst = (uint8_t*)Oh + out_row * ((uint32_t)p.o_stride_n * 2u);
#pragma unroll
        for (int i = 0; i < kPieces; ++i) {
            const int piece = i * TPR + sub;
            float x[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) x[e] = 0.f;
#pragma unroll
            for (int w = 0; w < TEAMS; ++w)
#pragma unroll
                for (int u = 0; u < 2; ++u) {
                    const float4 v = *(const float4*)(part + (w * BM + row) * D + 4 * ((2 * piece + u) ^ (row % kChunks)));
                    x[4 * u] = fmaf(f[w], v.x, x[4 * u]);
                    x[4 * u + 1] = fmaf(f[w], v.y, x[4 * u + 1]);
                    x[4 * u + 2] = fmaf(f[w], v.z, x[4 * u + 2]);
                    x[4 * u + 3] = fmaf(f[w], v.w, x[4 * u + 3]);
                }
            uint4 v;
            v.x = E::pack(x[0] * inv, x[1] * inv);
            v.y = E::pack(x[2] * inv, x[3] * inv);
            v.z = E::pack(x[4] * inv, x[5] * inv);
            v.w = E::pack(x[6] * inv, x[7] * inv);
            *(uint4*)(dst + 16 * piece) = v;
        }
        return;
    }

    // ---- epilogue: normalise, round to bf16, store ------------------------------------------
    // In the accumulator layout a lane holds 4 consecutive head dims (8 bytes) at a time of ITS
    // query; stored like that every store instruction would touch 64 different rows.  So each wave
    // turns its 32 x 128 output tile through 4 KiB of LDS, 64 head dims at a time: lanes write
    // their 8-byte pieces, then read back 16-byte chunks as (row = 8*i + lane/8, chunk = lane%8)
    // and store 8 rows x 128 contiguous bytes per instruction.  The K buffers are free by now (last
    // read before the final barrier, nothing in flight); a wave only touches its own 4 KiB, so
    // the only ordering needed is between its own LDS writes and reads.
    const float inv = 1.f / sum_across_halves(l_run);
    {
        static_assert(NWAVES * 4096 <= 2 * kTileBytes, "the epilogue stages 4 KiB per wave in the K buffers");
        uint8_t* stage = &sK[0][0] + wave * 4096;   // [32 rows][8 chunks of 16 B], chunk ^= row & 7
        const int srow = lane >> 3, schunk = lane & 7;
        uint64_t st_off[4];
        bool st_ok[4];
        const uint32_t o_pitch = (uint32_t)p.o_stride_n * 2u;   // O may have a token stride of its own
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const int row = 8 * i + srow;
            st_ok[i] = !dense || q_first + row < p.n_dense_rows;
            if (MODE == kRagged) st_ok[i] = coord_inside(s_coord[q_first + row], q_limit);
            uint64_t off = q_row_off(row);
            if (o_pitch != row_pitch) {   // back to the row index (table entries are whole rows)
                const uint32_t r = dense ? (uint32_t)(off / row_pitch) : q_base + s_rowbytes[q_first + row] / row_pitch;
                off = (uint64_t)r * o_pitch;
            }
            st_off[i] = off + schunk * 16;
        }
        uint8_t* wr = stage + qcol * 128 + 8 * half;
#pragma unroll
        for (int pass = 0; pass < D / 64; ++pass) {
#pragma unroll
            for (int dbp = 0; dbp < 2; ++dbp)
#pragma unroll
                for (int rq = 0; rq < 4; ++rq) {
                    const f32x16& o = oacc[2 * pass + dbp];
                    uint2 v;
                    v.x = E::pack(o[4 * rq] * inv, o[4 * rq + 1] * inv);
                    v.y = E::pack(o[4 * rq + 2] * inv, o[4 * rq + 3] * inv);
                    *(uint2*)(wr + (((4 * dbp + rq) ^ (qcol & 7)) << 4)) = v;
                }
            __builtin_amdgcn_wave_barrier();   // (compiler: keep the reads below the writes above)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int row = 8 * i + srow;
                const uint4 x = *(const uint4*)(stage + row * 128 + ((schunk ^ (row & 7)) << 4));
                if (st_ok[i]) *(uint4*)((uint8_t*)Oh + st_off[i] + pass * 128) = x;
            }
            __builtin_amdgcn_wave_barrier();   // (... and the next pass's writes below these reads)
        }
    }
}

// Wavefronts per SIMD the registers are held down to.  head_dim 128 needs 200 and more: two.  head_dim 64 has
// half the MFMAs per score but the same vector work and fragment latencies, so two waves a SIMD left the kernel
// waiting (720 cycles per wave and 32-key block, as many as at 128, of which the MFMAs are 256): three waves of
// 4-wave workgroups (168 registers) took 256x256 tokens, 3x3 groups of 16x16, 24 heads from 997 to 866 us
// (855 -> 984 TFLOP/s); four spill (1 186 us), and so do two 8-wave workgroups (1 160 us).  Joint sequences spill 17 registers
// (40 bytes) at three and none at two, and are still better off at three: 128x128 tokens in 16x16 groups, 24 heads,
// 512 prompt tokens, 3x3 lists 335 against 355 us, 77 prompt tokens, criss-cross 457 against 497; 256x256 packed 1 369
// against 1 450.
// The 2-wave workgroups on 64-key tiles are held to two waves a SIMD by their 32 KiB of LDS.  Whole groups do best
// with no bound (192 registers; 512x512 tokens, criss-cross in 8x8 groups, 8 heads: 5.22 ms against 5.83 with the 141
// registers of a bound of three), clipped ones with a bound of three (145 registers; 500x500 tokens: 5.99 ms against
// 6.27 with the 208 of none); the joint variant spills below two.
constexpr int waves_per_simd(int nwaves, int bn, int mode, int d) {
    if (d == 128) return 2;
    if (nwaves == 2 && bn == 64) return mode == kJoint ? 2 : mode == kRagged ? 3 : 1;
    return 3;
}

// The kernel: picks this workgroup's query tile (tile_order.h) and runs it.  In joint mode the long-running
// dense tiles over the prompt rows get the lowest block indices, dealt round-robin over the XCDs, and the
// grouped tiles follow.  (Both ways to pick a grouped tile lead to one copy of its code: with a copy each, of the 512x512
// token kernels some spilled 5 to 21 scalar registers, clipped grids 13 to 66; 250x250 tokens 1 640 -> 1 620 us, ranked launches of
// 256-row workgroups 0.5 to 1.3 % more time.  At head_dim 128 the 4-wave grouped kernel has two, and the joint ones: us, two | one copy,
// ranked launches of 128-row workgroups, 5x5 lists, 48x64 tokens, 24 / 26 heads 117 / 119 | 122 / 133, 48x96, 16 heads 126 | 134, 64x80, 14 heads 134 |
// 140; criss-cross 1 to 2 %; joint, 4 waves, 64x64 tokens, 256 prompt tokens, 24 heads 114 | 116.5, 8 waves, 128x128, 512 prompt tokens
// 537 | 543.)
template <int NWAVES, int BN, int MODE, bool F16, int D>
__global__ __launch_bounds__(NWAVES * 64, waves_per_simd(NWAVES, BN, MODE, D)) void attn_mfma_kernel(AttnParams p) {
    __shared__ __attribute__((aligned(1024))) uint8_t sK[2][BN * D * 2];
    __shared__ __attribute__((aligned(1024))) uint8_t sV[2][BN * D * 2];
    const int first_grouped = MODE == kDense ? p.n_dense_tiles : MODE == kJoint ? (p.n_dense_tiles + kNumXcd - 1) / kNumXcd * kNumXcd : 0;
    const int block = (int)blockIdx.x - first_grouped;
    int bh, tile;
    if constexpr (MODE == kDense || MODE == kJoint) {
        if (MODE == kDense || block < 0) {
            if (MODE == kJoint && (int)blockIdx.x >= p.n_dense_tiles) return;
            dense_tile(p, (int)blockIdx.x, bh, tile);
            attn_tile<NWAVES, BN, MODE, F16, D, true, 1>(p, bh, tile, sK, sV);
            return;
        }
    }
    if constexpr (D == 128 && ((MODE == kJoint && NWAVES >= 4) || (MODE == kGrouped && NWAVES == 4))) {
        int gamma;
        if (p.longest_first) {
            if (longest_first_tile(p, block, bh, tile, gamma))
                attn_tile<NWAVES, BN, MODE, F16, D, false, 1>(p, bh, tile, sK, sV, gamma);
        } else if (head_sync_tile(p, block % kNumXcd, block / kNumXcd, bh, tile)) {
            attn_tile<NWAVES, BN, MODE, F16, D, false, 1>(p, bh, tile, sK, sV);
        }
    } else if constexpr (MODE != kDense) {
        int gamma = -1;
        if (p.longest_first ? longest_first_tile(p, block, bh, tile, gamma) : head_sync_tile(p, block % kNumXcd, block / kNumXcd, bh, tile))
            attn_tile<NWAVES, BN, MODE, F16, D, false, 1>(p, bh, tile, sK, sV, gamma);
    }
}

// Small launches: eight waves in teams of NWAVES that share the keys.  (The lines that pick the tile stand here again: in a
// function of their own they cost the kernel above registers, 8192^2 pixels in 16x16 groups 1 %.)
template <int NWAVES, int BN, int MODE, bool F16, int D, int TEAMS>
__global__ __launch_bounds__(NWAVES * TEAMS * 64, 2) void attn_mfma_teams_kernel(AttnParams p) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[4 * TEAMS][BN * D * 2];
    const int first_grouped = MODE == kDense ? p.n_dense_tiles : MODE == kJoint ? (p.n_dense_tiles + kNumXcd - 1) / kNumXcd * kNumXcd : 0;
    const int block = (int)blockIdx.x - first_grouped;
    int bh, tile;
    if constexpr (MODE == kDense || MODE == kJoint) {
        if (MODE == kDense || block < 0) {
            if (MODE == kJoint && (int)blockIdx.x >= p.n_dense_tiles) return;
            dense_tile(p, (int)blockIdx.x, bh, tile);
            attn_tile<NWAVES, BN, MODE, F16, D, true, TEAMS>(p, bh, tile, lds, lds + 2 * TEAMS);
            return;
        }
    }
    if constexpr (MODE != kDense) {
        int gamma = -1;
        if (p.longest_first ? longest_first_tile(p, block, bh, tile, gamma) : head_sync_tile(p, block % kNumXcd, block / kNumXcd, bh, tile))
            attn_tile<NWAVES, BN, MODE, F16, D, false, TEAMS>(p, bh, tile, lds, lds + 2 * TEAMS, gamma);
    }
}

// Launches of little more than one round: p.n_whole tiles of 256 rows, one for every compute unit, the others as two 128-row
// workgroups of two teams each, all longest list first (80x80 tokens in 16x16 groups, 3x3 lists, 12 heads: 78 us as 128-row
// workgroups, 70; 64x80 tokens, 16 heads 79, 71).
template <bool F16>
__global__ __launch_bounds__(512, 2) void attn_mfma_mixed_kernel(AttnParams p) {
    __shared__ __attribute__((aligned(1024))) uint8_t lds[8][64 * 128 * 2];
    const int b = (int)blockIdx.x;
    const bool whole = b < p.n_whole;
    int bh, tile, gamma;
    if (!longest_first_tile(p, whole ? b : p.n_whole + (b - p.n_whole) / 2, bh, tile, gamma)) return;
    if (whole) attn_tile<8, 64, kGrouped, F16, 128, false, 1>(p, bh, tile, lds, lds + 2, gamma);
    else attn_tile<4, 64, kGrouped, F16, 128, false, 2>(p, bh, 2 * tile + ((b - p.n_whole) & 1), lds, lds + 4, gamma);
}

template <int NWAVES, int BN, bool F16, int D>
inline hipError_t launch_one(const AttnParams& p, int mode, hipStream_t stream) {
    const dim3 block(NWAVES * 64);
    const size_t dyn = mode == kDense ? 0 : sizeof(int32_t) * (mode == kRagged ? 2 : 1) * ((size_t)p.geo.group_tokens + p.max_kv);
    const int grouped_blocks = tile_blocks<false>(p), dense_blocks = tile_blocks<true>(p);
    if (mode == kRagged) {
        hipLaunchKernelGGL((attn_mfma_kernel<NWAVES, BN, kRagged, F16, D>), dim3(grouped_blocks), block, dyn, stream, p);
    } else if (mode == kDense) {
        if constexpr (BN == 64 && NWAVES >= 4)   // (the tile heights dense launches use)
            hipLaunchKernelGGL((attn_mfma_kernel<NWAVES, BN, kDense, F16, D>), dim3(dense_blocks), block, dyn, stream, p);
        else
            return hipErrorInvalidValue;
    } else if (mode == kGrouped) {
        hipLaunchKernelGGL((attn_mfma_kernel<NWAVES, BN, kGrouped, F16, D>), dim3(grouped_blocks), block, dyn, stream, p);
    } else {
        if constexpr (BN == 64) {
            const int blocks = xcd_padded_blocks(p.n_dense_tiles) + grouped_blocks;
            hipLaunchKernelGGL((attn_mfma_kernel<NWAVES, BN, kJoint, F16, D>), dim3(blocks), block, dyn, stream, p);
        } else {
            return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

// Workgroups of several teams (p.teams).
template <int NWAVES, int BN, int TEAMS, bool F16, int D>
inline hipError_t launch_teams(const AttnParams& p, int mode, hipStream_t stream) {
    const dim3 block(NWAVES * TEAMS * 64);
    const size_t dyn = mode == kDense ? 0 : sizeof(int32_t) * ((size_t)p.geo.group_tokens + p.max_kv);
    const int grouped_blocks = tile_blocks<false>(p), dense_blocks = tile_blocks<true>(p);
    if (mode == kDense) {
        hipLaunchKernelGGL((attn_mfma_teams_kernel<NWAVES, BN, kDense, F16, D, TEAMS>), dim3(dense_blocks), block, dyn, stream, p);
    } else if (mode == kGrouped) {
        hipLaunchKernelGGL((attn_mfma_teams_kernel<NWAVES, BN, kGrouped, F16, D, TEAMS>), dim3(grouped_blocks), block, dyn, stream, p);
    } else {
        if constexpr (BN == 64) {
            if (mode != kJoint) return hipErrorInvalidValue;
            const int blocks = xcd_padded_blocks(p.n_dense_tiles) + grouped_blocks;
            hipLaunchKernelGGL((attn_mfma_teams_kernel<NWAVES, BN, kJoint, F16, D, TEAMS>), dim3(blocks), block, dyn, stream, p);
        } else {
            return hipErrorInvalidValue;
        }
    }
    return hipGetLastError();
}

// p.q_tiles (and p.q_tiles_dense) were computed by the host for p.q_rows: 256 (head_dim 128 only), 128 or
// 64 rows.
template <bool F16, int D>
inline hipError_t launch_by_tile(const AttnParams& p, int mode, hipStream_t stream) {
    if (p.teams == 4) return launch_teams<2, 32, 4, F16, D>(p, mode, stream);   // 64 rows
    if (p.teams == 2) return launch_teams<4, 64, 2, F16, D>(p, mode, stream);   // 128 rows
    if constexpr (D == 128)
        if (p.n_whole > 0) {
            const size_t dyn = sizeof(int32_t) * ((size_t)p.geo.group_tokens + p.max_kv);
            const int tiles = p.batch * p.heads * p.geo.num_groups * p.q_tiles;
            hipLaunchKernelGGL((attn_mfma_mixed_kernel<F16>), dim3(2 * tiles - p.n_whole), dim3(512), dyn, stream, p);
            return hipGetLastError();
        }
    if constexpr (D == 128)
        if (p.q_rows == 256) return launch_one<8, 64, F16, D>(p, mode, stream);
    if (p.q_rows >= 128) return launch_one<4, 64, F16, D>(p, mode, stream);
    if (mfma_tile_keys(p, mode) == 32) return launch_one<2, 32, F16, D>(p, mode, stream);
    return launch_one<2, 64, F16, D>(p, mode, stream);
}

}  // namespace grat
