// fp32 attention (grouped and dense) on the matrix instructions, head_dim 64 or 128.
//
// Sec. 3.1 Eq. 1 restricted to the attendable KV groups of Sec. 3.2.  This is the precision path: inputs, softmax
// and accumulation are fp32, and products are as good as fp32 ones (v_mfma_f32_*_f32, or all 24 bits of an fp32
// number as three bf16 numbers).
// Group dims need not divide the grid (Eq. 2-4 are floor divisions): a group at the far border is the
// part of its box that lies inside the grid, and its tokens are enumerated over that part only, so no
// work is done for tokens that are not there.  Any group size.
//
// Both kernels form S^T = K Q^T and O^T += V^T P^T.  A lane then owns one query and the weights P^T come
// out of the first product in the layout the second one takes them in: register r of the S^T accumulator
// is the B operand of MFMA r of the second product, whose contraction index runs over the keys that
// register holds across the lane groups (of bf16 MFMAs: of an MFMA for every eight registers).  The A operands of
// fp32 MFMAs are read as 16-byte pieces of K and V rows: one piece feeds four MFMAs, with the head dims taken in
// the order in which the pieces hold them.
//
//   attn_f32_kernel        32 queries a wave, K and V shared through LDS: launches that fill the chip.
//   attn_f32_split_kernel  16 queries a workgroup, whose eight waves share its KEYS and merge at the end, or whose
//                          only wave takes them all: launches too small to give every SIMD a wave of its own, groups
//                          (or sequences) of at most 48 tokens.
#include <algorithm>

#include "grat_common.h"
#include "tile_order.h"

namespace grat {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(8))) short frag8;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(16))) float f32x16;

#define LDS_PTR(T) __attribute__((address_space(3))) T*

// attn_f32_kernel takes weights against a reference that is refreshed only once one of them would exceed
// 2^kTopWeight; the largest then becomes 2^kNewWeight.  Any reference gives the same quotient O / l; the exponent of
// a weight is rounded by its own magnitude, so the reference stays near the largest score (with the largest
// weights at 2^32: error 7.1e-7 instead of 3.9e-7 in the first case below).
constexpr float kTopWeight = 8.f, kNewWeight = 0.f;

// A group as the part of its box inside the grid.
struct Box {
    uint32_t origin;    // row of its first token
    uint32_t tokens;    // tokens inside the grid
    FastDiv f1, f2;     // extents along the last two axes
};
__device__ __forceinline__ Box group_box(const AttnParams& p, uint32_t gid) {
    const Geometry& geo = p.geo;
    uint32_t u, p0, p1, p2;
    fdivmod(gid, p.fd_G2, u, p2);
    fdivmod(u, p.fd_G1, p0, p1);
    const bool last1 = (int)p1 == geo.G[1] - 1, last2 = (int)p2 == geo.G[2] - 1;
    const uint32_t v0 = (int)p0 == geo.G[0] - 1 ? (uint32_t)p.last0 : (uint32_t)geo.g[0];
    Box b;
    b.f1.d = last1 ? p.fd_last1.d : p.fd_g1.d;
    b.f1.m = last1 ? p.fd_last1.m : p.fd_g1.m;
    b.f1.sh = last1 ? p.fd_last1.sh : p.fd_g1.sh;
    b.f2.d = last2 ? p.fd_last2.d : p.fd_g2.d;
    b.f2.m = last2 ? p.fd_last2.m : p.fd_g2.m;
    b.f2.sh = last2 ? p.fd_last2.sh : p.fd_g2.sh;
    b.origin = (p0 * geo.g[0] * geo.T[1] + p1 * geo.g[1]) * geo.T[2] + p2 * geo.g[2];
    b.tokens = v0 * b.f1.d * b.f2.d;
    return b;
}
// token row of the t-th token of a group (last axis fastest inside its box), t < b.tokens
__device__ __forceinline__ uint32_t token_row(const AttnParams& p, const Box& b, uint32_t t) {
    uint32_t u, c0, c1, c2;
    fdivmod(t, b.f2, u, c2);
    fdivmod(u, b.f1, c0, c1);
    return b.origin + (c0 * p.geo.T[1] + c1) * p.geo.T[2] + c2;
}
// listed group i of query group gamma (caller-made lists are forced into range: a bad one gives wrong
// numbers, never an access outside the tensors)
__device__ __forceinline__ uint32_t list_entry(const AttnParams& p, int gamma, int i) {
    return (uint32_t)min(max(p.kv_index[(int64_t)gamma * p.max_kv + i], 0), p.geo.num_groups - 1);
}

__device__ __forceinline__ float* out_row(const AttnParams& p, int b_idx, int h_idx, uint32_t row) {
    return (float*)p.O + (int64_t)b_idx * p.o_stride_b + (int64_t)h_idx * p.o_stride_h + (int64_t)row * p.o_stride_n;
}
// An empty list is outside the contract; the mean of nothing is NaN.
template <int N>
__device__ __forceinline__ void nothing_attended(float* dst) {   // N times four head dims
    const float nan = __builtin_nanf("");
#pragma unroll
    for (int i = 0; i < N; ++i) *(f32x4*)(dst + 4 * i) = f32x4{nan, nan, nan, nan};
}

__device__ __forceinline__ float swap32(float x) { return __shfl_xor(x, 32); }

// ---- 32 queries a wave -------------------------------------------------------------------------
// The products run on the bf16 matrix pipe: a number is the sum of three bf16 numbers, x = x0 + x1 + x2, exactly (8
// significand bits each, rounded to nearest: x - x0 has at most 16 of the 24 left, x - x0 - x1 at most 8), and
// x y = x0 y0 + (x0 y1 + x1 y0) + (x0 y2 + x1 y1 + x2 y0) but for x1 y2 + x2 y1 + x2 y2, which is at most 1.01 * 2^-24
// |x y| (and seldom near it), what an fp32 rounding of the product may be off by.  Products of bf16 numbers are
// exact in fp32 and are added up in fp32.  Six 32x32x16 bf16 MFMAs of 32 cycles do the work of eight 32x32x2 fp32
// MFMAs of 64.  (Two halfs and three products take 290 us instead of 475 in the first case below, but hold 23 bits, and
// fewer of a number that is small beside its neighbours: the range of a half is met by scaling whole tiles.)
// bf16 has the exponents of fp32, so that every number keeps its own 24 bits whatever stands beside it.  At the lower
// end the last term would get lost (numbers from 2^-102 down): Q, K and V are split kScale times as large.  At
// the upper end nothing may overflow: numbers from kLimit on, infinities and huge scores send a workgroup through
// the fp32 instructions (fp32_walk) after all.
struct Split {
    uint32_t t[3];   // the terms of a pair of numbers, first number in the low half
};
__device__ __forceinline__ Split split_pair(float x, float y) {
    Split r;
#pragma unroll
    for (int i = 0; i < 3; ++i) {
        const f32x2 v = {x, y};
        r.t[i] = __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
        x -= __builtin_bit_cast(float, r.t[i] << 16);
        y -= __builtin_bit_cast(float, r.t[i] & 0xffff0000u);
    }
    return r;
}
// Scores: 2^7 dims times kLimit^2 kScale^2 = 2^123; O: weights (2^kTopWeight) times kLimit kScale = 2^66 a key.
// A weight below 2^-126 of 2^kNewWeight is taken as 0: with |V| < kLimit that is less than 2^-92 of an output.
constexpr float kScale = 0x1p+24f, kLimit = 0x1p+34f;
// x is worked out here and not further down, with what it is made of kept in registers until then (left to itself the
// compiler moves sums and maxima that are needed after the walk, or late in a step, behind everything else: 100
// registers more in the walk at head_dim 128, which has none to spare).
template <typename T>
__device__ __forceinline__ void pin(T& x) { asm volatile("" : "+v"(x)); }
__device__ __forceinline__ f32x16 mfma_bf16(frag8 a, frag8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
__device__ __forceinline__ frag8 frag_of(const Split (&s)[4], int term) {
    return __builtin_bit_cast(frag8, make_uint4(s[0].t[term], s[1].t[term], s[2].t[term], s[3].t[term]));
}

// o and the sum of a query follow a new reference of its weights.
template <int N, typename Vec>
__device__ __forceinline__ void rescale(Vec (&o)[N], float& l, float alpha) {
    l *= alpha;
#pragma unroll
    for (int b = 0; b < N; ++b) o[b] *= alpha;
}
// Scores are weighted by exp2(c * (score - m_ref)), m_ref the largest so far (no score is below kNoScore, so that a block
// of nothing but -infinity weighs 0).  For any numbers: the difference of huge scores is formed first, no
// weight is above 1, so that O overflows only where its sum does, and weights below 2^-126 are kept as far as fp32
// has them (exp2f; the bare instruction gives 0 there.  Where lists are a block or two long that is 5 to 10 % of the
// eight-wave kernel's time; a test that picks one of the two costs more).
constexpr float kNoScore = -3.4028234e38f;
template <int R, int N, typename Scores, typename Vec>
__device__ __forceinline__ void weigh(Scores& S, float mx, Vec (&o)[N], float& m_ref, float& l, float c) {
    if (__builtin_amdgcn_ballot_w64(mx > m_ref) != 0) {
        const float m_new = fmaxf(m_ref, mx);
        rescale(o, l, exp2f((m_ref - m_new) * c));
        m_ref = m_new;
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
        S[r] = exp2f((S[r] - m_ref) * c);
        l += S[r];
    }
}
__device__ __forceinline__ float block_max(const f32x16& S) {
    float mx = S[0];
#pragma unroll
    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, S[r]);
    return fmaxf(mx, swap32(mx));
}

// The walk on the fp32 instructions (any numbers): the same operand layouts, K and V shared through LDS as they are.
// K(t+1) is fetched while the waves add tile t to O, V(t) while they form its scores.
// active: this wave has queries; stored: this lane's query exists; lds: room for 256 * D bytes.
template <int D, bool DENSE, int NW>
__device__ __forceinline__ void fp32_walk(const AttnParams& p, uint8_t* lds, int gamma, int cnt, const float* q_src,
                                          const uint8_t* Kh, const uint8_t* Vh, bool active, bool stored, float* dst) {
    constexpr int kKeys = 32, NB = D / 32, CPR = D / 4;   // O^T blocks of 32 head dims; 16-byte chunks in a row
    constexpr int RPP = 64 / CPR;                         // rows in a 1-KiB load of one wave
    constexpr int LPW = kKeys / RPP / NW;                 // such loads per wave and tile
    float* const sK = (float*)lds;
    float* const sV = sK + kKeys * D;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int qcol = lane & 31, half = lane >> 5;
    const uint64_t pitch = (uint64_t)(uint32_t)p.stride_n * 4u;

    // Q^T (B operand): q[4 * j + s] = dim 8 * j + 4 * half + s of this lane's query
    float q[D / 2];
    {
        const float* src = q_src + 4 * half;
#pragma unroll
        for (int j = 0; j < D / 8; ++j) {
            const f32x4 v = *(const f32x4*)(src + 8 * j);
#pragma unroll
            for (int s = 0; s < 4; ++s) q[4 * j + s] = v[s];
        }
    }

    // The walk: entry e of the list, tile j of its tokens; lane l looks after key l % 32 of a tile.
    int e = 0, j = 0;
    uint32_t gid_next = 0, key_row = 0;
    Box kb{};
    int kv_tokens = p.n_tokens;
    auto enter = [&](uint32_t gid) {   // the walk reaches entry e, which is group gid
        if (DENSE) return;
        kb = group_box(p, gid);
        kv_tokens = (int)kb.tokens;
        if (e + 1 < cnt) gid_next = list_entry(p, gamma, e + 1);
    };
    auto find_rows = [&]() {
        const uint32_t t = (uint32_t)min(32 * j + qcol, kv_tokens - 1);
        key_row = DENSE ? t : token_row(p, kb, t);
    };
    // direct-to-LDS loads as inline assembly: the compiler would wait for a load it can see ahead of every
    // later LDS read; completion is waited for explicitly before the barrier that publishes the tile
    auto issue = [&](const uint8_t* head, float* tile, bool swizzle) {
#pragma unroll
        for (int k = 0; k < LPW; ++k) {
            const int piece = wave * LPW + k, row = RPP * piece + lane / CPR, pos = lane % CPR;
            const uint32_t src_row = (uint32_t)__shfl((int)key_row, row);
            const uint8_t* src = head + src_row * pitch + 16 * (swizzle ? pos ^ (row & 15) : pos);
            const uint32_t dst = __builtin_amdgcn_readfirstlane((uint32_t)(uintptr_t)(LDS_PTR(uint8_t))((uint8_t*)tile + piece * 1024));
            asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" :: "s"(dst), "v"(src) : "memory", "m0");
        }
    };
    auto landed = [&]() {
        __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    };

    f32x16 o[NB];
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[b][r] = 0.f;
    float m_ref = kNoScore, l = 0.f;   // l: this lane's share of the sum (its 16 keys of every tile)
    const float c = p.scale_log2;

    enter(DENSE ? 0u : list_entry(p, gamma, 0));
    find_rows();
    issue(Kh, sK, true);
    for (;;) {
        const int n_valid = min(kKeys, kv_tokens - kKeys * j);
        landed();   // K(t) is there, and everyone has finished with V(t-1)
        issue(Vh, sV, false);
        f32x16 S;
        if (active) {
#pragma unroll
            for (int r = 0; r < 16; ++r) S[r] = 0.f;
#pragma unroll
            for (int jj = 0; jj < D / 8; ++jj) {
                const f32x4 kf = *(const f32x4*)&sK[qcol * D + 4 * ((2 * jj + half) ^ (qcol & 15))];
#pragma unroll
                for (int s = 0; s < 4; ++s) S = __builtin_amdgcn_mfma_f32_32x32x2f32(kf[s], q[4 * jj + s], S, 0, 0, 0);
            }
            if (n_valid < kKeys) {
#pragma unroll
                for (int r = 0; r < 16; ++r)
                    if (8 * (r >> 2) + 4 * half + (r & 3) >= n_valid) S[r] = -INFINITY;
            }
            weigh<16>(S, block_max(S), o, m_ref, l, c);
        }
        landed();   // V(t) is there, and everyone has finished with K(t)
        bool more = true;
        if (kKeys * (j + 1) < kv_tokens) {
            ++j;
        } else {
            j = 0;
            more = ++e < cnt;
            if (more) enter(gid_next);
        }
        if (more) {
            find_rows();
            issue(Kh, sK, true);
        }
        if (active) {
            // A operand: rows 4*qcol .. (NB dims of the row's piece): block b holds head dims NB * i + b
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float* src = &sV[(8 * (r >> 2) + 4 * half + (r & 3)) * D + NB * qcol];
                // (rows past the end are copies of the last token: weight 0, but 0 times an infinity is none)
                const bool exists = 8 * (r >> 2) + 4 * half + (r & 3) < n_valid;
                float v[NB];
#pragma unroll
                for (int b = 0; b < NB; ++b) v[b] = exists ? src[b] : 0.f;
#pragma unroll
                for (int b = 0; b < NB; ++b) o[b] = __builtin_amdgcn_mfma_f32_32x32x2f32(v[b], S[r], o[b], 0, 0, 0);
            }
        }
        if (!more) break;
    }

    if (stored) {
        const float inv = 1.f / (l + swap32(l));
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            float* d = dst + NB * (8 * (r >> 2) + 4 * half + (r & 3));
#pragma unroll
            for (int b = 0; b < NB; ++b) d[b] = o[b][r] * inv;
        }
    }
}

// Bound: the bf16 matrix pipe; a 32-key tile takes a wave 6 * D / 8 MFMAs of 32 cycles.  K and V are split once per
// workgroup on their way into LDS (memory -> registers -> three planes each), Q once per wave, the weights where they
// are formed: while the waves form the scores of tile t they split V(t), while they add tile t to O they split
// K(t+1), with a barrier between the halves; the fp32 rows of the next half are in registers or on their way.  Two
// waves per SIMD, from different workgroups (LDS: 56 KiB each at head_dim 128), cover each other's softmax and
// barriers; 64-row workgroups get one.  256 registers (head_dim 128): 27 to 60 spilled ones belong to fp32_walk, the
// walk itself reloads 6 a tile.
// 24 heads x 128, us on the fp32 instructions -> here, error against float64: 64x64 tokens in 16x16 groups,
// criss-cross 699 -> 475, 9.1e-7 -> 3.9e-7 (170 TFLOP/s where a large fp32 library product reaches 141 to 154); 2 079
// tokens dense 518 -> 324, 9.7e-7 -> 4.2e-7; 8 heads, 128x128 tokens in 8x8 groups 344 -> 286.  All products of a score
// in one sum 470 us, 4.8e-7; those of O straight into O 454 us, 7.4e-7.
template <int D, bool DENSE, int NW>
__global__ __launch_bounds__(NW * 64, 2) void attn_f32_kernel(AttnParams p) {
    constexpr int kKeys = 32, NB = D / 32, NK = D / 16, NT = NW * 64;
    constexpr int CPR = D / 4, PIECES = kKeys * CPR / NT; // 16-byte pieces of an fp32 row; ... of a tile, per thread
    constexpr int RPP = NT / CPR;                         // rows from one piece of a thread to its next
    // Rows of the planes are padded so that fragment reads are free of bank conflicts and all their addresses
    // differ by constants.  K: 16 bytes, consecutive rows start at different 16-byte positions.  V, read in blocks
    // of 4 rows x 64 bytes by the transpose read: 64 bytes.
    constexpr int kRowK = 2 * D + 16, kRowV = 2 * D + (D == 128 ? 64 : 192), kPlaneK = kKeys * kRowK, kPlaneV = kKeys * kRowV;
    __shared__ __attribute__((aligned(1024))) uint8_t lds[3 * kPlaneK + 3 * kPlaneV];
    static_assert(sizeof(lds) >= 256 * D, "fp32_walk's tiles");
    uint8_t* const sK = lds;
    uint8_t* const sV = lds + 3 * kPlaneK;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qcol = lane & 31, half = lane >> 5;
    int bh, qt, gamma = 0;
    if (!pick_tile<DENSE>(p, bh, qt, gamma)) return;

    const int b_idx = (int)fdiv((uint32_t)bh, p.fd_heads), h_idx = bh - b_idx * p.heads;
    const int64_t head_off = (int64_t)b_idx * p.stride_b + (int64_t)h_idx * p.stride_h;
    const uint8_t* Kh = (const uint8_t*)((const float*)p.K + head_off);
    const uint8_t* Vh = (const uint8_t*)((const float*)p.V + head_off);
    const uint64_t pitch = (uint64_t)(uint32_t)p.stride_n * 4u;

    const int q_first = (qt * NW + wave) * 32;
    Box qb{};
    if (!DENSE) qb = group_box(p, (uint32_t)gamma);
    const int q_tokens = DENSE ? p.n_tokens : (int)qb.tokens;
    if (qt * NW * 32 >= q_tokens) return;    // a clipped group with fewer query tiles
    const int q_t = min(q_first + qcol, q_tokens - 1);
    const uint32_t q_row = DENSE ? (uint32_t)q_t : token_row(p, qb, (uint32_t)q_t);

    // Q^T (B operand): term t of dims 16 * ks + 8 * half .. + 7 of this lane's query
    const float* q_src = (const float*)p.Q + head_off + (int64_t)q_row * p.stride_n;
    frag8 qf[NK][3];
    const float c = p.scale_log2 * (1.f / (kScale * kScale));   // base-2 exponent per unit of a score, as the scaled operands give it
    bool plain = !(p.scale_log2 > 0x1p-60f);   // this thread has met numbers that cannot be split
    {
        float mx = 0.f;
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            const f32x4 x0 = *(const f32x4*)(q_src + 16 * ks + 8 * half), x1 = *(const f32x4*)(q_src + 16 * ks + 8 * half + 4);
            Split s[4];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                mx = fmaxf(fmaxf(mx, fmaxf(fabsf(x0[2 * i]), fabsf(x0[2 * i + 1]))), fmaxf(fabsf(x1[2 * i]), fabsf(x1[2 * i + 1])));
                s[i] = split_pair(x0[2 * i] * kScale, x0[2 * i + 1] * kScale);
                s[2 + i] = split_pair(x1[2 * i] * kScale, x1[2 * i + 1] * kScale);
            }
#pragma unroll
            for (int u = 0; u < 3; ++u) qf[ks][u] = frag_of(s, u);
        }
        pin(mx);
        plain |= !(mx < kLimit);
    }

    // The walk: entry e of the list, tile j of its tokens; lane l looks after key l % 32 of a tile.
    const int cnt = DENSE ? 1 : min(max(p.kv_count[gamma], 0), p.max_kv);
    if (cnt == 0) {
        if (q_first + qcol < q_tokens) nothing_attended<D / 8>(out_row(p, b_idx, h_idx, q_row) + half * (D / 2));
        return;
    }
    int e = 0, j = 0;
    uint32_t gid_next = 0, key_row = 0;
    Box kb{};
    int kv_tokens = p.n_tokens;
    auto enter = [&](uint32_t gid) {   // the walk reaches entry e, which is group gid
        if (DENSE) return;
        kb = group_box(p, gid);
        kv_tokens = (int)kb.tokens;
        if (e + 1 < cnt) gid_next = list_entry(p, gamma, e + 1);
    };
    auto find_rows = [&]() {
        const uint32_t t = (uint32_t)min(32 * j + qcol, kv_tokens - 1);
        key_row = DENSE ? t : token_row(p, kb, t);
    };
    f32x4 stage[PIECES];
    auto load = [&](const uint8_t* head) {
#pragma unroll
        for (int i = 0; i < PIECES; ++i) {
            const int at = i * NT + tid;
            stage[i] = *(const f32x4*)(head + (uint32_t)__shfl((int)key_row, at / CPR) * pitch + 16 * (at % CPR));
        }
    };
    float stage_max = 0.f;   // largest magnitude of K and V that this thread has split
    uint8_t* k_write = sK + (tid / CPR) * kRowK + 8 * (tid % CPR);
    uint8_t* v_write = sV + (tid / CPR) * kRowV + 8 * (tid % CPR);
    auto split_piece = [&](bool is_v, int i) {
        const f32x4 x = stage[i];
        stage_max = fmaxf(stage_max, fmaxf(fmaxf(fabsf(x[0]), fabsf(x[1])), fmaxf(fabsf(x[2]), fabsf(x[3]))));
        pin(stage_max);
        const Split a = split_pair(x[0] * kScale, x[1] * kScale), b = split_pair(x[2] * kScale, x[3] * kScale);
        uint8_t* dst = is_v ? v_write + i * RPP * kRowV : k_write + i * RPP * kRowK;
        const int plane = is_v ? kPlaneV : kPlaneK;
#pragma unroll
        for (int u = 0; u < 3; ++u) *(uint2*)(dst + u * plane) = make_uint2(a.t[u], b.t[u]);
    };
    // K fragment: row qcol, dims 16 * ks + 8 * half ..  V through the LDS transpose read, whose 16-lane blocks
    // take (row of a quad, 4-dim column)
    const uint8_t* k_lane = sK + qcol * kRowK + 16 * half;
    const uint8_t* v_lane = sV + (4 * half + ((lane & 15) >> 2)) * kRowV + 32 * ((lane >> 4) & 1) + 8 * (lane & 3);
    auto k_frag = [&](int u, int ks) -> frag8 { return *(const frag8*)(k_lane + u * kPlaneK + 32 * ks); };
    auto v_frag = [&](int u, int s2, int db) -> frag8 {
        const uint8_t* src = v_lane + u * kPlaneV + 16 * s2 * kRowV + 64 * db;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))src);
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_PTR(s16x4))(src + 8 * kRowV));
        return __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    };
    auto zero16 = [](f32x16& x) {
#pragma unroll
        for (int r = 0; r < 16; ++r) x[r] = 0.f;
    };

    f32x16 o[NB];   // o[b]: head dims 32 * b + 8 * (r / 4) + 4 * half + r % 4 of this lane's query
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[b][r] = 0.f;
    // exponent of a weight: c * score - m_ref, one multiply-add (fp32_walk takes over where the product is too
    // large for that); l: this lane's share of the sum (its 16 keys of every tile)
    float m_ref = kNoScore, l = 0.f;
    enter(DENSE ? 0u : list_entry(p, gamma, 0));
    find_rows();
    load(Kh);
#pragma unroll
    for (int i = 0; i < PIECES; ++i) split_piece(false, i);
    load(Vh);
    for (;;) {
        const int n_valid = min(kKeys, kv_tokens - kKeys * j);
        bool more = true;
        auto next_tile = [&]() {   // V(t) is split: on to K(t+1)
            if (kKeys * (j + 1) < kv_tokens) {
                ++j;
            } else {
                j = 0;
                more = ++e < cnt;
                if (more) enter(gid_next);
            }
            if (more) {
                find_rows();
                load(Kh);
            }
        };
        __syncthreads();   // K(t) is there, and everyone has finished with V(t-1)
        // (the leading products in a sum of their own: every MFMA rounds, by the magnitude of its sum)
        f32x16 S, S_low;
        zero16(S);
        zero16(S_low);
        frag8 f2 = k_frag(2, 0), f1 = k_frag(1, 0), f0;
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            f0 = k_frag(0, ks);
            S_low = mfma_bf16(f2, qf[ks][0], S_low);
            __builtin_amdgcn_sched_barrier(0);
            if (ks + 1 < NK) f2 = k_frag(2, ks + 1);
            S_low = mfma_bf16(f1, qf[ks][1], S_low);
            S_low = mfma_bf16(f1, qf[ks][0], S_low);
            __builtin_amdgcn_sched_barrier(0);
            if (ks + 1 < NK) f1 = k_frag(1, ks + 1);
            S_low = mfma_bf16(f0, qf[ks][2], S_low);
            S_low = mfma_bf16(f0, qf[ks][1], S_low);
            S = mfma_bf16(f0, qf[ks][0], S);
#pragma unroll
            for (int k = ks * PIECES / NK; k < (ks + 1) * PIECES / NK; ++k) split_piece(true, k);
            __builtin_amdgcn_sched_barrier(0);
        }
        S += S_low;
        next_tile();
        frag8 pf[2][3];   // weights P^T (B operand): keys 16 * s2 ..
        if (n_valid < kKeys) {
            const int left = n_valid - 4 * half;   // (one register instead of 16 kept through the walk)
#pragma unroll
            for (int r = 0; r < 16; ++r)
                if (8 * (r >> 2) + (r & 3) >= left) S[r] = -INFINITY;
        }
        const float mx = block_max(S) * c;
        if (__builtin_amdgcn_ballot_w64(mx > m_ref + kTopWeight) != 0) {
            const float m_new = fmaxf(m_ref, mx - kNewWeight);
            rescale(o, l, __builtin_amdgcn_exp2f(m_ref - m_new));
            m_ref = m_new;
        }
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            S[r] = __builtin_amdgcn_exp2f(fmaf(S[r], c, -m_ref));
            l += S[r];
        }
        pin(l);
#pragma unroll
        for (int s2 = 0; s2 < 2; ++s2) {
            Split w[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) w[i] = split_pair(S[8 * s2 + 2 * i], S[8 * s2 + 2 * i + 1]);
#pragma unroll
            for (int u = 0; u < 3; ++u) pf[s2][u] = frag_of(w, u);
        }
        __syncthreads();   // V(t) is there, and everyone has finished with K(t)
        f32x16 add;   // what this tile adds to 32 head dims, so that O is rounded once a tile
        f2 = v_frag(2, 0, 0);
        f1 = v_frag(1, 0, 0);
#pragma unroll
        for (int i = 0; i < 2 * NB; ++i) {
            const int s2 = i % 2, db = i / 2, s2n = (i + 1) % 2, dbn = (i + 1) / 2;
            if (s2 == 0) zero16(add);
            f0 = v_frag(0, s2, db);
            add = mfma_bf16(f2, pf[s2][0], add);
            __builtin_amdgcn_sched_barrier(0);
            if (i + 1 < 2 * NB) f2 = v_frag(2, s2n, dbn);
            add = mfma_bf16(f1, pf[s2][1], add);
            add = mfma_bf16(f1, pf[s2][0], add);
            __builtin_amdgcn_sched_barrier(0);
            if (i + 1 < 2 * NB) f1 = v_frag(1, s2n, dbn);
            add = mfma_bf16(f0, pf[s2][2], add);
            add = mfma_bf16(f0, pf[s2][1], add);
            add = mfma_bf16(f0, pf[s2][0], add);
            // (after the last tile the registers still hold V: split again for nothing, but without a branch)
#pragma unroll
            for (int k = i * PIECES / (2 * NB); k < (i + 1) * PIECES / (2 * NB); ++k) split_piece(false, k);
            if (s2 == 1) {
                o[db] += add;
                pin(o[db]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        if (!more) break;
        load(Vh);
    }

    plain |= !(stage_max < kLimit) || !(fabsf(m_ref) < 0x1p20f);
    const bool stored = q_first + qcol < q_tokens;
    float* dst = out_row(p, b_idx, h_idx, q_row);
    if (__syncthreads_or(plain)) {
        fp32_walk<D, DENSE, NW>(p, lds, gamma, cnt, q_src, Kh, Vh, q_first < q_tokens, stored, dst);
    } else if (stored) {
        const float inv = 1.f / (l + swap32(l)) * (1.f / kScale);
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
            for (int rq = 0; rq < 4; ++rq) {
                f32x4 v;
#pragma unroll
                for (int i = 0; i < 4; ++i) v[i] = o[b][4 * rq + i] * inv;
                *(f32x4*)(dst + 32 * b + 8 * rq + 4 * half) = v;
            }
    }
}

// ---- 16 queries a workgroup, keys split over its waves -------------------------------------------
// Bound: latency.  A small launch cannot give each of the 1 024 SIMDs 32 queries, and one wave's walk over
// a list is a serial chain of 64-cycle MFMAs; so the tile is 16 queries (16x16x4 MFMAs: the same rate,
// half the chain), wave w takes every eighth block of 16 keys, straight from memory into registers (nobody
// else reads it), one block ahead, and the eight partial results are merged through LDS.  Blocks are cut
// from the listed groups laid end to end, each padded to a multiple of 16 tokens - groups of fewer than
// 16 tokens are not padded but packed, several to a block.  Where the tiles alone fill the chip a workgroup is one
// wave (NW = 1), which has all the keys and nothing to merge.  32x32 tokens in 8x8 groups, 2 heads x 64, 3x3 lists,
// with the list building: 390 us with one query per lane (32 waves in all), 15.3 us here (this kernel alone 12.9 back to back, of which the matrix instructions of its 128
// workgroups are 4; with the entries read behind the count and the lists ranked 14.3).
// Two workgroups a compute unit where LDS has room for them (head_dim 64: 33 of 160 KiB, four waves a SIMD, 128
// registers; the compiler wants 129 and 133 and would leave one: 128x128 tokens in 4x4 groups, 8 heads, eight waves, 182
// us against 122).
template <int D, bool DENSE, int NW>
__global__ __launch_bounds__(NW * 64, D == 64 ? 4 : 2) void attn_f32_split_kernel(AttnParams p) {
    constexpr int NP = D / 64;   // 64-dim parts of a V row

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int col = lane & 15, quarter = lane >> 4;
    int bh, qt, gamma = 0;
    if (!pick_tile<DENSE>(p, bh, qt, gamma)) return;

    const int b_idx = (int)fdiv((uint32_t)bh, p.fd_heads), h_idx = bh - b_idx * p.heads;
    const int64_t head_off = (int64_t)b_idx * p.stride_b + (int64_t)h_idx * p.stride_h;
    const float* Kh = (const float*)p.K + head_off;
    const float* Vh = (const float*)p.V + head_off;
    Box qb{};
    if (!DENSE) qb = group_box(p, (uint32_t)gamma);
    const int q_tokens = DENSE ? p.n_tokens : (int)qb.tokens;
    if (qt * 16 >= q_tokens) return;
    auto query_row = [&](int i) {
        const uint32_t t = (uint32_t)min(qt * 16 + i, q_tokens - 1);
        return DENSE ? t : token_row(p, qb, t);
    };

    // block b: lane looks after key `col` of it.  The group it belongs to is read one block before its rows
    // are needed, its K and V one block before they are multiplied.  (Entries are read without regard to the list's
    // count, so that the first of them do not wait for it: those behind the last one are padding, forced into range
    // like any other, and their keys do not exist.)
    auto entry_of = [&](int b, uint32_t& t) -> int {
        uint32_t e;
        fdivmod((uint32_t)(16 * b + col), p.fd_pad_tokens, e, t);
        return (int)e;
    };
    auto read_gid = [&](int b) -> uint32_t {
        if (DENSE) return 0;
        uint32_t t;
        return list_entry(p, gamma, min(entry_of(b, t), p.max_kv - 1));
    };
    uint32_t gid0 = read_gid(wave), gid1 = read_gid(wave + NW);
    const int cnt = DENSE ? 1 : min(max(p.kv_count[gamma], 0), p.max_kv);
    if (cnt == 0) {
        if (wave == 0 && qt * 16 + col < q_tokens) nothing_attended<D / 16>(out_row(p, b_idx, h_idx, query_row(col)) + quarter * (D / 4));
        return;
    }
    const int n_blocks = DENSE ? (p.n_tokens + 15) / 16 : (int)(((int64_t)cnt * p.pad_tokens + 15) / 16);
    struct Block {
        f32x4 k[D / 16], v[4][NP];
        uint64_t valid;   // bit l: lane l's key exists
    };
    auto fetch = [&](Block& x, int b, uint32_t gid) {
        uint32_t row;
        bool ok;
        if (DENSE) {
            row = (uint32_t)min(16 * b + col, p.n_tokens - 1);
            ok = 16 * b + col < p.n_tokens;
        } else {
            uint32_t t;
            const int e = entry_of(b, t);
            const Box kb = group_box(p, gid);
            ok = e < cnt && t < kb.tokens;
            row = token_row(p, kb, ok ? t : 0u);
        }
        x.valid = __builtin_amdgcn_ballot_w64(ok);
        const float* src = Kh + (int64_t)row * p.stride_n + 4 * quarter;
#pragma unroll
        for (int j = 0; j < D / 16; ++j) x.k[j] = *(const f32x4*)(src + 16 * j);
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t vrow = (uint32_t)__shfl((int)row, 4 * quarter + r);
#pragma unroll
            for (int n = 0; n < NP; ++n) x.v[r][n] = *(const f32x4*)(Vh + (int64_t)vrow * p.stride_n + 64 * n + 4 * col);
        }
    };

    // Q^T (B operand): q[j][s] = dim 16 * j + 4 * quarter + s of query `col`
    f32x4 q[D / 16];
    {
        const float* src = (const float*)p.Q + head_off + (int64_t)query_row(col) * p.stride_n + 4 * quarter;
#pragma unroll
        for (int j = 0; j < D / 16; ++j) q[j] = *(const f32x4*)(src + 16 * j);
    }
    f32x4 o[4 * NP];   // o[4 * n + s]: head dims 64 * n + 4 * i + s, i = 4 * quarter + register
#pragma unroll
    for (int b = 0; b < 4 * NP; ++b) o[b] = f32x4{0.f, 0.f, 0.f, 0.f};
    float m_ref = kNoScore, l = 0.f;
    const float c = p.scale_log2;

    auto add_block = [&](Block& x) {
        if (x.valid == 0) return;   // padding of a clipped group
        f32x4 S = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int j = 0; j < D / 16; ++j)
#pragma unroll
            for (int s = 0; s < 4; ++s) S = __builtin_amdgcn_mfma_f32_16x16x4f32(x.k[j][s], q[j][s], S, 0, 0, 0);
        // lane holds keys 4 * quarter + r of its query.  Keys that do not exist stand for another token of the
        // sequence: weight 0, and no V either (0 times an infinity is no 0)
        if (~x.valid != 0) {
            const uint32_t mine = (uint32_t)x.valid >> (4 * quarter);
#pragma unroll
            for (int r = 0; r < 4; ++r)
                if (!(mine >> r & 1u)) {
                    S[r] = -INFINITY;
#pragma unroll
                    for (int n = 0; n < NP; ++n) x.v[r][n] = f32x4{0.f, 0.f, 0.f, 0.f};
                }
        }
        float mx = fmaxf(fmaxf(S[0], S[1]), fmaxf(S[2], S[3]));
        mx = fmaxf(mx, __shfl_xor(mx, 16));
        mx = fmaxf(mx, __shfl_xor(mx, 32));
        weigh<4>(S, mx, o, m_ref, l, c);
#pragma unroll
        for (int r = 0; r < 4; ++r)
#pragma unroll
            for (int n = 0; n < NP; ++n)
#pragma unroll
                for (int s = 0; s < 4; ++s)
                    o[4 * n + s] = __builtin_amdgcn_mfma_f32_16x16x4f32(x.v[r][n][s], S[r], o[4 * n + s], 0, 0, 0);
    };

    Block x0, x1;
    int b = wave;
    if (b < n_blocks) fetch(x0, b, gid0);
    while (b < n_blocks) {
        gid0 = read_gid(b + 2 * NW);
        if (b + NW < n_blocks) fetch(x1, b + NW, gid1);
        add_block(x0);
        b += NW;
        if (b >= n_blocks) break;
        gid1 = read_gid(b + 2 * NW);
        if (b + NW < n_blocks) fetch(x0, b + NW, gid0);
        add_block(x1);
        b += NW;
    }

    l += __shfl_xor(l, 16);
    l += __shfl_xor(l, 32);
    if constexpr (NW == 1) {
        if (qt * 16 + col < q_tokens) {
            const float inv = 1.f / l;
            float* dst = out_row(p, b_idx, h_idx, query_row(col));
#pragma unroll
            for (int n = 0; n < NP; ++n)
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    *(f32x4*)(dst + 64 * n + 4 * (4 * quarter + r)) =
                        f32x4{o[4 * n][r] * inv, o[4 * n + 1][r] * inv, o[4 * n + 2][r] * inv, o[4 * n + 3][r] * inv};
        }
    } else {   // every wave leaves its reference, sum and O; a thread then adds up one query's share of dims
        __shared__ __attribute__((aligned(16))) float s_o[NW][16][D];
        __shared__ float s_m[NW][16], s_l[NW][16];
        if (quarter == 0) {
            s_m[wave][col] = m_ref;
            s_l[wave][col] = l;
        }
#pragma unroll
        for (int n = 0; n < NP; ++n)
#pragma unroll
            for (int r = 0; r < 4; ++r)
                *(f32x4*)&s_o[wave][col][64 * n + 4 * (4 * quarter + r)] =
                    f32x4{o[4 * n][r], o[4 * n + 1][r], o[4 * n + 2][r], o[4 * n + 3][r]};
        __syncthreads();
        constexpr int DPT = 16 * D / 512;   // head dims per thread: 2 or 4
        const int qi = threadIdx.x / 32, d0 = (threadIdx.x % 32) * DPT;
        float M = s_m[0][qi];
#pragma unroll
        for (int w = 1; w < NW; ++w) M = fmaxf(M, s_m[w][qi]);
        float sum = 0.f, acc[DPT];
#pragma unroll
        for (int d = 0; d < DPT; ++d) acc[d] = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float f = exp2f((s_m[w][qi] - M) * c);   // (a wave without keys: 0)
            sum = fmaf(f, s_l[w][qi], sum);
#pragma unroll
            for (int d = 0; d < DPT; ++d) acc[d] = fmaf(f, s_o[w][qi][d0 + d], acc[d]);
        }
        if (qt * 16 + qi < q_tokens) {
            const float inv = 1.f / sum;
            float* dst = out_row(p, b_idx, h_idx, query_row(qi)) + d0;
#pragma unroll
            for (int d = 0; d < DPT; ++d) dst[d] = acc[d] * inv;
        }
    }
}

// A launch holds fewer than 2^32 threads (with more it silently runs a part of them): workgroups of 512 reach that with
// 2^23 small groups, all heads together, so launches go out in parts of 2^22 workgroups (a multiple of the XCDs, so
// that every workgroup stays on its own).
template <int D, bool DENSE>
static hipError_t launch_d(AttnParams p, int rows, int key_waves, hipStream_t stream) {
    constexpr int kPart = 1 << 22;
    const int blocks = tile_blocks<DENSE>(p);
    for (int first = 0; first < blocks; first += kPart) {
        p.first_block = first;
        const dim3 grid(std::min(kPart, blocks - first));
        if (rows == 16 && key_waves == 1) hipLaunchKernelGGL((attn_f32_split_kernel<D, DENSE, 1>), grid, dim3(64), 0, stream, p);
        else if (rows == 16) hipLaunchKernelGGL((attn_f32_split_kernel<D, DENSE, 8>), grid, dim3(512), 0, stream, p);
        else if (rows == 64) hipLaunchKernelGGL((attn_f32_kernel<D, false, 2>), grid, dim3(128), 0, stream, p);   // (groups only)
        else hipLaunchKernelGGL((attn_f32_kernel<D, DENSE, 4>), grid, dim3(256), 0, stream, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess || blocks - first <= kPart) return e;   // (first + kPart may not fit an int)
    }
    return hipSuccess;
}

// rows: query rows per workgroup, 16, 64 or 128 (f32_tile_rows), for which p's tile counts were made; key_waves: waves
// that share the keys of 16 rows, 1 or 8
hipError_t launch_attn_f32(const AttnParams& p, int rows, int key_waves, int head_dim, bool dense, hipStream_t stream) {
    if (head_dim == 64)
        return dense ? launch_d<64, true>(p, rows, key_waves, stream) : launch_d<64, false>(p, rows, key_waves, stream);
    return dense ? launch_d<128, true>(p, rows, key_waves, stream) : launch_d<128, false>(p, rows, key_waves, stream);
}

}  // namespace grat
