// Host side of libgrat: argument validation and dispatch.  No allocation, no synchronisation.
#include <algorithm>
#include <cmath>
#include <cstdint>

#include "grat_common.h"
#include "grat_probe.h"

namespace grat {
namespace {

constexpr int64_t kMaxElems = (int64_t)1 << 31;
constexpr int32_t kMaxListLen = 8192;

// Validate (ndim, grid, group) and normalise to three axes by prepending unit axes.
grat_status make_geometry(int32_t ndim, const int32_t* grid, const int32_t* group, Geometry* out) {
    if (!grid || !group) return GRAT_ERR_NULL;
    if (ndim < 1 || ndim > 3) return GRAT_ERR_BAD_DIMS;
    Geometry geo;
    int64_t n = 1, ng = 1, G = 1;
    for (int k = 0; k < 3; ++k) {
        const int src = k - (3 - ndim);
        const int32_t T = src >= 0 ? grid[src] : 1;
        const int32_t g = src >= 0 ? group[src] : 1;
        if (T < 1 || g < 1) return GRAT_ERR_BAD_DIMS;
        geo.T[k] = T;
        geo.g[k] = g;
        geo.G[k] = (T + g - 1) / g;
        n *= T;
        ng *= g;
        G *= geo.G[k];
        if (n >= kMaxElems || ng >= kMaxElems) return GRAT_ERR_BAD_DIMS;
    }
    geo.n_tokens = n;
    geo.group_tokens = (int32_t)ng;
    geo.num_groups = (int32_t)G;
    *out = geo;
    return GRAT_OK;
}

grat_status make_radius(int32_t ndim, grat_pattern pattern, const int32_t* radius, int32_t out[3]) {
    out[0] = out[1] = out[2] = 0;
    if (pattern != GRAT_BLOCK) return GRAT_OK;
    if (!radius) return GRAT_ERR_NULL;
    for (int k = 0; k < ndim; ++k) {
        if (radius[k] < 0) return GRAT_ERR_BAD_DIMS;
        out[k + (3 - ndim)] = radius[k];
    }
    return GRAT_OK;
}

bool valid_pattern(grat_pattern p) {
    return p == GRAT_BLOCK || p == GRAT_CROSS || p == GRAT_CROSS_PLANES || p == GRAT_DENSE;
}

int64_t longest_list(const Geometry& geo, int32_t ndim, grat_pattern pattern, const int32_t r[3]) {
    const int first = 3 - ndim;
    int64_t v;
    switch (pattern) {
        case GRAT_BLOCK:
            v = 1;
            for (int k = first; k < 3; ++k) v *= std::min<int64_t>(2 * (int64_t)r[k] + 1, geo.G[k]);
            return v;
        case GRAT_CROSS:
            v = -(ndim - 1);
            for (int k = first; k < 3; ++k) v += geo.G[k];
            return v;
        case GRAT_CROSS_PLANES:
            v = 1;
            for (int k = first; k < 3; ++k) v *= geo.G[k] - 1;
            return geo.num_groups - v;
        default:
            return geo.num_groups;
    }
}

bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }
bool is16(grat_dtype t) { return t == GRAT_BF16 || t == GRAT_F16; }   // the MFMA path's element types

// O's strides when they are not Q's: same rules as in check_tensors.
grat_status check_out_strides(grat_dtype dtype, int32_t head_dim, int64_t b, int64_t h, int64_t n) {
    if (n < head_dim || b < 0 || h < 0) return GRAT_ERR_BAD_DIMS;
    const int vec = is16(dtype) ? 8 : 4;
    if (n % vec || b % vec || h % vec) return GRAT_ERR_UNSUPPORTED;
    if (n >= ((int64_t)1 << 24) || b >= ((int64_t)1 << 46) || h >= ((int64_t)1 << 46)) return GRAT_ERR_UNSUPPORTED;
    return GRAT_OK;
}

// Checks shared by the grouped and the dense attention entry points.
grat_status check_tensors(const void* Q, const void* K, const void* V, void* O, grat_dtype dtype,
                          int32_t batch, int32_t heads, int32_t head_dim, int64_t n_tokens,
                          int64_t stride_b, int64_t stride_h, int64_t stride_n, float scale) {
    if (!Q || !K || !V || !O) return GRAT_ERR_NULL;
    if (batch < 1 || heads < 1 || head_dim < 1 || n_tokens < 1) return GRAT_ERR_BAD_DIMS;
    if (!(scale > 0.f) || !std::isfinite(scale)) return GRAT_ERR_BAD_DIMS;
    if (stride_n < head_dim || stride_b < 0 || stride_h < 0) return GRAT_ERR_BAD_DIMS;
    if (!is16(dtype) && dtype != GRAT_F32) return GRAT_ERR_UNSUPPORTED;
    if (is16(dtype) && head_dim != 64 && head_dim != 128) return GRAT_ERR_UNSUPPORTED;
    if (dtype == GRAT_F32 && head_dim != 64 && head_dim != 128) return GRAT_ERR_UNSUPPORTED;
    // rows are read and written as 16-byte vectors
    const int vec = is16(dtype) ? 8 : 4;
    if (stride_n % vec || stride_b % vec || stride_h % vec) return GRAT_ERR_UNSUPPORTED;
    if (!aligned16(Q) || !aligned16(K) || !aligned16(V) || !aligned16(O)) return GRAT_ERR_UNSUPPORTED;
    // the token stride is kept in 32 bits (a 64-row tile then spans less than 4 GiB); the tensor
    // itself may be larger than that: row addresses are formed in 64 bits
    if (stride_n >= ((int64_t)1 << 24)) return GRAT_ERR_UNSUPPORTED;
    if (stride_b >= ((int64_t)1 << 46) || stride_h >= ((int64_t)1 << 46)) return GRAT_ERR_UNSUPPORTED;
    if ((int64_t)batch * heads >= ((int64_t)1 << 24)) return GRAT_ERR_UNSUPPORTED;
    return GRAT_OK;
}

}  // namespace
}  // namespace grat

using namespace grat;

extern "C" grat_status grat_block_list_shape(int32_t ndim, const int32_t* grid, const int32_t* group,
                                             grat_pattern pattern, const int32_t* radius,
                                             int32_t* num_groups, int32_t* max_kv) {
    if (!num_groups || !max_kv) return GRAT_ERR_NULL;
    Geometry geo;
    grat_status st = make_geometry(ndim, grid, group, &geo);
    if (st != GRAT_OK) return st;
    if (!valid_pattern(pattern)) return GRAT_ERR_BAD_PATTERN;
    int32_t r[3];
    st = make_radius(ndim, pattern, radius, r);
    if (st != GRAT_OK) return st;
    *num_groups = geo.num_groups;
    *max_kv = (int32_t)longest_list(geo, ndim, pattern, r);
    return GRAT_OK;
}

extern "C" grat_status grat_build_block_lists(int32_t ndim, const int32_t* grid, const int32_t* group,
                                              grat_pattern pattern, const int32_t* radius,
                                              int32_t* d_kv_count, int32_t* d_kv_index,
                                              int32_t max_kv, void* hip_stream) {
    if (!d_kv_count || !d_kv_index) return GRAT_ERR_NULL;
    Geometry geo;
    grat_status st = make_geometry(ndim, grid, group, &geo);
    if (st != GRAT_OK) return st;
    if (!valid_pattern(pattern)) return GRAT_ERR_BAD_PATTERN;
    int32_t r[3];
    st = make_radius(ndim, pattern, radius, r);
    if (st != GRAT_OK) return st;
    if (max_kv < longest_list(geo, ndim, pattern, r)) return GRAT_ERR_BUFFER_TOO_SMALL;
    if ((int64_t)geo.num_groups * max_kv >= kMaxElems) return GRAT_ERR_UNSUPPORTED;
    const hipError_t e = launch_build_block_lists(geo, ndim, pattern, r, d_kv_count, d_kv_index,
                                                  max_kv, (hipStream_t)hip_stream);
    return e == hipSuccess ? GRAT_OK : GRAT_ERR_HIP;
}

extern "C" grat_status grat_validate_block_lists(int32_t ndim, const int32_t* grid, const int32_t* group,
                                                 const int32_t* d_kv_count, const int32_t* d_kv_index,
                                                 int32_t max_kv, int32_t* d_status, void* hip_stream) {
    if (!d_kv_count || !d_kv_index || !d_status) return GRAT_ERR_NULL;
    Geometry geo;
    const grat_status st = make_geometry(ndim, grid, group, &geo);
    if (st != GRAT_OK) return st;
    if (max_kv < 1) return GRAT_ERR_BUFFER_TOO_SMALL;
    if ((int64_t)geo.num_groups * max_kv >= kMaxElems) return GRAT_ERR_UNSUPPORTED;
    const hipError_t e = launch_validate_block_lists(geo, d_kv_count, d_kv_index, max_kv, d_status,
                                                     (hipStream_t)hip_stream);
    return e == hipSuccess ? GRAT_OK : GRAT_ERR_HIP;
}

// Tokens a listed group takes up in the key order of the fp32 kernel that works in blocks of 16 keys.
static int32_t pad_tokens(int32_t group_tokens) { return group_tokens < 16 ? group_tokens : (group_tokens + 15) / 16 * 16; }

// Divisors of the MFMA kernel's index decompositions, from the finished launch parameters.
static void fill_fastdivs(AttnParams& p) {
    const Geometry& geo = p.geo;
    p.per_xcd = (geo.num_groups * p.q_tiles + kNumXcd - 1) / kNumXcd;
    p.fd_per_xcd = make_fastdiv((uint32_t)p.per_xcd);
    p.fd_tiles_per_head_dense = make_fastdiv((uint32_t)p.q_tiles_dense);
    p.fd_heads = make_fastdiv((uint32_t)p.heads);
    p.fd_q_tiles = make_fastdiv((uint32_t)p.q_tiles);
    const int rows = geo.G[0] * geo.G[1], cols = geo.G[2], sw = p.strip_w > 0 ? p.strip_w : 1;
    p.strip_full = cols / sw;
    p.fd_strip = make_fastdiv((uint32_t)rows * (uint32_t)sw);
    p.fd_strip_w = make_fastdiv((uint32_t)sw);
    p.fd_strip_tail = make_fastdiv((uint32_t)(cols - p.strip_full * sw));   // (0 becomes 1: no tail strip, never used)
    p.fd_g1 = make_fastdiv((uint32_t)geo.g[1]);
    p.fd_g2 = make_fastdiv((uint32_t)geo.g[2]);
    p.fd_G1 = make_fastdiv((uint32_t)geo.G[1]);
    p.fd_G2 = make_fastdiv((uint32_t)geo.G[2]);
    p.last0 = geo.T[0] - (geo.G[0] - 1) * geo.g[0];
    p.fd_last1 = make_fastdiv((uint32_t)(geo.T[1] - (geo.G[1] - 1) * geo.g[1]));
    p.fd_last2 = make_fastdiv((uint32_t)(geo.T[2] - (geo.G[2] - 1) * geo.g[2]));
    p.pad_tokens = pad_tokens(geo.group_tokens);
    p.fd_pad_tokens = make_fastdiv((uint32_t)p.pad_tokens);
    p.fd_group_tiles = make_fastdiv((uint32_t)(geo.group_tokens / (p.teams == 4 ? 32 : 64)));
}

// Query rows per workgroup of the fp32 path: 16 selects the kernel whose waves own 16 queries (all of them, or a share
// of the keys each), 64 / 128 the one whose waves own 32 queries each.  `rows` = query rows of a group (or of the
// sequence), `problems` = groups x heads x batch, `keys` = an upper bound of a list's keys.
// Where the lines lie, first against second kind, us.
// 512 waves of the second kind (one workgroup a compute unit): up to there its time is that of one walk, the first kind's
// grows with their number.  64x64 tokens in 16x16 groups, 3x3 lists, 256 / 384 / 512 / 640 waves 101 / 146 / 190 / 229
// against 214 to 224; 8 192 tokens dense, 64 dims, 256 / 512 / 768 waves 192 / 357 / 529 against 432; 2 048 tokens dense,
// 256 / 512 waves 112 / 211 against 197; 512 tokens, 256 / 512 waves 37 / 71 against 56.
// 48 tokens: a workgroup of the second kind has at least 64 rows.  128x128 tokens, 8 heads x 128, 3x3 lists in groups of
// 1x17 / 4x8 / 5x8 / 6x8 371 / 231 / 390 / 332 against 515 / 302 / 472 / 407, criss-cross 5x8 / 6x8 1 728 / 1 263 against
// 2 104 / 1 638; 8x8 groups, 64x64 tokens 150 against 76.
// Up to 64 tokens a group 64 rows; beyond, 128 even where a wave or two have no query (6x11 groups, 96x176 tokens, 16
// heads: 1 087 us, 1 126 as three 32-row workgroups were).  Sequences (dense) 128: 5 000 of 64 tokens, head_dim 64 / 128,
// 102 / 206 (first kind 114 / 217), 2 500 of 128 95 / 205 (203 / 395); 2 000 of 48 35 / 67 (31 / 58).
static int f32_tile_rows(int64_t rows, int64_t problems, int64_t keys, bool dense) {
    const int64_t waves = problems * ((rows + 31) / 32);   // of the 32-query kernel
    if (keys < kMaxElems - 65536 && (rows <= 48 || waves < 512)) return 16;
    return rows <= 64 && !dense ? 64 : 128;
}
// Waves that share the keys of 16 rows: one where the launch gives every SIMD a wave that way, or nearly so and there is
// little to share; `tiles` = 16-row tiles of the launch.  One against eight, us, head_dim 64 / 128: 1 024 tiles, 256
// keys 21 / 32 against 22 / 45, 512 keys 36 / 54 against 34 / 72; 512 tiles, 64 keys 10 / 12 against 10 / 17, 256 keys 19 / 28
// against 13 / 24; 256 tiles, 16 keys 11 / 11 against 11 / 17; 1x1, 2x2 and 4x4 groups,
// 128x128 tokens, 8 heads x 64: 157, 90, 70 against 870, 253, 120.
static int f32_key_waves(int64_t tiles, int64_t keys) { return tiles >= 1024 || (tiles >= 256 && keys <= 64) ? 1 : 8; }

// Query rows per workgroup of a dense 16-bit launch.  head_dim 64: 128, three such workgroups share a compute unit (no
// difference to 256 rows otherwise: 8 200 tokens, 16 heads 342 against 341 us).
// head_dim 128: one 256-row workgroup fills a compute unit, or two 128-row ones.  256 rows share K and V among more
// queries, so 128 rows are taken where they leave enough less of the last round idle: a round of them that is at most
// half full takes 0.7 of one (a workgroup alone on its compute unit is faster), and they have to win 6 %.  us for
// 256 / 128 rows (heads x tokens): 1 x 10 240 197 / 144, 24 x 2 816 142 / 126, 8 x 9 216 435 / 390, 24 x 4 096 (1.5
// rounds) 205 / 195; 64 x 1 024 38 / 45, 24 x 2 560 78 / 81, 16 x 4 096 (1.0 rounds) 122 / 129, 24 x 8 192 674 / 710.
// Over 448 launches of 1 to 384 heads, 256 tokens to 200 000, the rule is within 0.4 % of the better of the two, 19 %
// ahead of 256 rows with padded launches (see dense_tile), and more than 3.5 % behind those in five (96 x 768 and 96 x
// 1 024: 7 and 9 %).
static int dense_tile_rows(int head_dim, int64_t rows, int64_t problems) {
    if (head_dim == 64) return 128;
    const int64_t tiles128 = problems * ((rows + 127) / 128), tiles256 = problems * ((rows + 255) / 256);
    const int64_t last = tiles128 % 512;
    const int64_t cost128 = tiles128 / 512 * 10 + (last == 0 ? 0 : last <= 256 ? 7 : 10), cost256 = (tiles256 + 255) / 256 * 10;
    return cost128 * 106 < cost256 * 100 ? 128 : 256;
}

// Teams of waves that share the keys of a 16-bit workgroup: 4 of two waves (64 rows), 2 of four (128 rows), or 1.  A
// launch that cannot give every compute unit a workgroup waits for one workgroup's walk, and that for the memory latency
// of each of its steps (a lone 128-row workgroup takes 1 us for 64 keys, of which its products are 0.45).
// `tiles64` / `tiles128` = workgroups of the launch with that many rows (0: not possible), `keys` = an upper bound of a
// list's keys, `tables` = LDS for them.  us, 1 / 2 / 4 teams, head_dim 128 | 64:
//   64x64 tokens in 16x16 groups, 3x3 lists, 1 head 35 / 30 / 22 | 25.5 / 21.7 / 15.7, 4 heads 36 / 32 / 25 | 26 / 22 / 16.5, 8 heads
//   (256 tiles of 128 rows) 39 / 36 / 43 | 26 / 23 / 27; 32x32 tokens in 8x8 groups 13.0 / - / 10.4 | 10.0 / - / 7.4;
//   own group only (256 keys) 8.0 / 9.2 / 8.6 | 6.1 / 6.5 / 6.2; video 8x32x48, 2 heads 67 / 58 / 61 | 48 / 40 / 40;
//   sequences x tokens: 16 x 512 11.1 / 11.5 / 10.4 | 8.3 / 8.0 / 6.8, 24 x 512 11.2 / 11.7 / 12.5 | 8.4 / 8.1 / 7.1, 8 x 1 024 18.2 / 17.4 /
//   14.1 | 13.5 / 11.8 / 9.2, 10 x 1 024 18.3 / 17.8 / 14.6 | 13.5 / 11.9 / 9.4, 16 x 1 024 18.5 / 18.7 / 16.5 | 13.9 / 12.2 / 10.2, 24 x 1 200 25 / 25 / 33 |
//   18 / 15 / 21, 14 x 1 500 27 / 25 / 35 | 21 / 16 / 23, 8 x 2 048 33 / 30 / 24 | 24 / 20 / 15.5, 1 x 16 384 228 / 189 / 148 | 168 / 130 / 89,
//   1 x 32 768 542 / 485 / 586 | 355 / 292 / 348.
// (Sequences at head_dim 128: the line was drawn with a kernel that spilled registers, which those figures no longer show; four teams
// would now win down to about max(384, 4 * tiles64) keys, 10 x 1 024 18.3 -> 14.6.)
static int key_teams(int head_dim, int64_t tiles64, int64_t tiles128, int64_t keys, int64_t tables, bool dense) {
    if (head_dim * 1024 + 4096 + tables > 160 * 1024) return 1;
    // (groups that could have 128-row workgroups, half as many, short lists: 512 keys, 120 / 168 / 216 tiles of 64 rows 12.1 / 12.6 / 12.9 us as
    // those, 10.5 / 13.2 / 14.7 as four teams; 640 keys, 210 tiles 14.5, 11.7)
    const int64_t enough4 = head_dim == 64   ? 384
                            : dense          ? std::max<int64_t>(640, 8 * tiles64)
                            : tiles128 > 0   ? std::max<int64_t>(512, 2 * tiles64 + 200)
                                             : 512;
    if (tiles64 > 0 && tiles64 <= 256 && keys >= enough4) return 4;
    if (tiles128 > 0 && tiles128 <= 256 && keys >= (head_dim == 64 ? 1024 : 1408)) return 2;
    return 1;
}
// Lists as long as those of a criss-cross, of planes or of all groups: then they are all of one length.
static bool one_length(const Geometry& geo, int64_t max_kv) {
    const int64_t a = geo.G[0], b = geo.G[1], c = geo.G[2], n = geo.num_groups;
    return max_kv == a + b + c - 2 || max_kv == n - (a - 1) * (b - 1) * (c - 1) || max_kv == n;
}
// Joint sequences: a prompt tile walks the whole sequence, which such a launch waits for where the rest of it is done
// sooner.  `rest` = steps of 128 rows x 64 keys of the launch, for each of 512 places; 1 / 2 teams, us, head_dim 128 | 64 with
// (walk / rest): 128x128 tokens, criss-cross, 100 prompt tokens 2 / 8 / 12 / 24 heads (8.1 / 2.0 / 1.3 / 0.7) 252 / 199,
// 356 / 310, 419 / 445, 771 / 868 | 183 / 131, 216 / 202, 257 / 288, 456 / 545; 64x64 tokens, 3x3 lists, 256 prompt tokens, 12 / 24
// heads (2.1 / 1.0) 79 / 64, 113 / 125 | 50 / 43, 70 / 81; 128x128 tokens, 3x3, 512 prompt tokens, 8 heads (2.5) 352 / 246 | 198 / 144.
// Of two teams only 256 workgroups have a place.  Up to that many two teams are always ahead.  With more a second round of theirs has
// to be shorter than what the prompt tiles save.  It is where lists differ in length, most being shorter than the longest, which `rest`
// counts: of 235 such launches with a ratio of at least 1.7 one loses (6 %), and they gain 38 % (8x24x24 tokens in 2x8x8 groups, 10 heads, 74 prompt
// tokens (1.8) 82 / 64; 80x144 in 16x16, 7x7 lists, 4 heads, 21 (1.8) 197 / 176).  Where all have one length (one_length) it is not if they are
// nearly the whole walk (21 launches, 7 to 21 % slower: 64x64, 7x7 lists, 8 heads 98 / 117), nor on walks shorter than 90 tiles with
// a ratio below 2.5 (64x64 in 32x32, criss-cross, 8 heads, 835 prompt tokens (2.0) 104 / 119) or than 44 with one below 3 (23, 9 to 21 %: 64x32,
// 20 heads, 96 prompt tokens (2.3) 44 / 51; but 4x24x24 in 2x8x8, criss-cross, 16 heads, 87 (4.2) 43.5 / 38.2).  Of 420 launches 382 stay and gain 36 %, 3 of them lose more than 2 % (criss-cross, 256x160 in 32x32, 3
// heads (1.7) 853 / 899); the others would lose 13 %.
static int joint_teams(int head_dim, int64_t prompt_tiles, int64_t walk, int64_t group_tiles, int64_t list, int64_t tables, bool equal_lists) {
    if (head_dim * 1024 + 4096 + tables > 160 * 1024) return 1;
    const int64_t rest = prompt_tiles * walk + group_tiles * list;
    const bool short_round = prompt_tiles + group_tiles <= 256 || !equal_lists;
    if (!short_round && 10 * list > 9 * walk) return 1;
    return walk * 512 * 10 >= rest * (short_round || walk >= 90 ? 17 : walk >= 44 ? 25 : 30) ? 2 : 1;
}

// Whole tiles of a mixed launch (attn_mfma_mixed_kernel), 0: not one.  A compute unit each for the first 256 tiles of
// 256 rows; what is left, if it is at most 128 tiles, keeps the others busy as twice as many workgroups of half the walk,
// where 128-row workgroups, two a compute unit, would take another 0.7 of a round.  256-token groups, head_dim 128, us as
// those | mixed, 3x3 lists, means of four allocations: 64x64 tokens, 19 / 21 / 23 / 24 heads 78 / 87 / 95 / 87 | 69 / 74 / 86 / 87 (24 with
// the lists built in the pass 86.3 | 84.4); 64x80, 16 heads 79 | 71; 80x80, 12 heads 78 | 70; 96x128, 8 heads 105 | 96.
// `problems` = batch x heads.  Over 708 launches of 257 to 384 tiles (8 to 64 groups, images and video, 3x3, 5x5 and criss-cross
// lists) mixed launches gain 6.5 % on average, and 53 of them lose more than 2 % (up to 13).  Left out:
//   multiples of four problems with short lists, or few groups and lists that differ in length: ranked 128-row workgroups then
//   have every head on the same two XCDs and miss their L2 less (64x64 tokens, 24 heads 17 MiB a head; 23 heads, where every XCD reads
//   every head, 22), and mixed ones lose 2.0 % (48x64 tokens, 32 heads 80 | 87; 64x64 criss-cross, 24 heads 90 | 92).  Other numbers
//   of problems gain 8.2 %;
//   a second round of up to 32 tiles where lists are longer than half of the groups, which differ most (-0.1 %, but up to -13: 12x24x32 tokens,
//   3x3x3, 8 heads; 96x96, 5x5, 8 heads 151 | 161), or few, short and of an even number of problems (-2.1 %: 64x64, 18 heads 65 | 68).
// The 642 that stay gain 7.3 %, up to 30; 22 lose more than 2 %, the most 8x16x32 tokens, 3x3x3, 20 heads (108 | 116).  Of 155 launches
// of 2 to 7 groups 95 stay, gain 8.9 %, two lose more than 2 %; the others would lose 1.7 %.  After two full rounds
// of 256-row workgroups there is nothing in it (36 heads 118.3 | 117.8), after three it loses (56 heads 177.4 | 184.1), and so do
// 1 024-token groups (96x96 tokens, 8 heads 211 | 221).
static int32_t mixed_whole(int64_t tiles256, int64_t problems, int64_t groups, int64_t max_kv, int64_t tables) {
    if (128 * 1024 + 4096 + tables > 160 * 1024) return 0;
    const int64_t rest = tiles256 - 256;
    if (rest <= 0 || rest > 128) return 0;
    if (problems % 4 == 0 && ((max_kv < 8 && groups < 24) || (groups < 16 && max_kv < groups))) return 0;
    if (rest <= 32 && groups >= 20 && 2 * max_kv > groups) return 0;
    if (rest <= 32 && rest > 16 && groups <= 20 && max_kv < 10 && problems % 2 == 0) return 0;
    return 256;
}

struct OutStrides { int64_t b, h, n; };   // O's own strides (elements)

// LDS the MFMA kernel needs beside its four 16-KiB tiles: the row-offset table of a group and the
// list's group origins, twice that with clipped border groups (box coordinates, in-grid limits).
static bool tables_fit_lds(const Geometry& geo, int32_t max_kv, bool ragged) {
    const int64_t tables = (ragged ? 2 : 1) * ((int64_t)geo.group_tokens + max_kv) * (int64_t)sizeof(int32_t);
    return 4 * 16384 + tables <= 160 * 1024;
}

// A checked call and everything that is decided about its launch.
struct Plan {
    AttnParams p{};
    int mode = kGrouped;    // AttnMode
    int key_waves = 0;      // fp32: f32_key_waves
    int64_t xcd_tiles = 0;  // tiles of the XCD that gets most
};

static grat_status launch(const Plan& plan, grat_dtype dtype, int32_t head_dim, void* hip_stream) {
    const hipError_t e = is16(dtype) ? launch_attn_bf16(plan.p, plan.mode, dtype == GRAT_F16, head_dim, (hipStream_t)hip_stream)
                                     : launch_attn_f32(plan.p, plan.p.q_rows, plan.key_waves, head_dim, plan.mode == kDense,
                                                       (hipStream_t)hip_stream);
    return e == hipSuccess ? GRAT_OK : GRAT_ERR_HIP;
}

// Tiles of the XCD that gets most of a launch: workgroups go to the XCDs in turn, grouped ones either by rank
// (consecutive) or as head_sync_tile deals them (an eighth of a head's tiles each, rounded up; which eighth rotates).
static int64_t most_tiles_of_an_xcd(const AttnParams& p, int64_t heads, bool grouped, bool ranked) {
    int64_t most = 0;
    const int64_t tiles = grouped ? (int64_t)p.geo.num_groups * p.q_tiles : 0, per = (tiles + kNumXcd - 1) / kNumXcd;
    for (int xcd = 0; xcd < kNumXcd; ++xcd) {
        int64_t n = (p.n_dense_tiles + kNumXcd - 1 - xcd) / kNumXcd;
        if (ranked) n += (heads * tiles + kNumXcd - 1 - xcd) / kNumXcd;
        else n += heads / kNumXcd * tiles;
        for (int64_t h = 0; !ranked && h < heads % kNumXcd; ++h) n += std::clamp<int64_t>(tiles - (xcd + h) % kNumXcd * per, 0, per);
        most = std::max(most, n);
    }
    return most;
}

// Shared by grat_attention_fwd (n_global = 0), grat_attention_global_fwd and grat_attention_packed_fwd.
static grat_status plan_attention(const void* Q, const void* K, const void* V, void* O,
                                  grat_dtype dtype, int32_t batch, int32_t heads, int32_t head_dim,
                                  int64_t stride_b, int64_t stride_h, int64_t stride_n,
                                  OutStrides os, float scale,
                                  int32_t n_global, int32_t global_first, int32_t ndim,
                                  const int32_t* grid, const int32_t* group,
                                  const int32_t* d_kv_count, const int32_t* d_kv_index,
                                  int32_t max_kv, Plan& plan) {
    if (!d_kv_count || !d_kv_index) return GRAT_ERR_NULL;
    Geometry geo;
    grat_status st = make_geometry(ndim, grid, group, &geo);
    if (st != GRAT_OK) return st;
    if (n_global < 0) return GRAT_ERR_BAD_DIMS;
    const int64_t seq_len = geo.n_tokens + n_global;
    if (seq_len >= kMaxElems) return GRAT_ERR_BAD_DIMS;
    st = check_tensors(Q, K, V, O, dtype, batch, heads, head_dim, seq_len, stride_b, stride_h,
                       stride_n, scale);
    if (st != GRAT_OK) return st;
    st = check_out_strides(dtype, head_dim, os.b, os.h, os.n);
    if (st != GRAT_OK) return st;
    bool ragged = false;   // a group dim does not divide its grid dim: groups at the far border are clipped
    for (int k = 0; k < 3; ++k) ragged = ragged || geo.T[k] % geo.g[k] != 0;
    if (ragged && n_global > 0) return GRAT_ERR_INDIVISIBLE;   // joint sequences: whole groups only
    if (max_kv < 1) return GRAT_ERR_BUFFER_TOO_SMALL;
    if (max_kv > kMaxListLen) return GRAT_ERR_UNSUPPORTED;
    if (n_global > 0 && !is16(dtype)) return GRAT_ERR_UNSUPPORTED;

    AttnParams& p = plan.p;
    p.Q = Q; p.K = K; p.V = V; p.O = O;
    p.stride_b = stride_b; p.stride_h = stride_h; p.stride_n = (int32_t)stride_n;
    p.o_stride_b = os.b; p.o_stride_h = os.h; p.o_stride_n = (int32_t)os.n;
    p.batch = batch; p.heads = heads;
    p.scale_log2 = scale * 1.4426950408889634f;
    p.geo = geo;
    p.kv_count = d_kv_count; p.kv_index = d_kv_index; p.max_kv = max_kv;
    p.n_tokens = (int32_t)seq_len;

    const int n_g = geo.group_tokens;
    p.teams = 1;
    int bm;   // query rows per workgroup
    const int64_t f32_keys = (int64_t)max_kv * pad_tokens(n_g);   // at most, of a list
    if (is16(dtype)) {
        if (n_g % 64) return GRAT_ERR_UNSUPPORTED;
        // byte offsets inside one group are kept in 32 bits
        const int64_t span_rows = (int64_t)(geo.g[0] - 1) * geo.T[1] * geo.T[2] + (int64_t)(geo.g[1] - 1) * geo.T[2] + geo.g[2];
        if (span_rows * stride_n * 2 >= ((int64_t)1 << 32)) return GRAT_ERR_UNSUPPORTED;
        if (n_g > 4096) return GRAT_ERR_UNSUPPORTED;   // intra-group offset table lives in LDS
        if (!tables_fit_lds(geo, max_kv, ragged)) return GRAT_ERR_UNSUPPORTED;
        // (head_dim 64: three 128-row workgroups share a compute unit, see waves_per_simd)
        bm = n_g % 256 == 0 && head_dim == 128 ? 256 : (n_g % 128 == 0 ? 128 : 64);
        // A launch of fewer than two rounds of 256-row workgroups (one per compute unit) runs as 128-row
        // workgroups, two per compute unit, so that one's prologue and epilogue lie under the other's
        // walk (measured: +5 % at 64x64 tokens, nothing either way from 128x128 tokens on).
        if (bm == 256 && (int64_t)batch * heads * geo.num_groups < 2 * 256) bm = 128;
        if (!ragged) {
            const int64_t bh = (int64_t)batch * heads, tables = ((int64_t)n_g + max_kv) * (int64_t)sizeof(int32_t);
            const int64_t tiles64 = bh * geo.num_groups * (n_g / 64), tiles128 = n_g % 128 ? 0 : tiles64 / 2;
            if (n_global == 0) p.teams = key_teams(head_dim, tiles64, tiles128, (int64_t)max_kv * n_g, tables, false);
            else if (tiles128 > 0) p.teams = joint_teams(head_dim, bh * ((n_global + 127) / 128), (seq_len + 63) / 64, tiles128,
                                                         (int64_t)max_kv * (n_g / 64) + (n_global + 63) / 64, tables, one_length(geo, max_kv));
            if (p.teams == 4) bm = 64;
            else if (p.teams == 2) bm = 128;
            if (p.teams == 1 && n_global == 0 && head_dim == 128 && n_g == 256 && geo.num_groups <= 64)
                p.n_whole = mixed_whole(tiles64 / 4, bh, geo.num_groups, max_kv, tables);
            if (p.n_whole > 0) bm = 256;
        }
    } else {
        bm = f32_tile_rows(n_g, (int64_t)batch * heads * geo.num_groups, f32_keys, false);
    }
    p.q_rows = bm;
    p.q_tiles = (n_g + bm - 1) / bm;
    p.strip_w = geo.G[2] >= 16 ? 8 : geo.G[2];
    // (the launch pads every head's tiles to a multiple of 8: up to 7 more per head)
    const int64_t total = (int64_t)batch * heads * geo.num_groups * p.q_tiles;
    if ((int64_t)batch * heads * ((int64_t)geo.num_groups * p.q_tiles + 8) >= kMaxElems - 8) return GRAT_ERR_UNSUPPORTED;

    plan.mode = ragged ? kRagged : kGrouped;
    // the clipped-box tests of the bf16 kernel pack box coordinates into 12 + 10 + 10 bits
    if (ragged && is16(dtype) && (geo.g[1] > 1024 || geo.g[2] > 1024)) return GRAT_ERR_UNSUPPORTED;
    if (n_global > 0) {   // joint sequence: prompt rows become dense tiles launched ahead of the rest
        plan.mode = kJoint;
        p.n_global = n_global;
        p.global_row0 = global_first ? 0 : (int32_t)geo.n_tokens;
        p.grid_row0 = global_first ? n_global : 0;
        p.n_dense_rows = n_global;
        p.dense_row0 = p.global_row0;
        p.q_tiles_dense = (n_global + bm - 1) / bm;
        p.n_dense_tiles = batch * heads * p.q_tiles_dense;
    }
    // A launch of few rounds of workgroups over few groups hands its tiles out by list length, longest
    // first (measured at 128x128 tokens in 16x16 groups, 24 heads: +14 % for 3x3 lists, +10 % for 5x5,
    // nothing either way for the equally long criss-cross lists; at 64x64 tokens +7 %).  Larger launches
    // keep the order that lets neighbouring groups share their K/V in the L2.
    // (head_dim 64 splits 256-token groups in two: the line lies at the same number of queries)
    // A launch that gives no compute unit more than one workgroup starts them all at once, in whatever order: there the
    // ranking, a memory round trip and 64 steps in every wave, only delays them (1.1 of 13.6 us at 32x32 tokens in 8x8
    // groups, 2 heads x 64, fp32).  But the order without it deals every head's tiles in eighths that are rounded up, and
    // the workgroups that only fill these up need places too: with them the launch has to fit as well.  us ranked | not, at
    // most 256 tiles, 3x3 lists in 16x16 groups: 80x80 tokens, 5 heads 41.7 | 55.3, 48x48 tokens, 14 heads 38.2 | 49.2, at head_dim 64
    // 24.5 | 33.1, 12 heads with 86 prompt tokens 34 | 47.6; 517 launches of up to 256 workgroups are 6 % (up to 22) faster without
    // ranking, 92 of more 13 % (up to 60) slower.  A full 256 of undivided workgroups, which do not have a compute unit to
    // themselves, are ranked (fp32, 16x64 tokens in 8x8 groups, 16 heads x 64 45 | 48), but not the lists of fewer than four groups, which differ little
    // (32x32 tokens in one group, 32 heads 24.8 | 23.8).
    const int64_t workgroups = (int64_t)batch * heads * (((int64_t)geo.num_groups * p.q_tiles + kNumXcd - 1) / kNumXcd * kNumXcd) +
                               xcd_padded_blocks(p.n_dense_tiles);
    p.longest_first = geo.num_groups <= 64 && workgroups > (p.teams > 1 || geo.num_groups < 4 ? 256 : 255) &&
                      (is16(dtype) && head_dim == 64 && n_g % 256 == 0 ? total / 2 : total) <= 16 * 256;
    p.fd_tiles_per_rank = make_fastdiv((uint32_t)(batch * heads * p.q_tiles));
    fill_fastdivs(p);
    plan.key_waves = f32_key_waves(total, f32_keys);
    plan.xcd_tiles = most_tiles_of_an_xcd(p, (int64_t)batch * heads, true, p.longest_first);
    return GRAT_OK;
}

static grat_status attention_fwd(const void* Q, const void* K, const void* V, void* O,
                                 grat_dtype dtype, int32_t batch, int32_t heads, int32_t head_dim,
                                 int64_t stride_b, int64_t stride_h, int64_t stride_n,
                                 OutStrides os, float scale,
                                 int32_t n_global, int32_t global_first, int32_t ndim,
                                 const int32_t* grid, const int32_t* group,
                                 const int32_t* d_kv_count, const int32_t* d_kv_index,
                                 int32_t max_kv, void* hip_stream) {
    Plan plan;
    const grat_status st = plan_attention(Q, K, V, O, dtype, batch, heads, head_dim, stride_b, stride_h, stride_n, os, scale, n_global,
                                          global_first, ndim, grid, group, d_kv_count, d_kv_index, max_kv, plan);
    return st == GRAT_OK ? launch(plan, dtype, head_dim, hip_stream) : st;
}

extern "C" grat_status grat_attention_fwd(const void* Q, const void* K, const void* V, void* O,
                                          grat_dtype dtype, int32_t batch, int32_t heads,
                                          int32_t head_dim, int64_t stride_b, int64_t stride_h,
                                          int64_t stride_n, float scale, int32_t ndim,
                                          const int32_t* grid, const int32_t* group,
                                          const int32_t* d_kv_count, const int32_t* d_kv_index,
                                          int32_t max_kv, void* hip_stream) {
    return attention_fwd(Q, K, V, O, dtype, batch, heads, head_dim, stride_b, stride_h, stride_n,
                         OutStrides{stride_b, stride_h, stride_n}, scale, 0, 1, ndim, grid, group,
                         d_kv_count, d_kv_index, max_kv, hip_stream);
}

extern "C" grat_status grat_attention_global_fwd(const void* Q, const void* K, const void* V, void* O,
                                                 grat_dtype dtype, int32_t batch, int32_t heads,
                                                 int32_t head_dim, int64_t stride_b, int64_t stride_h,
                                                 int64_t stride_n, float scale, int32_t n_global,
                                                 int32_t global_first, int32_t ndim,
                                                 const int32_t* grid, const int32_t* group,
                                                 const int32_t* d_kv_count, const int32_t* d_kv_index,
                                                 int32_t max_kv, void* hip_stream) {
    return attention_fwd(Q, K, V, O, dtype, batch, heads, head_dim, stride_b, stride_h, stride_n,
                         OutStrides{stride_b, stride_h, stride_n}, scale, n_global, global_first,
                         ndim, grid, group, d_kv_count, d_kv_index, max_kv, hip_stream);
}

extern "C" grat_status grat_attention_packed_fwd(const void* QKV, void* O, grat_dtype dtype,
                                                 int32_t batch, int32_t heads, int32_t head_dim,
                                                 float scale, int32_t n_global, int32_t global_first,
                                                 int32_t ndim, const int32_t* grid, const int32_t* group,
                                                 const int32_t* d_kv_count, const int32_t* d_kv_index,
                                                 int32_t max_kv, void* hip_stream) {
    if (!QKV || !O) return GRAT_ERR_NULL;
    if (batch < 1 || heads < 1 || head_dim < 1) return GRAT_ERR_BAD_DIMS;
    if (!is16(dtype) && dtype != GRAT_F32) return GRAT_ERR_UNSUPPORTED;
    Geometry geo;
    const grat_status st = make_geometry(ndim, grid, group, &geo);
    if (st != GRAT_OK) return st;
    if (n_global < 0) return GRAT_ERR_BAD_DIMS;
    const int64_t seq_len = geo.n_tokens + n_global;
    const int64_t hd = (int64_t)heads * head_dim;            // one of Q, K, V of one token
    const size_t esize = is16(dtype) ? 2 : 4;
    const char* base = (const char*)QKV;
    return attention_fwd(base, base + hd * esize, base + 2 * hd * esize, O, dtype, batch, heads,
                         head_dim, seq_len * 3 * hd, head_dim, 3 * hd,
                         OutStrides{seq_len * hd, head_dim, hd}, scale, n_global, global_first, ndim,
                         grid, group, d_kv_count, d_kv_index, max_kv, hip_stream);
}

static grat_status plan_dense(const void* Q, const void* K, const void* V, void* O, grat_dtype dtype, int32_t batch, int32_t heads,
                              int64_t n_tokens, int32_t head_dim, int64_t stride_b, int64_t stride_h, int64_t stride_n, float scale,
                              Plan& plan) {
    if (n_tokens >= kMaxElems) return GRAT_ERR_BAD_DIMS;
    grat_status st = check_tensors(Q, K, V, O, dtype, batch, heads, head_dim, n_tokens, stride_b,
                                   stride_h, stride_n, scale);
    if (st != GRAT_OK) return st;

    AttnParams& p = plan.p;
    p.Q = Q; p.K = K; p.V = V; p.O = O;
    p.stride_b = stride_b; p.stride_h = stride_h; p.stride_n = (int32_t)stride_n;
    p.o_stride_b = stride_b; p.o_stride_h = stride_h; p.o_stride_n = (int32_t)stride_n;
    p.batch = batch; p.heads = heads;
    p.scale_log2 = scale * 1.4426950408889634f;
    p.n_tokens = (int32_t)n_tokens;
    const int64_t bh = (int64_t)batch * heads;
    p.teams = is16(dtype) ? key_teams(head_dim, bh * ((n_tokens + 63) / 64), bh * ((n_tokens + 127) / 128), n_tokens, 0, true) : 1;
    const int bm = p.teams == 4     ? 64
                   : p.teams == 2   ? 128
                   : is16(dtype)    ? dense_tile_rows(head_dim, n_tokens, bh)
                                    : f32_tile_rows(n_tokens, bh, n_tokens, true);
    p.q_rows = bm;
    p.q_tiles = (int32_t)((n_tokens + bm - 1) / bm);
    p.q_tiles_dense = p.q_tiles;
    p.n_dense_tiles = batch * heads * p.q_tiles;
    p.n_dense_rows = (int32_t)n_tokens;
    p.dense_row0 = 0;
    if ((int64_t)batch * heads * ((int64_t)p.q_tiles + 8) >= kMaxElems - 8) return GRAT_ERR_UNSUPPORTED;

    fill_fastdivs(p);
    plan.mode = kDense;
    plan.key_waves = f32_key_waves(bh * p.q_tiles, n_tokens);
    plan.xcd_tiles = most_tiles_of_an_xcd(p, bh, false, false);
    return GRAT_OK;
}

extern "C" grat_status grat_dense_attention_fwd(const void* Q, const void* K, const void* V, void* O,
                                                grat_dtype dtype, int32_t batch, int32_t heads,
                                                int64_t n_tokens, int32_t head_dim,
                                                int64_t stride_b, int64_t stride_h,
                                                int64_t stride_n, float scale, void* hip_stream) {
    Plan plan;
    const grat_status st = plan_dense(Q, K, V, O, dtype, batch, heads, n_tokens, head_dim, stride_b, stride_h, stride_n, scale, plan);
    return st == GRAT_OK ? launch(plan, dtype, head_dim, hip_stream) : st;
}

extern "C" grat_status grat_probe_launch(grat_dtype dtype, int32_t batch, int32_t heads, int32_t head_dim, int32_t n_global,
                                         int32_t ndim, const int32_t* grid, const int32_t* group, int32_t max_kv,
                                         grat_launch_info* info) {
    if (!info) return GRAT_ERR_NULL;
    // a contiguous [B, H, N, d] call; what the pointers point to is not looked at
    void* const t = (void*)(uintptr_t)4096;
    const int32_t* const list = (const int32_t*)t;
    Plan plan;
    if (ndim == 0) {
        const int64_t h = (int64_t)n_global * head_dim;
        const grat_status st = plan_dense(t, t, t, t, dtype, batch, heads, n_global, head_dim, heads * h, h, head_dim, 1.f, plan);
        if (st != GRAT_OK) return st;
    } else {
        Geometry geo;
        grat_status st = make_geometry(ndim, grid, group, &geo);
        if (st != GRAT_OK) return st;
        if (n_global < 0 || head_dim < 1 || heads < 1) return GRAT_ERR_BAD_DIMS;
        const int64_t h = (geo.n_tokens + n_global) * head_dim;
        st = plan_attention(t, t, t, t, dtype, batch, heads, head_dim, heads * h, h, head_dim, OutStrides{heads * h, h, head_dim}, 1.f,
                            n_global, 1, ndim, grid, group, list, list, max_kv, plan);
        if (st != GRAT_OK) return st;
    }
    const AttnParams& p = plan.p;
    *info = grat_launch_info{};
    info->mode = plan.mode;
    info->rows = p.q_rows;
    info->teams = p.teams;
    info->whole_tiles = p.n_whole;
    info->longest_first = p.longest_first;
    if (is16(dtype)) info->tile_keys = mfma_tile_keys(p, plan.mode);
    else if (p.q_rows == 16) info->key_waves = plan.key_waves;
    const int64_t grouped = plan.mode == kDense ? 0 : (int64_t)batch * heads * p.geo.num_groups * p.q_tiles;
    info->tiles = p.n_dense_tiles + (int32_t)grouped;
    info->xcd_tiles = (int32_t)plan.xcd_tiles;
    return GRAT_OK;
}

extern "C" const char* grat_status_string(grat_status status) {
    switch (status) {
        case GRAT_OK: return "ok";
        case GRAT_ERR_NULL: return "a required pointer is NULL";
        case GRAT_ERR_BAD_DIMS: return "bad dimensions, radius, strides or scale";
        case GRAT_ERR_INDIVISIBLE: return "a group dim does not divide its grid dim";
        case GRAT_ERR_BAD_PATTERN: return "unknown pattern";
        case GRAT_ERR_BUFFER_TOO_SMALL: return "max_kv is smaller than the longest list";
        case GRAT_ERR_UNSUPPORTED: return "shape, dtype, alignment or size not supported";
        case GRAT_ERR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}
