// Which query tile a workgroup takes.  Shared by the attention kernels.
#pragma once
#include "grat_common.h"

namespace grat {

// Order in which the query groups of one head are handed to consecutive workgroups: column strips
// of the group grid, `strip_w` groups wide, each walked row by row.  The ~32 workgroups an XCD
// runs at a time then cover a compact 2D patch of groups (4 rows x 8 columns for strip_w = 8)
// whose K/V neighbourhoods overlap in both directions, instead of one long group-row.
// rows = all leading group axes flattened, cols = the last group axis; returns the linear group id.
__device__ __forceinline__ int strip_order_group(uint32_t u, int rows, int cols, const AttnParams& p) {
    uint32_t s = fdiv(u, p.fd_strip);
    int w = p.strip_w;
    FastDiv fw = p.fd_strip_w;
    if ((int)s >= p.strip_full) { s = p.strip_full; w = cols - p.strip_full * p.strip_w; fw = p.fd_strip_tail; }
    const uint32_t v = u - s * (uint32_t)(rows * p.strip_w);
    const uint32_t vq = fdiv(v, fw);
    return (int)(vq * cols + s * p.strip_w + (v - vq * w));
}

// Workgroups are dealt round-robin to the 8 XCDs; block b runs on XCD b % 8 as that XCD's (b / 8)-th
// workgroup.  The XCDs walk the heads TOGETHER: within a head every XCD owns one eighth of the head's tile
// order (a compact range of query groups; which eighth rotates from head to head, so that the short lists
// of border groups are spread evenly), so at any time the whole chip reads the K/V of one or two heads
// (which the memory-side cache holds) and every XCD's L2 sees a compact patch of neighbouring groups.
__device__ __forceinline__ bool head_sync_tile(const AttnParams& p, int xcd, int idx, int& bh, int& t_in_head) {
    const int per = p.per_xcd, tph = p.geo.num_groups * p.q_tiles;
    bh = (int)fdiv((uint32_t)idx, p.fd_per_xcd);
    t_in_head = ((xcd + bh) % kNumXcd) * per + (idx - bh * per);   // (rotated per head: border groups have shorter lists)
    return t_in_head < tph && bh < p.batch * p.heads;
}
// Dense tiles all walk the whole sequence, so which XCD has which is all the same: block b is tile b, head after head,
// and no workgroup only pads the launch.  (One that does has to wait for a place as well, and what is behind it in the
// order waits with it: 64 heads of 1 024 tokens as 256 workgroups of 256 rows, one for each compute unit, took 58.5 us
// among as many empty ones and take 37.6 without; 448 launches on average 11 % more time with them.)
__device__ __forceinline__ void dense_tile(const AttnParams& p, int block, int& bh, int& t_in_head) {
    bh = (int)fdiv((uint32_t)block, p.fd_tiles_per_head_dense);
    t_in_head = block - bh * p.q_tiles_dense;
}
// Small launches (p.longest_first; at most 64 groups): the hardware hands out workgroups in block order
// and a launch of only a few rounds of workgroups ends when its last long one does, so the groups with
// the longest lists go first and the short ones fill the tail.  Block b is query tile b % q_tiles of
// (batch, head) (b / q_tiles) % (batch * heads) of the group whose list is the (b / (q_tiles * batch *
// heads))-th longest (ties: lower id first); lane j ranks group j against the others, every wave for
// itself.
__device__ __forceinline__ bool longest_first_tile(const AttnParams& p, int b, int& bh, int& qt, int& gamma) {
    const int G = p.geo.num_groups;
    const int rank = (int)fdiv((uint32_t)b, p.fd_tiles_per_rank), rem = b - rank * p.batch * p.heads * p.q_tiles;
    if (rank >= G) return false;
    bh = (int)fdiv((uint32_t)rem, p.fd_q_tiles);
    qt = rem - bh * p.q_tiles;
    const int lane = threadIdx.x & 63;
    const int key = lane < G ? min(max(p.kv_count[lane], 0), p.max_kv) * 64 + (63 - lane) : -1;
    int r = 0;
#pragma unroll
    for (int k = 0; k < 64; ++k) r += __builtin_amdgcn_readlane(key, k) > key ? 1 : 0;
    const uint64_t m = __ballot(lane < G && r == rank);   // (the keys differ, so exactly one lane)
    gamma = __builtin_amdgcn_readfirstlane(__ffsll((long long)m) - 1);
    return true;
}
// The query tile of this workgroup in a launch of one kind of tile: tile qt of (batch, head) bh, or (grouped)
// tile qt of query group gamma there.  false: a workgroup that only pads the launch.
template <bool DENSE>
__device__ __forceinline__ bool pick_tile(const AttnParams& p, int& bh, int& qt, int& gamma) {
    const int block = p.first_block + (int)blockIdx.x;
    if (DENSE) {
        dense_tile(p, block, bh, qt);
        return true;
    }
    if (p.longest_first) return longest_first_tile(p, block, bh, qt, gamma);
    int t;
    if (!head_sync_tile(p, block % kNumXcd, block / kNumXcd, bh, t)) return false;
    const uint32_t u = fdiv((uint32_t)t, p.fd_q_tiles);
    qt = t - (int)u * p.q_tiles;
    gamma = strip_order_group(u, p.geo.G[0] * p.geo.G[1], p.geo.G[2], p);
    return true;
}
// workgroups of such a launch
template <bool DENSE>
inline int tile_blocks(const AttnParams& p) {
    return DENSE ? p.n_dense_tiles : kNumXcd * p.per_xcd * p.batch * p.heads;
}

}  // namespace grat
