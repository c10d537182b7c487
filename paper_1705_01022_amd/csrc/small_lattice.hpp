// Whole MCS of a small lattice (L <= 128, 8 x 8-site cells, double tiling at
// device level) in one wave: the lattice lies in LDS as rows of bits, a lane
// holds one cell of one of the step's tiles (L^2 / 256 <= 64 of them, and 64
// is what bounds L).  Launched step by step, an MCS of L = 64 is four launches
// of a few lanes each (p = 1: DT 90, DB 159 us an MCS); here any number of MCS
// is one launch, a round has no barrier, the tiles' block draws are worked out
// by all lanes at the start of a step, and the draws of the next round while
// this round's slope words are on their way: DT 44, DB 64 us (p = .6, q = .4:
// 101 -> 60 and 175 -> 83; L = 128, D = 64: DT 116 -> 43, DB 187 -> 69).  What
// bounds it is one wave's serial chain, 0.17 us a round of about 70
// instructions and one LDS round trip.
#pragma once

#include "kernels.hpp"
#include "mcs_draw.hpp"

namespace okpz {

constexpr uint32_t kSmallLatticeL = 128;
constexpr uint32_t kSmallFieldPitch = 33;  // 32 words a tile; odd, so that tiles read from different banks

template <int SCHEME, bool ACCEPT>
__global__ void __launch_bounds__(64) run_small_kernel(StepArgs A, uint64_t mcs0, uint32_t n_mcs, uint32_t origin_mode)
{
    // what the launch rule fixes, as constants
    A.log2Cx = A.log2Cy = 3u;
    A.s_bits = SCHEME == kDB ? 6u : 4u;
    if (!ACCEPT) A.F_log2 = SCHEME == kDB ? 3u : 2u;
    A.dev_db = 0u;
    __shared__ uint32_t fields[64 * kSmallFieldPitch];  // the tiles' block draws of a step
    __shared__ uint32_t sx[kSmallLatticeL * kSmallLatticeL / 32], sy[kSmallLatticeL * kSmallLatticeL / 32];
    const uint32_t lane = threadIdx.x;
    const uint32_t L = A.L_mask + 1u, log2L = A.nbx_log2 + 5u, site_mask = (1u << 2u * log2L) - 1u;
    // half blocks: the four sx or sy words of a block's rows; LDS rows are L bits
    const uint32_t halves = L * L / 64u;
    auto lds_of = [&](uint32_t t, uint32_t r) {
        const uint32_t blk = t >> 1;
        return ((4u * (blk >> A.nbx_log2) + r) << A.nbx_log2) + (blk & A.nbx_mask);
    };
    for (uint32_t t = lane; t < halves; t += 64u) {
        const uint4 v = reinterpret_cast<const uint4 *>(A.words)[t];
        uint32_t *p = (t & 1u) ? sy : sx;
        p[lds_of(t, 0)] = v.x;
        p[lds_of(t, 1)] = v.y;
        p[lds_of(t, 2)] = v.z;
        p[lds_of(t, 3)] = v.w;
    }
    // the lane's tile and cell
    const uint32_t log2ncell = (uint32_t)__builtin_ctz(A.ncell), ncx = 1u << A.log2ncx;
    const bool act = lane < (L * L >> 8);
    const uint32_t tile = act ? lane >> log2ncell : 0u, cell = lane & (A.ncell - 1u);
    const uint32_t cx = cell & (ncx - 1u), cy = cell >> A.log2ncx, ncy = A.ncell >> A.log2ncx;
    const uint32_t base_u = cx << 3, base_v = cy << 3;
    const uint32_t first = lane - cell;
    const int right = (int)(first + (cy << A.log2ncx) + ((cx + 1u) & (ncx - 1u))) << 2;
    const int below = (int)(first + (((cy + 1u) & (ncy - 1u)) << A.log2ncx) + cx) << 2;
    const uint32_t tx = tile & ((1u << A.log2ntx) - 1u), ty = tile >> A.log2ntx;
    const uint32_t ntiles = (L * L >> 8) >> log2ncell;
    const uint32_t *tile_fields = fields + tile * kSmallFieldPitch;
    wave_order();

    for (uint32_t n = 0; n < n_mcs; ++n) {
        const uint64_t m = mcs0 + n;
        uint32_t ox, oy;
        const u32x4 w = mcs_origin(A, origin_mode, m, ox, oy);
        const uint32_t pick = (uint32_t)(((uint64_t)w.z * 24u) >> 32);
        for (uint32_t k = 0; k < 4u; ++k) {
            const uint32_t set = perm_element(pick, k);
            A.c3 = (uint32_t)(m << 2) | k;
            const uint32_t X0 = ox + 2u * A.Dx * tx + (set & 1u) * A.Dx, Y0 = oy + 2u * A.Dy * ty + (set >> 1) * A.Dy;
            uint32_t rw[4] = {0u, 0u, 0u, 0u};
            for (uint32_t t = lane; t < 8u * ntiles; t += 64u) {
                const u32x4 r = philox4x32_10_lane(A.key0, A.key1, t & 7u, 0xFFFFFFFFu, t >> 3, A.c3);
                uint32_t *f = fields + (t >> 3) * kSmallFieldPitch + 4u * (t & 7u);
                f[0] = r.x;
                f[1] = r.y;
                f[2] = r.z;
                f[3] = r.w;
            }
            wave_order();
            uint32_t fw = 0u;
            // the draw of a round: site, place in the domain, flip mask, rim
            auto draw = [&](uint32_t rho, uint32_t &s, uint32_t &pos, uint32_t &mask, uint32_t &rim) {
                if ((rho & 1u) == 0u) fw = tile_fields[rho >> 1];
                const uint32_t f16 = (rho & 1u) ? fw >> 16 : fw & 0xFFFFu;
                const uint32_t field = next_field(A, rw, rho, cell, tile);
                uint32_t du, dv, u, v;
                drawn_site<SCHEME>(A, field, f16, base_u, base_v, du, dv, u, v);
                s = (((Y0 + v) & A.L_mask) << log2L) + ((X0 + u) & A.L_mask);
                pos = SCHEME == kDB ? u | (v << 16) : 0u;
                rim = SCHEME == kDB ? (du == 7u ? 1u : 0u) | (dv == 7u ? 2u : 0u) : 0u;
                uint32_t pre[1] = {ACCEPT ? field >> A.s_bits : A.flip_table};  // prefix until accept_draws()
                if (ACCEPT) {
                    const uint32_t ids[1] = {cell};
                    accept_draws<1>(A, pre, ids, rho, tile);
                }
                mask = pre[0];
            };
            auto try_site = [&](uint32_t s, uint32_t mask, bool enable) {
                const uint32_t sr = (s & ~A.L_mask) | ((s + 1u) & A.L_mask), sd = (s + L) & site_mask;
                const uint32_t w0 = sx[s >> 5], w1 = sx[sr >> 5], y0 = sy[s >> 5], y1 = sy[sd >> 5];
                const uint32_t key = __builtin_amdgcn_ubfe(w1, sr, 1) << 3 | __builtin_amdgcn_ubfe(w0, s, 1) << 2 |
                                     __builtin_amdgcn_ubfe(y0, s, 1) << 1 | __builtin_amdgcn_ubfe(y1, s, 1);
                if (enable && __builtin_amdgcn_ubfe(mask, key, 1) != 0u) {
                    const uint32_t b = 1u << (s & 31u);
                    atomicXor(&sx[s >> 5], b);
                    atomicXor(&sx[sr >> 5], 1u << (sr & 31u));
                    atomicXor(&sy[s >> 5], b);
                    atomicXor(&sy[sd >> 5], b);
                }
            };
            uint32_t s, pos, mask, rim;
            draw(0u, s, pos, mask, rim);
#pragma unroll 4
            for (uint32_t rho = 0; rho < 64u; ++rho) {
                uint32_t sn, posn, maskn, rimn;
                if (SCHEME != kDB) {
                    try_site(s, mask, act);
                    draw(rho + 1u, sn, posn, maskn, rimn);
                } else {
                    // delayed borders, as in db_round: in one wave every order is program order
                    const uint32_t pr = (uint32_t)__builtin_amdgcn_ds_bpermute(right, (int)pos);
                    const uint32_t pd = (uint32_t)__builtin_amdgcn_ds_bpermute(below, (int)pos);
                    const bool def = act && (((rim & 1u) && pr == pos + 1u) || ((rim & 2u) && pd == pos + 0x10000u));
                    try_site(s, mask, act && !def);
                    draw(rho + 1u, sn, posn, maskn, rimn);
                    if (__ballot(def)) {
                        wave_order();
                        try_site(s, mask, def && rim != 3u);
                        wave_order();
                        try_site(s, mask, def && rim == 3u);
                    }
                }
                wave_order();
                s = sn;
                pos = posn;
                mask = maskn;
                rim = rimn;
            }
        }
    }
    for (uint32_t t = lane; t < halves; t += 64u) {
        const uint32_t *p = (t & 1u) ? sy : sx;
        reinterpret_cast<uint4 *>(A.words)[t] = make_uint4(p[lds_of(t, 0)], p[lds_of(t, 1)], p[lds_of(t, 2)], p[lds_of(t, 3)]);
    }
}

}  // namespace okpz
