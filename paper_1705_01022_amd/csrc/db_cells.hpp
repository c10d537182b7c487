// DB device step with one cell per lane (square domains of 128 or 256 sites,
// 8 x 8-site cells), for steps with few tiles: then a tile has a compute unit
// to itself and a step takes 64 rounds one after the other, each a chain of
// LDS round trips and barriers.  Same attempts, random draws and delayed-border
// order as sweep_db_rows, on the same row-paired window; what differs shortens
// the round:
//
//  * 16 waves (D = 256) instead of 8 or 4 hide each other's latency.
//  * A wave holds 8 x 8 cells, so that a quarter of the cells, not half, have a
//    neighbour that they may wait for in another wave.
//  * Draws do not depend on the lattice: while a round's slope words are on
//    their way from LDS, the next round's dependencies are worked out and the
//    sites of the round after it drawn and published (every lane publishes
//    its own and reads its two neighbours').
//
// us a step, two cells per lane in the row-paired kernel against this, p = 0.7:
// D = 256, one tile 60.8 and 51.2, 64 tiles 63.5 and 53.0; D = 128, four tiles 46.7
// and 32.2, 256 tiles 48.6 and 33.6.  A round is then about 0.7 us: the waves'
// LDS and vector phases, 0.3 us each, fall together between barriers.  With
// more tiles than compute units the row-paired kernel's smaller workgroups
// win (1024 tiles of D = 256: 128 us against 226; 4096 of D = 128: 125 against 129).
#pragma once

#include "db_rows.hpp"

namespace okpz {

// Window as RowPairShape's, at the smallest pitch (LDS is not what limits a tile
// that is alone): cell rows, 8 window rows apart, fall on the bank offsets 0, 24, 16, 8.
template <int LD>
struct CellLaneShape {
    static constexpr uint32_t D = 1u << LD;
    static constexpr uint32_t NWX = D / 32 + 1, NB = D / 4 + 1, NR = 4 * NB;
    static constexpr uint32_t P = NWX | 1u;
    static constexpr uint32_t PITCH = 2 * P + 1;
    static constexpr uint32_t ROW = 32 * PITCH;  // bits per window row
    static constexpr uint32_t NCX = D / 8, LOG2NCX = LD - 3;
    static constexpr uint32_t NT = NCX * NCX;    // lanes
    static constexpr uint32_t WORDS = NR * PITCH;
    static constexpr uint32_t LDS_WORDS = WORDS + 2 * NT + 4;
};

template <bool ACCEPT, int LD, bool SHARED>
__device__ __forceinline__ void sweep_db_cells(const StepArgs &A, uint32_t *smem, uint32_t tile)
{
    using S = CellLaneShape<LD>;
    constexpr uint32_t P = S::P, PITCH = S::PITCH, NT = S::NT;
    constexpr uint32_t F = ACCEPT ? 16u : 8u, RPB = 128u / F, FPW = 32u / F;
    uint32_t tid = threadIdx.x;
    if (SHARED) asm volatile("" : "+v"(tid));
    uint32_t *lds = smem;
    uint32_t *pos = smem + S::WORDS;   // 2 x NT published sites
    uint32_t *flags = pos + 2u * NT;   // 4 round flags: 1 remote edges, 2 remote corners

    const uint32_t tx = tile & ((1u << A.log2ntx) - 1u), ty = tile >> A.log2ntx;
    const uint32_t X0 = (A.ox + 2u * S::D * tx + A.set_a * S::D) & A.L_mask;
    const uint32_t Y0 = (A.oy + 2u * S::D * ty + A.set_b * S::D) & A.L_mask;
    const uint32_t origin = (Y0 & 3u) * S::ROW + (X0 & 31u) + 8u * lds_address(lds);

    load_window_rows<S, NT, SHARED>(A, lds, X0 >> 5, Y0 >> 2);

    // a wave holds 8 x 8 cells
    constexpr uint32_t LOG2WX = S::LOG2NCX - 3u, WXM = (1u << LOG2WX) - 1u;
    const uint32_t lane = tid & 63u, wave = tid >> 6;
    const uint32_t cx = (wave & WXM) * 8u + (lane & 7u), cy = (wave >> LOG2WX) * 8u + (lane >> 3);
    auto slot_of = [](uint32_t x, uint32_t y) {
        x &= S::NCX - 1u;
        y &= S::NCX - 1u;
        return (((y >> 3) << LOG2WX | x >> 3) << 6) | (y & 7u) << 3 | (x & 7u);
    };
    const uint32_t right = slot_of(cx + 1u, cy), below = slot_of(cx, cy + 1u);
    const bool last_x = (lane & 7u) == 7u, last_y = (lane >> 3) == 7u;  // the neighbour is in another wave
    const uint32_t base_u = cx << 3, base_v = cy << 3, cell = cy * S::NCX + cx;

    // the block draws of all rounds: lane b holds those of rounds 8 b .. 8 b + 7
    const u32x4 bw = block_draws(A, tile);
    uint32_t r0 = 0u, r1 = 0u, r2 = 0u, r3 = 0u;  // what is left of the cell's current Philox block
    // the draw of round 8 b + k (in order; k known when compiled): its field and site
    auto draw = [&](uint32_t b, auto kc, uint32_t &f, uint32_t &s) {
        constexpr uint32_t K = decltype(kc)::value;
        if constexpr (RPB == 8u || K == 0u) {
            if (K == 0u && (RPB == 8u || (b & 1u) == 0u)) {
                const u32x4 r = philox4x32_10_lane(A.key0, A.key1, RPB == 8u ? b : b >> 1, cell, tile, A.c3);
                r0 = r.x; r1 = r.y; r2 = r.z; r3 = r.w;
            }
        }
        f = __builtin_amdgcn_ubfe(r0, (K % FPW) * F, F);
        if constexpr (K % FPW == FPW - 1u) {
            r0 = r1;
            r1 = r2;
            r2 = r3;
        }
        const uint32_t w = K / 2u == 0u ? bw.x : (K / 2u == 1u ? bw.y : (K / 2u == 2u ? bw.z : bw.w));
        const uint32_t f16 = (uint32_t)__builtin_amdgcn_readlane((int)w, (int)(b & 7u)) >> (16u * (K & 1u));
        const uint32_t u = wrap_column<LD>(f & 7u, base_u + ((f16 >> 2) & 7u));
        const uint32_t v = (((f >> 3) & 7u) + base_v + ((f16 >> 8) & 7u)) & (S::D - 1u);
        s = mad24(v, S::ROW, u) + origin;
    };
    auto corner_of = [](uint32_t f) { return (f & 63u) == 63u; };
    // A deferred attempt whose rim touches another wave's cells is remote: what
    // it waits for may be done only after the barrier.  What waits for a remote
    // attempt is a corner on the same rim, so it is remote too, and later.
    auto remote_of = [&](uint32_t f) { return (last_x && (f & 7u) == 7u) || (last_y && (f & 56u) == 56u); };

    uint32_t f0, s0, f1, s1;
    draw(0u, std::integral_constant<uint32_t, 0>(), f0, s0);
    pos[tid] = s0;
    draw(0u, std::integral_constant<uint32_t, 1>(), f1, s1);
    pos[NT + tid] = s1;
    if (tid < 4u) flags[tid] = 0u;
    __syncthreads();
    bool def = pos[right] == s0 + 1u || pos[below] == s0 + S::ROW;
    bool rem = def && remote_of(f0);
    auto publish = [&](uint32_t slot, bool r, uint32_t f) {
        const uint64_t edges = __ballot(r && !corner_of(f)), corners = __ballot(r && corner_of(f));
        if (lane == 0u && (edges | corners)) atomicOr(&flags[slot], (edges ? 1u : 0u) | (corners ? 2u : 0u));
    };
    publish(0u, rem, f0);
    __syncthreads();

    auto round = [&](uint32_t b, auto kc) {
        constexpr uint32_t K = decltype(kc)::value;
        const uint32_t rho = 8u * b + K;
        const SlopeWords v = read_rows<P, PITCH>(s0);
        const uint32_t nbuf = ((rho + 1u) & 1u) * NT;
        const uint32_t pr = pos[nbuf + right], pd = pos[nbuf + below];
        const uint32_t flag = flags[rho & 3u];
        __builtin_amdgcn_sched_barrier(0);
        uint32_t f2, s2;
        draw(K >= 6u ? b + 1u : b, std::integral_constant<uint32_t, (K + 2u) % 8u>(), f2, s2);
        pos[(rho & 1u) * NT + tid] = s2;
        const bool def1 = pr == s1 + 1u || pd == s1 + S::ROW;
        const bool rem1 = def1 && remote_of(f1);
        decide_rows<ACCEPT, P, PITCH>(A, v, s0, f0 >> 6, !def, rho, cell, tile);
        const bool local = def && !rem;
        if (__ballot(local)) {  // deferred attempts of this wave: edges, then corners
            wave_order();
            const bool cor = corner_of(f0);
            if (local && !cor) attempt_rows<ACCEPT, P, PITCH>(A, s0, f0 >> 6, true, rho, cell, tile);
            wave_order();
            if (local && cor) attempt_rows<ACCEPT, P, PITCH>(A, s0, f0 >> 6, true, rho, cell, tile);
        }
        publish((rho + 1u) & 3u, rem1, f1);
        if (tid == 0u) flags[(rho + 2u) & 3u] = 0u;
        __syncthreads();
        const uint32_t fl = (uint32_t)__builtin_amdgcn_readfirstlane((int)flag);
        if (fl) {  // those that wait for another wave's: edges, then corners
            const bool cor = corner_of(f0);
            if (rem && !cor) attempt_rows<ACCEPT, P, PITCH>(A, s0, f0 >> 6, true, rho, cell, tile);
            if (fl & 2u) {
                __syncthreads();
                if (rem && cor) attempt_rows<ACCEPT, P, PITCH>(A, s0, f0 >> 6, true, rho, cell, tile);
            }
            __syncthreads();
        }
        f0 = f1;
        s0 = s1;
        f1 = f2;
        s1 = s2;
        def = def1;
        rem = rem1;
    };
#pragma unroll 1
    for (uint32_t b = 0; b < 8u; ++b) {
        round(b, std::integral_constant<uint32_t, 0>());
        round(b, std::integral_constant<uint32_t, 1>());
        round(b, std::integral_constant<uint32_t, 2>());
        round(b, std::integral_constant<uint32_t, 3>());
        round(b, std::integral_constant<uint32_t, 4>());
        round(b, std::integral_constant<uint32_t, 5>());
        round(b, std::integral_constant<uint32_t, 6>());
        round(b, std::integral_constant<uint32_t, 7>());
    }
    store_window_rows<S, NT, SHARED>(A, lds, X0 >> 5, Y0 >> 2);
}

template <bool ACCEPT, int LD>
__global__ void __launch_bounds__(CellLaneShape<LD>::NT) step_db_cells_kernel(StepArgs A)
{
    extern __shared__ uint32_t smem[];
    sweep_db_cells<ACCEPT, LD, false>(A, smem, blockIdx.x);
}

}  // namespace okpz
