// DT device step with the domain in registers (square domains of 128 or 256
// sites, 8 x 8-site cells).  Same attempts and random draws as sweep_tile's DT
// path (Sec. 3 DT at block level, Sec. 3.1 single hit); the domain's state and
// the way a round tests it differ:
//
//  * One bit per site.  v(x, y) = ((h(x, y) - x - y) / 2) mod 2 (in a gauge of
//    the tile): v keeps its value along an up step (slope bit 1) and changes
//    along a down step.  An attempt's site is a local minimum iff
//    v(left) = v(above) != v = v(right) = v(below), a local maximum iff
//    v(left) = v(above) = v != v(right) = v(below), and either flip is the flip
//    of this one bit.
//  * Cells in registers.  Under DT the cell grid stands still and a round's
//    attempts all lie in the same quadrant of their cells, so a lane keeps a
//    stack of cells, two to a register: register [pair][qx][qy] holds the
//    4 x 4 sites of quadrant (qx, qy) of one cell in its low half and of the
//    cell half a stack further down in its high half, bit 4 row + column, which
//    is the order of the lane draw's site index.  A round forms the four
//    neighbours of all 32 sites by shifts (the neighbouring quadrants are other
//    registers of the lane, of the lane beside it, or of the lane row above or
//    below), tests them all at once and lets the drawn sites' bits through:
//    17 instructions for two attempts, no LDS and, inside a wave, no barrier.
//    Column -1, column D, row -1 and row D never change during the step.
//  * Random fields two cells to a register in the same halves: the drawn
//    sites' bits are one packed 16-bit shift, the acceptance masks a packed
//    subtraction and sign.
//
// The step is bound by vector issue (the counters read 100 % busy at p = 1,
// 89 % with draws, where two waves' 132 registers leave three waves a SIMD), where
// the row-paired LDS kernel it replaces was bound by LDS and issue together
// (73 % and 69 %).  D = 256, L = 2^16, a launch among many, rows against this: p = 1
// 0.845 and 0.394 ms (28.6 and 14.6 VALU instructions per wave-attempt), p = 0.95
// 0.924 and 0.777 (25.0 instructions); D = 128 p = 1 0.89 and 0.44 ms, p = 1/2 0.95
// and 0.63; 64 tiles (L = 4096), p = 1 31.3 and 23.2 us.  With few tiles and draws
// the row-paired kernel is faster and taken (dt_rows_few).  Two waves per tile
// rather than one (which needs no barrier and fewer instructions): a single
// wave holds 16 cells a lane, 168 registers with spills, three waves per
// SIMD, and took 0.51 ms a launch where two took 0.435 (0.97 with draws).
#pragma once

#include "kernels.hpp"

namespace okpz {

// How a round decides: every deposition and no removal (p = 1, q = 0), other
// rates of 0 and 1, or acceptance draws.
enum : int { kDeposit = 0, kSure = 1, kDraw = 2 };

// D = 2^LD sites a side, NW waves per tile.
template <int LD, int NW>
struct CellShape {
    static constexpr uint32_t D = 1u << LD;
    static constexpr uint32_t NCX = D / 8;             // cells per domain row: lanes side by side
    static constexpr uint32_t LOG2NCX = LD - 3;
    static constexpr uint32_t GPW = 64 / NCX;          // lane rows of a wave
    static constexpr uint32_t NG = GPW * NW;           // lane rows of the tile
    static constexpr uint32_t CPT = NCX / NG;          // cells stacked in a lane
    static constexpr int NP = (int)CPT / 2;            // pairs of them
    static constexpr uint32_t KW = D / 32;             // 32-site words of a domain row
    static constexpr uint32_t NWX = KW + 1, NB = D / 4 + 1;  // window blocks and bands
    static constexpr uint32_t PITCH = KW + 2;          // LDS row: word -1, the KW words, word KW
    static constexpr uint32_t PLANE = PITCH * (D + 2);  // rows -1 .. D
    static constexpr uint32_t TABLE = 3 * 64;          // per row quad: column 0, left and right halo
    static constexpr uint32_t EDGE = NW > 1 ? 4 * NW * NCX : 0;
    static constexpr uint32_t LDS_WORDS = PLANE + TABLE + EDGE;
    static_assert(NP >= 1 && CPT % 2 == 0, "a lane holds pairs of cells");
};

typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// a >> N and a << amounts in each 16-bit half (amounts mod 16)
template <int N>
__device__ __forceinline__ uint32_t pk_shr(uint32_t a)
{
    uint32_t r;
    asm("v_pk_lshrrev_b16 %0, %1, %2 op_sel_hi:[0,1]" : "=v"(r) : "n"(N), "v"(a));
    return r;
}

// bit (amount mod 16) of each half
__device__ __forceinline__ uint32_t pk_bit(uint32_t amount)
{
    uint32_t r;
    asm("v_pk_lshlrev_b16 %0, %1, 1 op_sel_hi:[1,0]" : "=v"(r) : "v"(amount));
    return r;
}

// a * b + c in each half; b a uniform constant in both halves
__device__ __forceinline__ uint32_t pk_mad16(uint32_t a, uint32_t b, uint32_t c)
{
    uint32_t r;
    asm("v_pk_mad_u16 %0, %1, %2, %3" : "=v"(r) : "v"(a), "s"(b), "v"(c));
    return r;
}

__device__ __forceinline__ uint32_t pk_sub16(uint32_t a, uint32_t b)
{
    uint32_t r;
    asm("v_pk_sub_i16 %0, %1, %2" : "=v"(r) : "v"(a), "s"(b));
    return r;
}

// the sign of each half as a mask
__device__ __forceinline__ uint32_t pk_sign(uint32_t a)
{
    uint32_t r;
    asm("v_pk_ashrrev_i16 %0, 15, %1 op_sel_hi:[0,1]" : "=v"(r) : "v"(a));
    return r;
}

__device__ __forceinline__ uint32_t pk_min16(uint32_t a, uint32_t b)
{
    uint32_t r;
    asm("v_pk_min_u16 %0, %1, %2" : "=v"(r) : "v"(a), "v"(b));
    return r;
}

// f(a, b, c) bit by bit, f given by its truth table (bit 4a + 2b + c)
template <uint32_t TT>
__device__ __forceinline__ uint32_t bit3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, TT);
}

// m ? a : b, bit by bit
__device__ __forceinline__ uint32_t select_bits(uint32_t m, uint32_t a, uint32_t b) { return bit3<0xCA>(m, a, b); }

// the value of the lane one to the left / to the right (of the wave)
__device__ __forceinline__ uint32_t from_left(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x138, 0xF, 0xF, true);  // wave_shr:1
}

__device__ __forceinline__ uint32_t from_right(uint32_t v)
{
    return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x130, 0xF, 0xF, true);  // wave_shl:1
}

// the value of the lane row above / below (lane -+ 64 / GPW); g the lane's row
template <uint32_t GPW>
__device__ __forceinline__ uint32_t from_above(uint32_t v, uint32_t g)
{
    if constexpr (GPW == 2) {
        return __builtin_amdgcn_permlane32_swap(v, v, false, false)[0];
    } else {
        const u32x2 ab = __builtin_amdgcn_permlane16_swap(v, v, false, false);  // rows 0 0 2 2, 1 1 3 3
        const uint32_t c = __builtin_amdgcn_permlane32_swap(ab[1], ab[1], false, false)[0];  // row 1 everywhere
        return g == 2u ? c : ab[0];
    }
}

template <uint32_t GPW>
__device__ __forceinline__ uint32_t from_below(uint32_t v, uint32_t g)
{
    if constexpr (GPW == 2) {
        return __builtin_amdgcn_permlane32_swap(v, v, false, false)[1];
    } else {
        const u32x2 ab = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        const uint32_t c = __builtin_amdgcn_permlane32_swap(ab[0], ab[0], false, false)[1];  // row 2 everywhere
        return g == 1u ? c : ab[1];
    }
}

// 4 x 4 byte transposition over the four lanes of a quad: byte m of lane i
// becomes byte i of lane m (s1, s2: the lane's selectors).
__device__ __forceinline__ uint32_t quad_transpose(uint32_t w, uint32_t s1, uint32_t s2)
{
    uint32_t t = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0xB1, 0xF, 0xF, true);  // quad_perm 1 0 3 2
    w = __builtin_amdgcn_perm(t, w, s1);
    t = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)w, 0x4E, 0xF, 0xF, true);  // quad_perm 2 3 0 1
    return __builtin_amdgcn_perm(t, w, s2);
}

// swaps the middle nibbles of both halves
__device__ __forceinline__ uint32_t swap_nibbles(uint32_t x)
{
    const uint32_t t = bit3<0x28>(x >> 4, x, 0x00F000F0u);  // (a ^ b) & c
    return bit3<0x96>(x, t, t << 4);
}

// running XOR over the bits of a word, lowest first
__device__ __forceinline__ uint32_t running_xor(uint32_t x)
{
    x ^= x << 1;
    x ^= x << 2;
    x ^= x << 4;
    x ^= x << 8;
    return x ^ (x << 16);
}

template <int MODE, int LD, int NW, bool SHARED>
__device__ __forceinline__ void sweep_dt_cells(const StepArgs &A, uint32_t *smem, uint32_t tile)
{
    using S = CellShape<LD, NW>;
    constexpr int NP = S::NP;
    constexpr uint32_t KW = S::KW, NCX = S::NCX, PITCH = S::PITCH;
    uint32_t *plane = smem;                  // v, rows -1 .. D, words -1 .. KW
    uint32_t *table = smem + S::PLANE;
    uint32_t *edge_a = table + S::TABLE;     // last row of cells of each wave, by quadrant column
    uint32_t *edge_b = edge_a + 2 * NW * NCX;  // first row of cells of each wave
    // opaque: in the batch kernel's loop the compiler otherwise keeps what it
    // derives from the lane's number in registers across all items
    uint32_t tid = threadIdx.x;
    if (SHARED) asm volatile("" : "+v"(tid));
    const uint32_t lane = tid & 63u;
    const uint32_t wave = NW > 1 ? (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid >> 6)) : 0u;
    const uint32_t cx = lane & (NCX - 1u), g = lane >> S::LOG2NCX, G = wave * S::GPW + g;
    const uint32_t i = cx & 3u, k = cx >> 2;  // place in the quad, word column
    const uint32_t tx = tile & ((1u << A.log2ntx) - 1u), ty = tile >> A.log2ntx;
    const uint32_t X0 = (A.ox + 2u * S::D * tx + A.set_a * S::D) & A.L_mask;
    const uint32_t Y0 = (A.oy + 2u * S::D * ty + A.set_b * S::D) & A.L_mask;
    const uint32_t offx = X0 & 31u, offy = Y0 & 3u, bx0 = X0 >> 5, by0 = Y0 >> 2;
    const uint32_t band_log2 = A.nbx_log2 + 5u;  // bytes of a band; the lattice is at most 2^32 bytes
    char *const base = reinterpret_cast<char *>(A.words);
    auto word_at = [&](uint32_t off) { return load_word<SHARED>(base + off); };
    auto block_off = [&](uint32_t kk) { return ((bx0 + kk) & A.nbx_mask) << 5; };

    // ---- loads, all in flight together: columns 0 and D of the row quads 4 l .. 4 l + 3 (lane l), row 0,
    // the row the lane's first one is reached from, the sy words of the lane's rows (the four lanes of a quad
    // take the four rows of a row quad), and the row past the domain
    const uint32_t lq = lane & (S::D / 4u - 1u);  // the upper lanes of D = 128 repeat the lower ones' loads
    const uint32_t q0 = 2u * G * S::CPT;          // the lane's first row quad
    const uint32_t row0 = ((Y0 >> 2) << band_log2) + ((Y0 & 3u) << 2);
    const uint32_t kb0 = block_off(k), kb1 = block_off(k + 1u);
    uint32_t c0x[4], c0y[4], cdy[4], across, first[2], sy0[2], syd[2], sy[2 * S::CPT][2];
    const uint32_t from = G == 0u ? 0u : 4u * q0 - 1u;
    {
        const char *const col0 = base + block_off(0u), *const cold = base + block_off(KW);
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            const uint32_t off = ((lq + ((Y0 + r) >> 2)) & A.nby_mask) << band_log2, srow = ((Y0 + r) & 3u) << 2;
            c0x[r] = load_word<SHARED>(col0 + srow + off);
            c0y[r] = load_word<SHARED>(col0 + (srow + 16u) + off);
            cdy[r] = load_word<SHARED>(cold + (srow + 16u) + off);
        }
        across = word_at(row0 + block_off(min(lane, KW)));
        const uint32_t yf = (Y0 + from) & A.L_mask;
        const uint32_t off = ((yf >> 2) << band_log2) + ((yf & 3u) << 2);
        first[0] = word_at(off + kb0);
        first[1] = word_at(off + kb1);
        sy0[0] = word_at(row0 + 16u + kb0);
        sy0[1] = word_at(row0 + 16u + kb1);
        const uint32_t band0 = ((Y0 + i) >> 2) + q0, rowb = (((Y0 + i) & 3u) << 2) + 16u;
        const uint32_t o0 = rowb + kb0, o1 = rowb + kb1;
#pragma unroll
        for (uint32_t b = 0; b < 2u * S::CPT; ++b) {
            const uint32_t bo = ((band0 + b) & A.nby_mask) << band_log2;
            sy[b][0] = word_at(bo + o0);
            sy[b][1] = word_at(bo + o1);
        }
        const uint32_t yd = (Y0 + S::D) & A.L_mask;
        const uint32_t offd = ((yd >> 2) << band_log2) + ((yd & 3u) << 2) + 16u;
        syd[0] = word_at(offd + kb0);
        syd[1] = word_at(offd + kb1);
    }

    // ---- v in columns 0, -1 and D
    {
        uint32_t nx = 0u, ny = 0u, nd = 0u;
#pragma unroll
        for (uint32_t r = 0; r < 4; ++r) {
            nx |= __builtin_amdgcn_ubfe(c0x[r], offx, 1) << r;
            ny |= __builtin_amdgcn_ubfe(c0y[r], offx, 1) << r;
            nd |= __builtin_amdgcn_ubfe(cdy[r], offx, 1) << r;
        }
        // down a column from 0 in row 0: a step of the surface up keeps v
        auto down = [&](uint32_t n) {
            uint32_t e = ~n & 15u;
            if (lane == 0u) e &= ~1u;
            e ^= e << 1;
            e = (e ^ (e << 2)) & 15u;
            uint64_t s = __ballot((e & 8u) != 0u);
            s ^= s << 1;
            s ^= s << 2;
            s ^= s << 4;
            s ^= s << 8;
            s ^= s << 16;
            s ^= s << 32;
            return __builtin_amdgcn_inverse_ballot_w64(s << 1) ? e ^ 15u : e;
        };
        const uint32_t n0 = down(ny);
        // v(D, 0) from v(0, 0) along row 0
        if (lane == 0u) across &= (~0u << offx) << 1;
        if (lane == KW) across &= (2u << offx) - 1u;
        const uint64_t odd = __ballot(lane <= KW && (__popc(across) & 1) != 0);
        const uint32_t nr = down(nd) ^ (((uint32_t)__popcll(odd) & 1u) ? 15u : 0u);
        const uint32_t nl = n0 ^ nx ^ 15u;
        auto spread = [](uint32_t n) { return (n & 1u) | (n & 2u) << 3 | (n & 4u) << 6 | (n & 8u) << 9; };
        if (lane < S::D / 4u) {
            table[lane] = n0;
            table[64u + lane] = spread(nl) << 3;
            table[128u + lane] = spread(nr);
#pragma unroll
            for (uint32_t r = 0; r < 4; ++r) {
                plane[(4u * lane + r + 1u) * PITCH] = nl << (31u - r);
                plane[(4u * lane + r + 1u) * PITCH + KW + 1u] = nr >> r;
            }
        }
        wave_order();
    }

    // ---- the lane's cells
    const uint32_t s1 = (i & 1u) ? 0x03070105u : 0x06020400u;
    const uint32_t s2 = (i & 2u) ? 0x03020706u : 0x05040100u;
    uint32_t q[NP][2][2];  // [pair][quadrant column][quadrant row]
    uint32_t halo[NP][2];  // column -1 (lanes of the first column) or D (of the last)
    uint32_t vhalo[2];     // by quadrant column: row -1 in bits 28-31, row D in bits 0-3
    {
        // the row above the lane's first one, along the row from column 0
        constexpr uint64_t seg4 = NCX == 32 ? 0xFFFFFFF0FFFFFFF0ull : 0xFFF0FFF0FFF0FFF0ull;
        constexpr uint64_t seg8 = NCX == 32 ? 0xFFFFFF00FFFFFF00ull : 0xFF00FF00FF00FF00ull;
        const uint32_t a = running_xor(__builtin_amdgcn_alignbit(first[1], first[0], offx) & (k == 0u ? ~1u : ~0u));
        uint64_t s = __ballot((int)a < 0);
        s ^= (s << 4) & seg4;
        s ^= (s << 8) & seg8;
        if (NCX == 32) s ^= (s << 16) & 0xFFFF0000FFFF0000ull;
        s = (s << 4) & seg4;
        const uint32_t c = __builtin_amdgcn_inverse_ballot_w64(s) ? 0x55555555u : 0xAAAAAAAAu;
        uint32_t v = bit3<0x96>(a, c, (uint32_t)__builtin_amdgcn_sbfe((int)table[from >> 2], from & 3u, 1));
        if (G == 0u) v = ~(v ^ __builtin_amdgcn_alignbit(sy0[1], sy0[0], offx));
        const uint32_t top = (v >> (8u * i)) & 255u;
        // then down the rows: byte r of p is the lane's eight columns of row r of the quad
        uint32_t prev = v << (24u - 8u * i);
        uint32_t p[2 * S::CPT];
#pragma unroll
        for (uint32_t b = 0; b < 2u * S::CPT; ++b) {
            uint32_t x = quad_transpose(__builtin_amdgcn_alignbit(sy[b][1], sy[b][0], offx), s1, s2);
            x ^= x << 8;
            x ^= x << 16;
            prev = bit3<0x96>(x, __builtin_amdgcn_perm(prev, prev, 0x07070707u), 0x00FF00FFu);
            p[b] = swap_nibbles(prev);
        }
        const uint32_t bot = ~((prev >> 24) ^ (__builtin_amdgcn_alignbit(syd[1], syd[0], offx) >> (8u * i))) & 255u;
        uint8_t *bytes = reinterpret_cast<uint8_t *>(plane);
        if (G == 0u) bytes[4u + cx] = (uint8_t)top;
        if (G == S::NG - 1u) bytes[4u * ((S::D + 1u) * PITCH + 1u) + cx] = (uint8_t)bot;
        vhalo[0] = top << 28 | (bot & 15u);
        vhalo[1] = (top >> 4) << 28 | bot >> 4;
        const uint32_t htab = (cx == NCX - 1u ? 128u : 64u) + q0;
#pragma unroll
        for (int j = 0; j < NP; ++j)
#pragma unroll
            for (int qy = 0; qy < 2; ++qy) {
                const uint32_t lo = p[2 * j + qy], hi = p[2 * (j + NP) + qy];
                q[j][0][qy] = __builtin_amdgcn_perm(hi, lo, 0x06040200u);
                q[j][1][qy] = __builtin_amdgcn_perm(hi, lo, 0x07050301u);
                halo[j][qy] = table[htab + 2u * (uint32_t)j + (uint32_t)qy] |
                              table[htab + 2u * (uint32_t)(j + NP) + (uint32_t)qy] << 16;
            }
    }
    if (NW > 1) {
#pragma unroll
        for (uint32_t qx = 0; qx < 2; ++qx) {
            if (g == S::GPW - 1u) edge_a[(qx * NW + wave) * NCX + cx] = q[NP - 1][qx][1];
            if (g == 0u) edge_b[(qx * NW + wave) * NCX + cx] = q[0][qx][0];
        }
        __syncthreads();
    }

    // ---- the rounds
    const bool first_col = cx == 0u, last_col = cx == NCX - 1u;
    uint32_t site[NP], take_p[NP], take_q[NP];
    auto round = [&](auto qxc, auto qyc) {
        constexpr uint32_t QX = decltype(qxc)::value, QY = decltype(qyc)::value;
        // the row of cells above / below the lane's, for its first or last pair
        uint32_t other;
        if (QY == 0) {
            const uint32_t e = NW > 1 && wave > 0u ? edge_a[(QX * NW + wave - 1u) * NCX + cx] : vhalo[QX];
            const uint32_t x = from_above<S::GPW>(q[NP - 1][QX][1], g);
            other = __builtin_amdgcn_alignbit(q[NP - 1][QX][1], g == 0u ? e : x, 16);
        } else {
            const uint32_t e = NW > 1 && wave + 1u < NW ? edge_b[(QX * NW + wave + 1u) * NCX + cx] : vhalo[QX];
            const uint32_t x = from_below<S::GPW>(q[0][QX][0], g);
            other = __builtin_amdgcn_alignbit(g == S::GPW - 1u ? e : x, q[0][QX][0], 16);
        }
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const uint32_t v = q[j][QX][QY], side = q[j][1 - QX][QY];
            uint32_t left, right;
            if (QX == 0) {
                const uint32_t n = from_left(side);
                left = first_col ? halo[j][QY] : n;
                right = side;
            } else {
                const uint32_t n = from_right(side);
                left = side;
                right = last_col ? halo[j][QY] : n;
            }
            const uint32_t above = QY == 1 ? q[j][QX][0] : (j > 0 ? q[j > 0 ? j - 1 : 0][QX][1] : other);
            const uint32_t below = QY == 0 ? q[j][QX][1] : (j < NP - 1 ? q[j < NP - 1 ? j + 1 : j][QX][0] : other);
            const uint32_t l = select_bits(0x11111111u, left >> 3, v << 1);
            const uint32_t r = select_bits(0x88888888u, right << 3, v >> 1);
            const uint32_t u = pk_mad16(v, 0x00100010u, pk_shr<12>(above));
            const uint32_t d = pk_mad16(below, 0x10001000u, pk_shr<4>(v));
            // extremal: l = u, r = d = not l
            const uint32_t x = bit3<0x42>(l, u, r);           // l == u and r != l
            const uint32_t y = bit3<0x28>(d, l, site[j]);     // d != l, at the drawn site
            if (MODE == kDeposit) {
                q[j][QX][QY] = select_bits(x & y, l, v);  // a minimum becomes a maximum (v = l), a maximum is one
            } else {
                const uint32_t m = select_bits(v ^ r, take_q[j], take_p[j]);  // a maximum has v != r
                q[j][QX][QY] = bit3<0x78>(v, x & y, m);                       // v ^ (b & c)
            }
        }
        if (NW > 1) {
            if (QY == 1 && g == S::GPW - 1u) edge_a[(QX * NW + wave) * NCX + cx] = q[NP - 1][QX][1];
            if (QY == 0 && g == 0u) edge_b[(QX * NW + wave) * NCX + cx] = q[0][QX][0];
            __syncthreads();
        }
    };
    auto any_round = [&](uint32_t sigma) {
        switch (sigma) {
        case 0: round(std::integral_constant<uint32_t, 0>(), std::integral_constant<uint32_t, 0>()); break;
        case 1: round(std::integral_constant<uint32_t, 1>(), std::integral_constant<uint32_t, 0>()); break;
        case 2: round(std::integral_constant<uint32_t, 0>(), std::integral_constant<uint32_t, 1>()); break;
        default: round(std::integral_constant<uint32_t, 1>(), std::integral_constant<uint32_t, 1>()); break;
        }
    };
    if (MODE == kSure) {
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            take_p[j] = (A.flip_table & kFlipMin) ? ~0u : 0u;
            take_q[j] = (A.flip_table & kFlipMax) ? ~0u : 0u;
        }
    }
    const uint32_t cell0 = G * S::CPT * NCX + cx;
    constexpr uint32_t RPB = MODE == kDraw ? 8u : 32u;  // rounds of one Philox block
    BlockDraw bd = {0u, 0u, 0u, 0u};
    const u32x4 draws = block_draws(A, tile);
#pragma unroll 1
    for (uint32_t blk = 0; blk < 64u / RPB; ++blk) {
        uint32_t rnd[NP][8];  // 16 bits of the pair's two cells each
#pragma unroll
        for (int j = 0; j < NP; ++j) {
            const u32x4 a = philox4x32_10_lane(A.key0, A.key1, blk, cell0 + (uint32_t)j * NCX, tile, A.c3);
            const u32x4 b = philox4x32_10_lane(A.key0, A.key1, blk, cell0 + (uint32_t)(j + NP) * NCX, tile, A.c3);
            const uint32_t wa[4] = {a.x, a.y, a.z, a.w}, wb[4] = {b.x, b.y, b.z, b.w};
#pragma unroll
            for (int m = 0; m < 4; ++m) {
                rnd[j][2 * m] = __builtin_amdgcn_perm(wb[m], wa[m], 0x05040100u);
                rnd[j][2 * m + 1] = __builtin_amdgcn_perm(wb[m], wa[m], 0x07060302u);
            }
        }
#pragma unroll 1
        for (uint32_t r = 0; r < 8u; ++r) {
            uint32_t cur[NP];
            auto fetch = [&](auto rc) {
                constexpr int R = decltype(rc)::value;
#pragma unroll
                for (int j = 0; j < NP; ++j) cur[j] = rnd[j][R];
            };
            switch (r) {
            case 0: fetch(std::integral_constant<int, 0>()); break;
            case 1: fetch(std::integral_constant<int, 1>()); break;
            case 2: fetch(std::integral_constant<int, 2>()); break;
            case 3: fetch(std::integral_constant<int, 3>()); break;
            case 4: fetch(std::integral_constant<int, 4>()); break;
            case 5: fetch(std::integral_constant<int, 5>()); break;
            case 6: fetch(std::integral_constant<int, 6>()); break;
            default: fetch(std::integral_constant<int, 7>()); break;
            }
            if constexpr (MODE != kDraw) {
#pragma unroll 1
                for (uint32_t n = 0; n < 4u; ++n) {
                    const uint32_t rho = (blk * 8u + r) * 4u + n;
                    const uint32_t f16 = next_block_field(draws, bd, rho);
#pragma unroll
                    for (int j = 0; j < NP; ++j) {
                        site[j] = pk_bit(cur[j]);
                        cur[j] >>= 4;
                    }
                    any_round((uint32_t)__builtin_amdgcn_readfirstlane((int)(f16 & 3u)));
                }
            } else {
                const uint32_t rho = blk * 8u + r;
                const uint32_t f16 = next_block_field(draws, bd, rho);
                const uint32_t pp = A.P_hi | A.P_hi << 16, qq = A.Q_hi | A.Q_hi << 16;
                uint32_t tie = ~0u;
#pragma unroll
                for (int j = 0; j < NP; ++j) {
                    site[j] = pk_bit(cur[j]);
                    const uint32_t pre = pk_shr<4>(cur[j]);
                    const uint32_t dp = pk_sub16(pre, pp), dq = pk_sub16(pre, qq);
                    take_p[j] = pk_sign(dp);
                    take_q[j] = pk_sign(dq);
                    tie = pk_min16(tie, pk_min16(dp, dq));
                }
                // a prefix equal to a threshold's: the low 32 bits of the variate decide
                if ((A.P_lo | A.Q_lo) != 0u && __ballot((tie & 0xFFFFu) == 0u || (tie >> 16) == 0u)) {
#pragma unroll
                    for (int j = 0; j < NP; ++j)
#pragma unroll
                        for (int t = 0; t < 2; ++t) {
                            const uint32_t pre = (cur[j] >> (16 * t + 4)) & 0xFFFu;
                            if (pre == A.P_hi || pre == A.Q_hi) {
                                const uint32_t cell = cell0 + (uint32_t)(j + t * NP) * NCX;
                                const uint32_t w =
                                    philox4x32_10_lane(A.key0, A.key1, rho, cell | 0x80000000u, tile, A.c3).x;
                                if (pre == A.P_hi && w < A.P_lo) take_p[j] |= 0xFFFFu << (16 * t);
                                if (pre == A.Q_hi && w < A.Q_lo) take_q[j] |= 0xFFFFu << (16 * t);
                            }
                        }
                }
                any_round((uint32_t)__builtin_amdgcn_readfirstlane((int)(f16 & 3u)));
            }
        }
    }

    // ---- the window's outer blocks, which keep bits of other domains: loads in flight
    constexpr uint32_t RIM = 2u * S::NB + 2u * (KW - 1u), TURNS = (RIM + 64u * NW - 1u) / (64u * NW);
    auto rim_block = [&](uint32_t t, uint32_t &b, uint32_t &kk) {
        if (t < 2u * S::NB) {
            b = t >> 1;
            kk = (t & 1u) ? KW : 0u;
        } else {
            const uint32_t u = min(t, RIM - 1u) - 2u * S::NB;
            b = (u & 1u) ? S::NB - 1u : 0u;
            kk = 1u + (u >> 1);
        }
    };
    auto block_at = [&](uint32_t b, uint32_t kk) {
        return base + ((((by0 + b) & A.nby_mask) << band_log2) + block_off(kk));
    };
    uint4 rim[TURNS][2];
#pragma unroll
    for (uint32_t n = 0; n < TURNS; ++n) {
        uint32_t b, kk;
        rim_block(tid + 64u * NW * n, b, kk);
        const char *p = block_at(b, kk);
        rim[n][0] = load_words<SHARED>(p);
        rim[n][1] = load_words<SHARED>(p + 16);
    }

    // ---- back to row words in LDS
#pragma unroll
    for (int j = 0; j < NP; ++j)
#pragma unroll
        for (int qy = 0; qy < 2; ++qy) {
            const uint32_t p0 = __builtin_amdgcn_perm(q[j][1][qy], q[j][0][qy], 0x05010400u);
            const uint32_t p1 = __builtin_amdgcn_perm(q[j][1][qy], q[j][0][qy], 0x07030602u);
            const uint32_t y = 4u * (q0 + 2u * (uint32_t)j + (uint32_t)qy) + i + 1u;
            plane[y * PITCH + k + 1u] = quad_transpose(swap_nibbles(p0), s1, s2);
            plane[(y + 8u * NP) * PITCH + k + 1u] = quad_transpose(swap_nibbles(p1), s1, s2);
        }
    if (NW > 1)
        __syncthreads();
    else
        wave_order();

    // ---- the slopes of a block: differences of v along the row and down the column
    auto slopes = [&](uint32_t b, uint32_t kk, auto clamp_c, uint32_t (&nx)[4], uint32_t (&ny)[4]) {
        constexpr bool CLAMP = decltype(clamp_c)::value;
        uint32_t above = 0u;
#pragma unroll
        for (int r = 0; r < 5; ++r) {
            int y = (int)(4u * b) + r - (int)offy;  // LDS row of domain row y - 1
            if (CLAMP) y = min(max(y, 0), (int)S::D + 1);
            const uint32_t *w = plane + (uint32_t)y * PITCH + kk;
            const uint32_t left = __builtin_amdgcn_alignbit(w[1], w[0], 31u - offx);  // one column to the left
            const uint32_t v = __builtin_amdgcn_alignbit(w[1] >> (31u - offx), left, 1u);
            if (r > 0) {
                nx[r - 1] = ~(v ^ left);
                ny[r - 1] = ~(v ^ above);
            }
            above = v;
        }
    };
    constexpr uint32_t INNER = (S::NB - 2u) * (KW - 1u);
    for (uint32_t t = tid; t < INNER; t += 64u * NW) {
        const uint32_t b = 1u + t / (KW - 1u), kk = 1u + t % (KW - 1u);
        uint32_t nx[4], ny[4];
        slopes(b, kk, std::false_type(), nx, ny);
        char *p = block_at(b, kk);
        store_words<SHARED>(p, nx);
        store_words<SHARED>(p + 16, ny);
    }
#pragma unroll
    for (uint32_t n = 0; n < TURNS; ++n) {
        const uint32_t t = tid + 64u * NW * n;
        if (t >= RIM) break;
        uint32_t b, kk;
        rim_block(t, b, kk);
        uint32_t nx[4], ny[4];
        slopes(b, kk, std::true_type(), nx, ny);
        const uint32_t my = kk == 0u ? ~0u << offx : (kk == KW ? (1u << offx) - 1u : ~0u);
        const uint32_t mx = kk == KW ? (2u << offx) - 1u : my;
        const uint32_t wx[4] = {rim[n][0].x, rim[n][0].y, rim[n][0].z, rim[n][0].w};
        const uint32_t wy[4] = {rim[n][1].x, rim[n][1].y, rim[n][1].z, rim[n][1].w};
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            const uint32_t y = 4u * b + (uint32_t)r - offy;  // domain row
            nx[r] = select_bits(y < S::D ? mx : 0u, nx[r], wx[r]);
            ny[r] = select_bits(y <= S::D ? my : 0u, ny[r], wy[r]);
        }
        char *p = block_at(b, kk);
        store_words<SHARED>(p, nx);
        store_words<SHARED>(p + 16, ny);
    }
}

template <int MODE, int LD, int NW>
__global__ void __launch_bounds__(64 * NW) step_dt_cells_kernel(StepArgs A)
{
    extern __shared__ uint32_t smem[];
    sweep_dt_cells<MODE, LD, NW, false>(A, smem, blockIdx.x);
}

}  // namespace okpz
