// jatam_device.hpp - device building blocks of JaTAM assembly on gfx950.
//
// Everything here is integer arithmetic in registers; nothing is shared with
// the CPU oracle.  The pieces:
//   philox4x32_10   counter-based generator (Salmon et al., SC'11) that
//                   replaces the paper's cuRAND XORWOW (§3)
//   oaat_*          Jenkins one-at-a-time hash (App. F.4), on unsigned bytes
//   Bonds           a decoded genotype: its tiles and, per colour, the tile
//                   that bonds to it, duplicate and symmetric orientations
//                   merged (§3.2; interaction rule of App. B.2: colours
//                   bond in adjacent pairs 1-2, 3-4, ...)
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

namespace jatam {

// ---------------------------------------------------------------------------
// Philox4x32-10: ten rounds of the published S-P network; the key is bumped
// by the two Weyl constants between rounds.
// ---------------------------------------------------------------------------
struct Words4 {
    uint32_t w[4];
};

__device__ __forceinline__ Words4 philox4x32_10(uint32_t c0, uint32_t c1, uint32_t c2,
                                                uint32_t c3, uint32_t k0, uint32_t k1)
{
    constexpr uint32_t kMul0 = 0xD2511F53u, kMul1 = 0xCD9E8D57u;
    constexpr uint32_t kWeyl0 = 0x9E3779B9u, kWeyl1 = 0xBB67AE85u;
#pragma unroll
    for (int round = 0; round < 10; ++round) {
        // each 32 x 32 -> 64-bit product as one multiply (v_mad_u64_u32)
        // rather than separate high and low halves
        const uint64_t p0 = (uint64_t)kMul0 * c0, p1 = (uint64_t)kMul1 * c2;
        const uint32_t hi0 = (uint32_t)(p0 >> 32), lo0 = (uint32_t)p0;
        const uint32_t hi1 = (uint32_t)(p1 >> 32), lo1 = (uint32_t)p1;
        const uint32_t n0 = hi1 ^ c1 ^ k0;
        const uint32_t n2 = hi0 ^ c3 ^ k1;
        c0 = n0;
        c1 = lo1;
        c2 = n2;
        c3 = lo0;
        k0 += kWeyl0;
        k1 += kWeyl1;
    }
    return Words4{{c0, c1, c2, c3}};
}

// ---------------------------------------------------------------------------
// One-at-a-time hash, split into its per-byte mix and its final avalanche.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t oaat_add(uint32_t h, uint32_t byte)
{
    h += byte;
    h += h << 10;
    h ^= h >> 6;
    return h;
}

__device__ __forceinline__ uint32_t oaat_finish(uint32_t h)
{
    h += h << 3;
    h ^= h >> 11;
    h += h << 15;
    return h;
}

// ---------------------------------------------------------------------------
// A decoded genotype of at most TM tiles (TM = 2 or 4) over at most 8 colours
// (kC16: 16).
//
// A colour tuple is a word of four bytes, byte d the colour of side d (N=0,
// E=1, S=2, W=3).  Oriented tile k = 4*i + r is tile i turned clockwise by r
// quarter turns: its tuple is tile i's word rotated left by 8r bits.  Of the
// orientations with one tuple only the first counts (the representative):
// turn r of a tile of period 1, 2 or 4 is turn r mod the period, and a tile
// in the orbit of an earlier one adds nothing.
//
// What bonds to a placed tile's side depends on the side's colour x alone,
// up to a turn: if side e of tile i has x's partner colour, turn
// r = d + 2 - e (mod 4) of tile i shows it towards a tile placed d-wards of
// the site.  So one byte per colour holds everything:
//   bit 7     some tile bonds to colour x
//   bit 6     two or more distinct tuples do (the rest is then meaningless)
//   bits 5-4  the tile's period - 1 (3, 1 or 0)
//   bits 3-2  the tile i
//   bits 1-0  (2 - e) mod 4
// and a byte permute looks up all four sides of a placed tile at once: about
// ten instructions for the four neighbours of a placement, where a SWAR
// comparison of each side with every oriented tile took about eighty.
// ---------------------------------------------------------------------------
constexpr uint32_t kSiteAny = 0x80808080u;     // bit 7 of every byte
constexpr uint32_t kSiteMulti = 0x40404040u;   // bit 6 of every byte

// A site's options as parts: any tile bonds, two or more do, the id of the
// tile if exactly one does.
struct SiteOpts {
    bool has, multi;
    uint32_t id;
};

__device__ __forceinline__ SiteOpts split_code(uint32_t code)
{
    return SiteOpts{(code & 0x80u) != 0, (code & 0x40u) != 0, code & 15u};
}

template <int TM, bool kC16>
struct Bonds {
    static_assert(TM == 2 || TM == 4, "TM must be 2 or 4");
    static constexpr bool kManyIds = TM == 4;   // ids up to 15, else up to 7
    // scalars, never arrays: a run-time index would put them in scratch memory
    uint32_t t0, t1, t2, t3;   // tiles (t2, t3 only for TM = 4)
    uint32_t lo, hi;           // the bytes of colours 0-3 and 4-7
    uint32_t lo2, hi2;         // of colours 8-11 and 12-15 (kC16 only)

    // Colour tuple of the seed: tile 0, unrotated.
    __device__ __forceinline__ uint32_t seed() const { return t0; }

    // by value: a choice between two members as lvalues makes the compiler
    // address the struct by a run-time offset, in scratch memory (a memory
    // round trip in every step)
    __device__ __forceinline__ static uint32_t pick(bool c, uint32_t x, uint32_t y)
    {
        return c ? x : y;
    }

    // Colour tuple of oriented tile k.
    __device__ __forceinline__ uint32_t oriented(uint32_t k) const
    {
        uint32_t w = pick((k & 4u) != 0, t1, t0);
        if constexpr (TM == 4)
            w = pick((k & 8u) != 0, pick((k & 4u) != 0, t3, t2), w);
        // rotate left by 8 (k mod 4): the shift amount counts mod 32
        return __builtin_amdgcn_alignbit(w, w, 0u - 8u * k);
    }

    // The four sites around a tile with colour tuple `tuple`: byte d is 0 if
    // nothing bonds in direction d, else 0x80, with 0x40 if two or more
    // distinct tiles do, and the representative's id in the low four bits.
    __device__ __forceinline__ uint32_t codes(uint32_t tuple) const
    {
        uint32_t w;
        if constexpr (kC16) {
            const uint32_t sel = tuple & 0x07070707u;
            const uint32_t up = (tuple >> 3) & 0x01010101u, mask = (up << 8) - up;
            w = (__builtin_amdgcn_perm(hi2, lo2, sel) & mask) |
                (__builtin_amdgcn_perm(hi, lo, sel) & ~mask);
        } else {
            w = __builtin_amdgcn_perm(hi, lo, tuple);
        }
        // turn d + 2 - e, reduced by the tile's period
        const uint32_t turn = ((w & 0x03030303u) + 0x03020100u) & (w >> 4) & 0x03030303u;
        return (w & 0xCCCCCCCCu) | turn;
    }
};

// The partner of colour y of c <= 8 colours, times 8, in byte y of the 64-bit
// constant (0 for a colour without a partner).
__device__ __forceinline__ uint64_t partner_shifts(int c)
{
    return c == 8 ? 0x0028301820081000ull : c == 4 ? 0x0000000000081000ull : 0ull;
}

template <class M>
struct BondsTraits;
template <int TM, bool kC16>
struct BondsTraits<Bonds<TM, kC16>> {
    static constexpr int kTiles = TM;
    static constexpr bool kWide = kC16;
};

template <class M>
__device__ __forceinline__ M build_bonds(uint64_t genome, int t, int bits, int c)
{
    constexpr int TM = BondsTraits<M>::kTiles;
    constexpr bool kC16 = BondsTraits<M>::kWide;
    const uint32_t cmask = (uint32_t)c - 1u;
    uint32_t tile[TM];
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        // tile i's 4 * bits <= 16 bits, N highest
        const uint32_t v = i < t ? (uint32_t)(genome >> (4 * bits * (t - 1 - i))) : 0u;
        tile[i] = ((v >> (3 * bits)) & cmask) | (((v >> (2 * bits)) & cmask) << 8) |
                  (((v >> bits) & cmask) << 16) | ((v & cmask) << 24);
    }
    const uint64_t shifts = partner_shifts(c);
    uint64_t tab = 0, tab2 = 0, multi = 0, multi2 = 0;
#pragma unroll
    for (int i = 0; i < TM; ++i) {
        const uint32_t w = tile[i];
        const uint32_t r1 = __builtin_amdgcn_alignbit(w, w, 24u);
        const uint32_t r2 = __builtin_amdgcn_alignbit(w, w, 16u);
        const uint32_t r3 = __builtin_amdgcn_alignbit(w, w, 8u);
        const bool sym4 = r1 == w, sym2 = r2 == w;
        bool repeated = false;
#pragma unroll
        for (int k = 0; k < i; ++k)
            repeated = repeated | (w == tile[k]) | (r1 == tile[k]) | (r2 == tile[k]) |
                       (r3 == tile[k]);
        const uint32_t base = (sym4 ? 0x80u : sym2 ? 0x90u : 0xB0u) | ((uint32_t)i << 2);
        // one entry per side of the first period; none for a repeated tile
        // (an absent tile shows colour 0 only, which has no partner)
        if constexpr (kC16) {
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t y = (w >> (8 * e)) & 0xFFu;
                const uint32_t x = ((y + 1u) ^ 1u) - 1u;   // its partner, if below c
                const bool keep = !repeated && x < (uint32_t)c && (e == 0 || !sym4) &&
                                  (e < 2 || !sym2);
                const uint64_t v = (uint64_t)(keep ? base | (uint32_t)((2 - e) & 3) : 0u)
                                   << (8u * (x & 7u));
                const uint64_t v1 = x < 8u ? v : 0ull, v2 = x < 8u ? 0ull : v;
                multi |= tab & v1;
                tab |= v1;
                multi2 |= tab2 & v2;
                tab2 |= v2;
            }
        } else {
            const uint32_t at = __builtin_amdgcn_perm((uint32_t)(shifts >> 32), (uint32_t)shifts, w);
            const uint32_t first = repeated ? 0u : base | 2u;
            const uint32_t rest = sym4 ? 0u : first, last = sym2 ? 0u : first;
#pragma unroll
            for (int e = 0; e < 4; ++e) {
                const uint32_t b = e == 0 ? first : e == 1 ? rest : last;
                // (2 - e) mod 4 = 2, 1, 0, 3 in the low bits of a kept entry
                const uint32_t flip = e == 0 ? 0u : e == 1 ? 3u : e == 2 ? 2u : 1u;
                const uint64_t v = (uint64_t)(b != 0u ? b ^ flip : 0u) << ((at >> (8 * e)) & 0xFFu);
                multi |= tab & v;
                tab |= v;
            }
        }
    }
    constexpr uint64_t kAny = 0x8080808080808080ull;
    tab |= (multi & kAny) >> 1;
    tab2 |= (multi2 & kAny) >> 1;
    if constexpr (!kC16)
        tab &= ~0xFFull;   // sides without a partner were entered at colour 0
    M m;
    m.t0 = tile[0];
    m.t1 = tile[1];
    m.t2 = TM == 4 ? tile[2 % TM] : 0u;
    m.t3 = TM == 4 ? tile[3 % TM] : 0u;
    m.lo = (uint32_t)tab;
    m.hi = (uint32_t)(tab >> 32);
    m.lo2 = (uint32_t)tab2;
    m.hi2 = (uint32_t)(tab2 >> 32);
    return m;
}

// The genotype types that the kernels are compiled for: up to two tiles, up
// to four, and any number over 16 colours.
using Bonds2 = Bonds<2, false>;
using Bonds4 = Bonds<4, false>;
using BondsC16 = Bonds<4, true>;

}  // namespace jatam
