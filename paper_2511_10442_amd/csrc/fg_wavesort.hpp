// Sorting one key per lane across a wavefront without the LDS crossbar: bitonic networks whose exchanges are DPP moves
// (inside rows of 16 lanes) and permlane swaps (across rows).  A shuffle through the crossbar takes more than a hundred
// clocks and the 21 exchanges of a sort wait for each other; these take a few instructions each.
#pragma once
#include "fg_sortnet.hpp"

namespace fg {

// value of lane (own number ^ J)
template <int J>
__device__ __forceinline__ uint32_t lane_xor(uint32_t v)
{
    static_assert(J == 1 || J == 2 || J == 3 || J == 4 || J == 7 || J == 8 || J == 15, "exchanges inside a row of 16");
    constexpr int ctrl = J == 1 ? 0xb1 : J == 2 ? 0x4e : J == 3 ? 0x1b : J == 7 ? 0x141 : J == 8 ? 0x128 : J == 15 ? 0x140 : 0;
    if constexpr (J == 4) return lane_xor<7>(lane_xor<3>(v));
    else return (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, ctrl, 0xf, 0xf, true);
}

// lanes in pairs (l, l + 16) or (l, l + 32): a = the lower one's value in both, b = the upper one's.
// A swap must not read a register in the two wait states after a vector instruction has written it; the compiler sees to
// that for its own instructions but does not look into the asm of the comparators, hence the wait.
template <int J>
__device__ __forceinline__ void pair_values(uint32_t v, uint32_t& a, uint32_t& b)
{
    asm("s_nop 1" : "+v"(v));
    static_assert(J == 16 || J == 32, "rows and halves");
    if constexpr (J == 16) { const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false); a = r[0]; b = r[1]; }
    else { const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false); a = r[0]; b = r[1]; }
}

// A key whose sign bit says which half of the coming exchange its lane is in.  With the upper lane's value negated both
// lanes want the same thing, min(own, -other): 2 moves, a minimum and a change of sign per exchange instead of 2 moves, a
// minimum, a maximum and two selects.  (Keys as doubles: see cmp_swap.)
struct WaveKey {
    uint32_t lo, hi;
    __device__ __forceinline__ void flip(uint32_t m) { hi ^= m; }
    template <int J> __device__ __forceinline__ void exchange()
    {
        const uint64_t own = ((uint64_t)hi << 32) | lo;
        const uint64_t other = ((uint64_t)lane_xor<J>(hi) << 32) | lane_xor<J>(lo);
        double mn;
        asm("v_min_f64 %0, %1, -%2" : "=v"(mn) : "v"(__longlong_as_double((long long)own)), "v"(__longlong_as_double((long long)other)));
        const uint64_t r = (uint64_t)__double_as_longlong(mn);
        lo = (uint32_t)r;
        hi = (uint32_t)(r >> 32);
    }
    template <int J> __device__ __forceinline__ void exchange_rows(bool upper)
    {
        uint32_t al, bl, ah, bh;
        pair_values<J>(lo, al, bl);
        pair_values<J>(hi, ah, bh);
        const uint64_t a = ((uint64_t)ah << 32) | al, b = ((uint64_t)bh << 32) | bl;
        const uint64_t mn = key_min(a, b), mx = key_max(a, b);
        const uint64_t r = upper ? mx : mn;
        lo = (uint32_t)r;
        hi = (uint32_t)(r >> 32);
    }
};

// sign bit of a word: bit B of the lane's number
template <int B> __device__ __forceinline__ uint32_t lane_sign(int lane) { return (uint32_t)lane << (31 - B) & 0x80000000u; }

// the last exchanges of every merge, distances 8, 4, 2, 1 (from FROM on); the sign of bit `S` (-1: none) is on the key
template <int FROM, int S>
__device__ __forceinline__ void merge_in_row(WaveKey& k, int lane)
{
    uint32_t on = S < 0 ? 0u : lane_sign<S < 0 ? 0 : S>(lane);
    if constexpr (FROM >= 8) { const uint32_t n = lane_sign<3>(lane); k.flip(on ^ n); on = n; k.template exchange<8>(); }
    if constexpr (FROM >= 4) { const uint32_t n = lane_sign<2>(lane); k.flip(on ^ n); on = n; k.template exchange<4>(); }
    if constexpr (FROM >= 2) { const uint32_t n = lane_sign<1>(lane); k.flip(on ^ n); on = n; k.template exchange<2>(); }
    const uint32_t n = lane_sign<0>(lane);
    k.flip(on ^ n);
    k.template exchange<1>();
    k.flip(n);
}

// ascending by lane
__device__ __forceinline__ uint64_t wave_sort64_dpp(uint64_t v, int lane)
{
    WaveKey k{(uint32_t)v, (uint32_t)(v >> 32)};
    const uint32_t s0 = lane_sign<0>(lane), s1 = lane_sign<1>(lane), s2 = lane_sign<2>(lane), s3 = lane_sign<3>(lane);
    const bool up16 = (lane & 16) != 0, up32 = (lane & 32) != 0;
    k.flip(s0);      k.exchange<1>();                      // runs of 2
    k.flip(s0 ^ s1); k.exchange<3>();                      // of 4
    k.flip(s1 ^ s0); k.exchange<1>();
    k.flip(s0 ^ s2); k.exchange<7>();                      // of 8
    k.flip(s2 ^ s1); k.exchange<2>();
    k.flip(s1 ^ s0); k.exchange<1>();
    k.flip(s0 ^ s3); k.exchange<15>();                     // of 16
    merge_in_row<4, 3>(k, lane);
    // of 32: the upper row of each pair reversed, then the pairs of rows
    auto reverse_upper = [&](bool upper) __attribute__((always_inline)) {
        const uint32_t l = lane_xor<15>(k.lo), h = lane_xor<15>(k.hi);
        k.lo = upper ? l : k.lo;
        k.hi = upper ? h : k.hi;
    };
    reverse_upper(up16);
    k.exchange_rows<16>(up16);
    merge_in_row<8, -1>(k, lane);
    // of 64: the upper half reversed row by row, its rows change places in the exchange with the other half
    {
        const uint32_t l = lane_xor<15>(k.lo), h = lane_xor<15>(k.hi);
        uint32_t al, bl, ah, bh;
        pair_values<16>(l, al, bl);
        pair_values<16>(h, ah, bh);
        const uint32_t rl = up16 ? al : bl, rh = up16 ? ah : bh;      // value of lane ^ 31
        k.lo = up32 ? rl : k.lo;
        k.hi = up32 ? rh : k.hi;
    }
    k.exchange_rows<32>(up32);
    k.exchange_rows<16>(up16);
    merge_in_row<8, -1>(k, lane);
    return ((uint64_t)k.hi << 32) | k.lo;
}

// value of lane 63 - own number
__device__ __forceinline__ uint32_t wave_reverse(uint32_t v, int lane)
{
    uint32_t a, b;
    v = lane_xor<15>(v);
    pair_values<16>(v, a, b);
    v = (lane & 16) ? a : b;
    pair_values<32>(v, a, b);
    return (lane & 32) ? a : b;
}

// the 64 smallest keys of two ascending lists, ascending
__device__ __forceinline__ uint64_t wave_merge_lists(uint64_t best, uint64_t sorted, int lane)
{
    const uint64_t r = ((uint64_t)wave_reverse((uint32_t)(sorted >> 32), lane) << 32) | wave_reverse((uint32_t)sorted, lane);
    const uint64_t v = key_min(best, r);
    WaveKey k{(uint32_t)v, (uint32_t)(v >> 32)};
    k.exchange_rows<32>((lane & 32) != 0);
    k.exchange_rows<16>((lane & 16) != 0);
    merge_in_row<8, -1>(k, lane);
    return ((uint64_t)k.hi << 32) | k.lo;
}

// ascending sort of one 32-bit word per lane
template <int J> __device__ __forceinline__ uint32_t word_exchange(uint32_t v, bool upper)
{
    if constexpr (J < 16) {
        const uint32_t o = lane_xor<J>(v);
        const uint32_t mn = min(v, o), mx = max(v, o);
        return upper ? mx : mn;
    } else {
        uint32_t a, b;
        pair_values<J>(v, a, b);
        const uint32_t mn = min(a, b), mx = max(a, b);
        return upper ? mx : mn;
    }
}
__device__ __forceinline__ uint32_t wave_sort64_words(uint32_t v, int lane)
{
    const bool u0 = lane & 1, u1 = lane & 2, u2 = lane & 4, u3 = lane & 8, u4 = lane & 16, u5 = lane & 32;
    v = word_exchange<1>(v, u0);
    v = word_exchange<3>(v, u1); v = word_exchange<1>(v, u0);
    v = word_exchange<7>(v, u2); v = word_exchange<2>(v, u1); v = word_exchange<1>(v, u0);
    v = word_exchange<15>(v, u3); v = word_exchange<4>(v, u2); v = word_exchange<2>(v, u1); v = word_exchange<1>(v, u0);
    const uint32_t m = lane_xor<15>(v);
    v = u4 ? m : v;
    v = word_exchange<16>(v, u4); v = word_exchange<8>(v, u3); v = word_exchange<4>(v, u2); v = word_exchange<2>(v, u1); v = word_exchange<1>(v, u0);
    uint32_t a, b;
    pair_values<16>(lane_xor<15>(v), a, b);
    const uint32_t r = u4 ? a : b;
    v = u5 ? r : v;
    v = word_exchange<32>(v, u5); v = word_exchange<16>(v, u4); v = word_exchange<8>(v, u3); v = word_exchange<4>(v, u2); v = word_exchange<2>(v, u1);
    return word_exchange<1>(v, u0);
}

}  // namespace fg
