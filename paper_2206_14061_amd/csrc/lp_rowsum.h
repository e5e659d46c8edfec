// Sums over the sixteen lanes of a DPP row, written over an exchange X, so that
// the order of the additions can be checked lane by lane on the host.
// X::pick(bit, a, b): a in the lanes whose number has the bit, else b;
// X::move<CTRL>(x): the DPP move of that control word.
#pragma once

namespace lp {

// Four sums at once, times s: in the quads each lane keeps one of the four
// (halving what is exchanged), which rotations by 8 and 4 lanes then add up
// over the quads, and every lane reads all four from its quad.  The half-turn
// comes first: it leaves quads 0 and 2 (and 1 and 3) with the same two
// operands added, and the quarter-turn then adds those two sums in every quad,
// so that all lanes end with the same bits.
template <class X, class T>
__attribute__((always_inline)) constexpr void row_sum4(const X& x, const T (&d)[4], const T& s,
                                                       T (&f)[4])
{
    const T e0 = x.pick(1, d[1], d[0]) + x.template move<0xB1>(x.pick(1, d[0], d[1]));
    const T e1 = x.pick(1, d[3], d[2]) + x.template move<0xB1>(x.pick(1, d[2], d[3]));
    T e = x.pick(2, e1, e0) + x.template move<0x4E>(x.pick(2, e0, e1));
    e = e + x.template move<0x128>(e);   // row_ror:8
    e = e + x.template move<0x124>(e);   // row_ror:4
    e = e * s;
    f[0] = x.template move<0x00>(e);
    f[1] = x.template move<0x55>(e);
    f[2] = x.template move<0xAA>(e);
    f[3] = x.template move<0xFF>(e);
}

}  // namespace lp
