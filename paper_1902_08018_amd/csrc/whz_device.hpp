// whz_device.hpp -- WHZ1 block codec, device side (gfx950).
//
// WHZ1 is this library's zfp-style fixed-rate code for FP32 matrices in 4x4
// blocks (the paper stores its matrices zfp-compressed in fixed-rate mode,
// Sec. 4.3, Table 2).  Per block, exactly maxbits = 16*rate bits, LSB-first:
//   bit 0          1 if any value is nonzero (else the block is all +0)
//   bits 1..8      E = emax + 127, emax = max binade exponent, >= -126
//   bits 9..       embedded bit-plane code of the 16 transform coefficients,
//                  planes 31 -> 0, truncated at maxbits, zero padded.
// Coefficients: i = trunc(f * 2^(30 - emax)); a 4-point lift along every
// block row then every block column; sequency order; negabinary.
//
// One lane decodes one block.  The bits of the lane's block sit in a
// lane-private LDS row (words 0..NW-1 plus three zero words).
//
// Included by the .hip translation units after <hip/hip_runtime.h>.
#pragma once

#include <stdint.h>

namespace wh {

constexpr uint32_t kNega = 0xAAAAAAAAu;

// Sequency order: coefficient number s of the code is the transform output
// at local index kOrder(s) = 4r + c (c: horizontal frequency, r: vertical).
// Ordered by c + r, then c^2 + r^2, then larger c first.
__device__ __forceinline__ constexpr int order_of(int s)
{
    constexpr int t[16] = {0, 1, 4, 5, 2, 8, 6, 9, 3, 12, 10, 7, 13, 11, 14, 15};
    return t[s];
}

// ((hi:lo) >> sh) & 0xffffffff for sh in [0, 31]
__device__ __forceinline__ uint32_t funnel(uint32_t hi, uint32_t lo, uint32_t sh)
{
    return __builtin_amdgcn_alignbit(hi, lo, sh);
}

// Issue cost of vector instructions on gfx950, cycles per wave64 instruction
// and SIMD (measured with 8 waves a SIMD, independent instructions): 2 for
// the 4-byte forms of add, sub, and, or, xor, not, right shifts, 16-bit
// shifts, mov and FP32 add, mul and fmac on VGPRs and inline constants; 3 for
// those with a literal and for bitop3 on VGPRs; 4 for every other one (left
// shifts of 32 bits, bfe, bfi, perm, alignbit, SDWA, compares, conversions,
// three-operand adds, FP64) and for any of them that reads an SGPR.  The
// decoder is bound by these cycles, so its constants sit in VGPRs and its
// fields are where right shifts and plain adds reach them.

// The constant c in a VGPR, set where the call stands.
__device__ __forceinline__ uint32_t vgpr_const(uint32_t c)
{
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t r;
    asm volatile("v_mov_b32 %0, %1" : "=v"(r) : "i"(c));
    return r;
#else
    return c;
#endif
}

// (a & m) | (b & ~m)
__device__ __forceinline__ uint32_t select_bits(uint32_t m, uint32_t a, uint32_t b)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_bitop3_b32(a, b, m, 0xE4);
#else
    return (a & m) | (b & ~m);
#endif
}

// (a & m) | c
__device__ __forceinline__ uint32_t and_or(uint32_t a, uint32_t m, uint32_t c)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_bitop3_b32(a, m, c, 0xEA);
#else
    return (a & m) | c;
#endif
}

// v + v, which issues in half the time of v << 1 (what the compiler makes of
// it).
__device__ __forceinline__ uint32_t twice(uint32_t v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t r;
    asm("v_add_u32 %0, %1, %1" : "=v"(r) : "v"(v));
    return r;
#else
    return v + v;
#endif
}

__device__ __forceinline__ uint32_t asr1(uint32_t v) { return (uint32_t)((int32_t)v >> 1); }

// ---------------------------------------------------------------- lifting
// Forward lift on (x, y, z, w), modulo 2^32, floor halving.
__device__ __forceinline__ void fwd_lift(uint32_t& x, uint32_t& y, uint32_t& z, uint32_t& w)
{
    x = asr1(x + w);
    w -= x;
    z = asr1(z + y);
    y -= z;
    x = asr1(x + z);
    z -= x;
    w = asr1(w + y);
    y -= w;
    w += asr1(y);
    y -= asr1(w);
}

// Inverse lift.  Each "a <- a + b; b <- 2b - a" pair is written in its
// equivalent form "a' = a + b; b' = b - a" (both modulo 2^32).
__device__ __forceinline__ void inv_lift(uint32_t& x, uint32_t& y, uint32_t& z, uint32_t& w)
{
    y += asr1(w);
    w -= asr1(y);
    uint32_t t = y;
    y += w;
    w -= t;
    t = z;
    z += x;
    x -= t;
    t = y;
    y += z;
    z -= t;
    t = w;
    w += x;
    x -= t;
}

// 2-D inverse transform, local index v = 4r + c: columns, then rows.
__device__ __forceinline__ void inv_xform(uint32_t (&v)[16])
{
#pragma unroll
    for (int c = 0; c < 4; ++c)
        inv_lift(v[c], v[c + 4], v[c + 8], v[c + 12]);
#pragma unroll
    for (int r = 0; r < 4; ++r)
        inv_lift(v[4 * r], v[4 * r + 1], v[4 * r + 2], v[4 * r + 3]);
}

__device__ __forceinline__ void fwd_xform(uint32_t (&v)[16])
{
#pragma unroll
    for (int r = 0; r < 4; ++r)
        fwd_lift(v[4 * r], v[4 * r + 1], v[4 * r + 2], v[4 * r + 3]);
#pragma unroll
    for (int c = 0; c < 4; ++c)
        fwd_lift(v[c], v[c + 4], v[c + 8], v[c + 12]);
}

// ------------------------------------------------------ bit-matrix transpose
// G[q] holds plane p0 + q of 16 planes in bits 0..15 and plane p0 + 8 + q in
// bits 16..31 (bit s of a plane = coefficient s).  Three stages of exchanges
// between registers trade the register number q for the low three bits of s:
// afterwards bytes 0 and 2 of G[t] are coefficient t's bits in the planes
// p0..p0+7 and p0+8..p0+15, bytes 1 and 3 those of coefficient t + 8.  Bytes
// are then put together by byte permutes (assemble_coeffs), so no stage moves
// bits by 8 or 16, and 16 planes take half the work of 32: blocks whose code
// ends above plane 16 transpose one half only.
// One stage: registers i and i + D (i & D == 0) exchange their D-wide column
// blocks; m selects the low D columns of every 2D-wide group.  Two registers
// at a time: one 64-bit shift, which takes no longer than one of 32 bits,
// serves both (the bits that cross are not selected).  65536 x 65536 at rate 8:
// 2.94 ms with single shifts, 2.88 ms.  Templates keep every index a
// compile-time constant (no register indexing, no loop).
template <int D, int I, int J>
__device__ __forceinline__ void transpose_two_pairs(uint32_t (&G)[8], uint32_t m)
{
    uint32_t up0, up1;
    if constexpr (D == 1) {
        up0 = twice(G[I + D]);
        up1 = twice(G[J + D]);
    } else {
        const uint64_t v = ((uint64_t)G[J + D] << 32 | G[I + D]) << D;
        up0 = (uint32_t)v;
        up1 = (uint32_t)(v >> 32);
    }
    const uint32_t a0 = G[I], b0 = G[I + D], a1 = G[J], b1 = G[J + D];
    G[I] = select_bits(m, a0, up0);
    G[I + D] = select_bits(m, a0 >> D, b0);
    G[J] = select_bits(m, a1, up1);
    G[J + D] = select_bits(m, a1 >> D, b1);
}

__device__ __forceinline__ void transpose_half(uint32_t (&G)[8])
{
    const uint32_t m4 = vgpr_const(0x0F0F0F0Fu), m2 = vgpr_const(0x33333333u), m1 = vgpr_const(0x55555555u);
    transpose_two_pairs<4, 0, 1>(G, m4);
    transpose_two_pairs<4, 2, 3>(G, m4);
    transpose_two_pairs<2, 0, 1>(G, m2);
    transpose_two_pairs<2, 4, 5>(G, m2);
    transpose_two_pairs<1, 0, 2>(G, m1);
    transpose_two_pairs<1, 4, 6>(G, m1);
}

// Complements the odd planes of a half (p0 is even): together with the
// transpose this yields n ^ 0xAAAAAAAA for each negabinary coefficient n, the
// first half of its conversion to two's complement.
__device__ __forceinline__ void complement_odd_planes(uint32_t (&G)[8])
{
#pragma unroll
    for (int q = 1; q < 8; q += 2)
        G[q] = ~G[q];
}

// The transform coefficients (two's complement, at their block positions
// 4r + c) from the two transposed halves, H of planes 31..16 and L of planes
// 15..0: (n ^ 0xAAAAAAAA) - 0xAAAAAAAA modulo 2^32.
__device__ __forceinline__ void assemble_coeffs(const uint32_t (&H)[8], const uint32_t (&L)[8], uint32_t (&cf)[16])
{
    const uint32_t plus = vgpr_const(0u - kNega);
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        cf[order_of(t)] = __builtin_amdgcn_perm(H[t], L[t], 0x06040200u) + plus;     // L.b0 L.b2 H.b0 H.b2
        cf[order_of(t + 8)] = __builtin_amdgcn_perm(H[t], L[t], 0x07050301u) + plus; // L.b1 L.b3 H.b1 H.b3
    }
}

// --------------------------------------------------------------- decoding
// Group-test sections are decoded with a lookup table of 9 stream bits at a
// time.  A section (after the verbatim bits of a plane) is a sequence of
// tokens: "0" (the plane ends), "1" followed by a run: zeros (coefficients
// that stay insignificant) up to a 1 (the next one becomes significant,
// another token follows); when a run reaches coefficient 15 its 1 is implied,
// and once all are significant the plane ends.
//
// Table entry for (nsig, 9 bits), at index (nsig << 9) + bits:
//   bits 16..31  coefficients that became significant, at their absolute
//                positions, including coefficient 15's implied 1
//   bits  0..15  what the decoder's state (below) advances by: the
//                coefficients passed in bits 0..4, the bits passed in bits
//                7..11
//   bit  12      the section is open: it goes on past the 9 bits.  The entry
//                then stops inside a run, in front of the last bit that
//                belongs to the run's part already read: the next lookup
//                takes that bit as the 1 that opens a run, so every lookup
//                starts at a token and the table needs no second state
//                (a section that stands between two runs is taken back to
//                just in front of its last 1)
// The bits passed count from the plane's start, verbatim bits included.  An
// open entry's count is reduced by the new nsig, so that the next lookup,
// which adds that many verbatim bits again, reads at the right place.
constexpr int kSecBits = 9;
constexpr int kSecN = 17; // nsig 0..16
constexpr int kSecRow = 1 << kSecBits;
constexpr int kSecEntries = kSecN * kSecRow;

// The decoder's state: S = (pos - 2) << 7 | nsig, pos the next bit to read,
// coefficients 0..nsig-1 significant.  Shift amounts and bit-field widths
// read the low five bits of a register, so S serves as nsig there as it is;
// pos - 2 because a window read from two bits early holds the section's bits
// at the byte offset of their table entry; << 7 because bits 12 and up then
// are the byte offset of the window's word in a staged row of 1024 lanes.  Blocks
// of up to 14 words keep it in 16 bits (pos stays below 32 NW + 48): whole
// entries are then added to it, and its high half gathers what the entries
// hold above their low half, which nothing reads.  WIDE: the others, whose
// state takes the entries' low halves only.
constexpr uint32_t kPosShift = 7;
constexpr uint32_t kEntOpen = 1u << 12;
template <int NW>
constexpr bool kWideState = NW > 14;
template <bool WIDE>
__device__ __forceinline__ uint32_t advance(uint32_t S, uint32_t e)
{
    return WIDE ? S + (e & 0xFFFFu) : S + e;
}
template <bool WIDE>
__device__ __forceinline__ uint32_t state_value(uint32_t S)
{
    return WIDE ? S : S & 0xFFFFu;
}
__host__ __device__ __forceinline__ constexpr uint32_t state_at(uint32_t pos) { return (pos - 2u) << kPosShift; }

// The lanes whose v has a low half of at least `least`, as a wave mask (one
// 16-bit compare; written plainly the compiler masks the half out first).
__device__ __forceinline__ uint64_t lanes_from_u16(uint32_t v, uint32_t least)
{
#if defined(__HIP_DEVICE_COMPILE__)
    uint64_t m;
    asm("v_cmp_le_u16_e64 %0, %1, %2" : "=s"(m) : "s"(least), "v"(v));
    return m;
#else
    return __ballot((v & 0xFFFFu) >= least);
#endif
}

// Whether this lane's section goes on after entry e.
__device__ __forceinline__ bool ent_open(uint32_t e)
{
#if defined(__HIP_DEVICE_COMPILE__)
    return __builtin_amdgcn_inverse_ballot_w64(lanes_from_u16(e, kEntOpen));
#else
    return (e & 0xFFFFu) >= kEntOpen;
#endif
}

__host__ __device__ constexpr uint32_t section_entry(int nsig, int bits)
{
    int used = 0, adv = 0;
    uint32_t ones = 0;
    bool run = false, open = false;
    for (;;) {
        if (!run) {
            if (nsig + adv == 16) // every coefficient significant: no group bit
                break;
            if (used == kSecBits) { // between runs: back to in front of the last 1
                open = true;
                used -= 2;
                --adv;
                ones &= ~(1u << (nsig + adv));
                break;
            }
            const int g = (bits >> used) & 1;
            ++used;
            if (!g)
                break;
            run = true;
        } else {
            if (nsig + adv == 15) { // coefficient 15: its 1 is implied, not read
                ones |= 1u << 15;
                ++adv;
                break;
            }
            if (used == kSecBits) { // inside a run: its last bit opens the next lookup
                open = true;
                --used;
                break;
            }
            const int b = (bits >> used) & 1;
            ++used;
            if (b) {
                ones |= 1u << (nsig + adv);
                run = false;
            }
            ++adv;
            if (!b)
                continue;
        }
    }
    const uint32_t passed = (uint32_t)(open ? used - adv : nsig + used);
    return ones << 16 | (uint32_t)adv | passed << kPosShift | (open ? kEntOpen : 0u);
}

struct SectionTable {
    uint32_t e[kSecEntries];
    constexpr SectionTable() : e()
    {
        for (int n = 0; n < kSecN; ++n)
            for (int b = 0; b < kSecRow; ++b)
                e[n * kSecRow + b] = section_entry(n, b);
    }
};

// What the decoder reads the section table with: the table (in LDS) and two
// masks that stay in VGPRs for the kernel's life.
struct SectionReader {
    const uint32_t* tab;
    uint32_t bits_mask; // a table entry's byte offset in its row
    uint32_t word_mask; // the byte offset of a window's word in S
};

template <bool WIDE>
__device__ __forceinline__ SectionReader section_reader(const uint32_t* tab)
{
    return SectionReader{tab, vgpr_const(4u * (kSecRow - 1)), vgpr_const(WIDE ? 0x1F000u : 0xF000u)};
}

// Byte offset of the table's row for state S: nsig << 11 (a 16-bit left
// shift drops the position and issues in half the time of a 32-bit one).
__device__ __forceinline__ uint32_t sec_row(uint32_t S)
{
#if defined(__HIP_DEVICE_COMPILE__)
    uint32_t r;
    asm("v_lshlrev_b16 %0, 11, %1" : "=v"(r) : "v"(S));
    return r;
#else
    return (S & 31u) << 11;
#endif
}

// The entry for state S whose window (from two bits early) is w: the section
// starts nsig bits behind the window's first two.  FIRST: the plane's first
// lookup; the later ones take the section's first bit as 1.
template <bool FIRST>
__device__ __forceinline__ uint32_t sec_lookup(const SectionReader& sec, uint32_t S, uint32_t w)
{
    uint32_t off = and_or(w >> (S & 31u), sec.bits_mask, sec_row(S));
    if constexpr (!FIRST)
        off |= 4u;
    return *(const uint32_t*)((const char*)sec.tab + off);
}

// The word of a block staged at lw[word * STRIDE] that holds the bit two bits in
// front of state S's position.
template <int STRIDE>
__device__ __forceinline__ const uint32_t* state_word(const uint32_t* lw, const SectionReader& sec, uint32_t S)
{
    if constexpr (STRIDE == 1024 || STRIDE == 512 || STRIDE == 256 || STRIDE == 64) {
        // the word's byte offset, from its place in S
        const uint32_t off = (S & sec.word_mask) / (1024 / STRIDE);
        return (const uint32_t*)((const char*)lw + off);
    } else {
        return lw + ((S & sec.word_mask) >> 12) * STRIDE;
    }
}

// Bits 32..63 from there.
template <int STRIDE>
__device__ __forceinline__ uint32_t bits_ahead(const uint32_t* lw, const SectionReader& sec, uint32_t S)
{
    const uint32_t* p = state_word<STRIDE>(lw, sec, S);
    return funnel(p[2 * STRIDE], p[STRIDE], S >> kPosShift);
}

// Plane P's word, ones' high half | xv's low half, into its half: the planes
// p0 + 8.. come first and go to the high halves (low halves zero), p0.. to the
// low ones.  One instruction each: an SDWA or writing one half of its
// destination (the other half zeroed, or kept).
template <int P>
__device__ __forceinline__ void store_plane(uint32_t (&G)[8], uint32_t ones, uint32_t xv)
{
#if defined(__HIP_DEVICE_COMPILE__)
    if constexpr (P & 8)
        asm volatile("v_or_b32_sdwa %0, %1, %2 dst_sel:WORD_1 dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:DWORD"
            : "=v"(G[P & 7])
            : "v"(ones), "v"(xv));
    else
        asm volatile("v_or_b32_sdwa %0, %1, %2 dst_sel:WORD_0 dst_unused:UNUSED_PRESERVE src0_sel:WORD_1 src1_sel:DWORD"
            : "+v"(G[P & 7])
            : "v"(ones), "v"(xv));
#else
    const uint32_t x = ones >> 16 | (xv & 0xFFFFu);
    if constexpr (P & 8)
        G[P & 7] = x << 16;
    else
        G[P & 7] = (G[P & 7] & 0xFFFF0000u) | x;
#endif
}

// Planes P and below of a half are zero: the high planes from P down were
// never written.
template <int P>
__device__ __forceinline__ void clear_planes(uint32_t (&G)[8])
{
    if constexpr (P & 8) {
#pragma unroll
        for (int q = 0; q <= (P & 7); ++q)
            G[q] = 0u;
    }
}

// A block between two planes: the state, and 32 bits from two bits in front of
// its position.
struct PlaneCursor {
    uint32_t S, w;
};

// One bit plane of the embedded code (decoded in lockstep by all lanes of the
// wave) at cursor c.  Returns the plane word in two parts: the significant
// coefficients' verbatim bits in xv (low half), and the new ones (high half).
// ahead() gives the 32 bits that follow c.w.  A plane spans at most 31 bits, so
// the windows of its later lookups and, if NEXT_W, the next plane's lie within
// these 64.
template <bool WIDE, bool NEXT_W, typename F>
__device__ __forceinline__ uint32_t plane_bits(const SectionReader& sec, PlaneCursor& c, F ahead, uint32_t& xv)
{
    // the window holds the verbatim bits (nsig <= 16) and the first 9 section
    // bits (v_bfe takes the width modulo 32: nsig)
    uint32_t e = sec_lookup<true>(sec, c.S, c.w);
    xv = __builtin_amdgcn_ubfe(c.w, 2u, c.S);
    uint32_t ones = e, moved = e; // bits 7..11 of moved: the bits passed
    const uint32_t at = c.S;
    c.S = advance<WIDE>(c.S, e);
    if (ent_open(e)) {
        const uint32_t more = ahead(at);
        do { // the lanes whose section goes on
            c.S -= kEntOpen;
            e = sec_lookup<false>(sec, c.S, funnel(more, c.w, moved >> kPosShift));
            c.S = advance<WIDE>(c.S, e);
            moved += e;
            ones |= e;
        } while (ent_open(e));
    }
    if constexpr (NEXT_W)
        c.w = funnel(ahead(at), c.w, moved >> kPosShift);
    return ones;
}

// Planes that no block of NW words can run past its end in: P planes take at
// most 25 + 17 P bits with the header (16 verbatim bits a plane after the
// first, one ending group bit a plane, and over all planes 16 run-opening
// bits and 16 run bits).
template <int NW>
constexpr int kSafePlanes = 32 * NW < 25 ? 0 : (32 * NW - 25) / 17;

// Planes below this one may be cut by the bit budget without the exact
// inverse lift leaving the int32 range: a cut at plane lo moves a
// coefficient by less than 2^(lo+1), the 2-D inverse lift multiplies that by
// at most 3.75^2, and the block's integers stay below 2^30 + 2^29.3 < 2^31.
constexpr int kSafeCutPlane = 26;
// whether a block of NW words can be cut above that plane at all
template <int NW>
constexpr bool kCanCut = 32 - kSafeCutPlane > kSafePlanes<NW>;

// What a fixed-rate block's planes share.
template <int NW, int STRIDE>
struct BlockReader {
    const uint32_t* lw;
    SectionReader sec;
    uint64_t past; // the wave's lanes past their budget
    bool cut;      // see decode_block_coeffs
};

// Plane P of a fixed-rate block into its half G (NEXT_W, ahead: as
// plane_bits).  A lane whose budget is spent keeps stepping over zero bits: a
// zero group bit ends each section at once, so its plane words stay zero.
// Bits past the end of the block read as zero.  That gives the exact result
// everywhere except when the bit budget runs out inside a run: there the zero
// bits walk on to coefficient 15, where the code instead sets the coefficient
// the run had reached when the budget ended.  The number of zeros read past
// the end says which one that was.  Only planes in which some lane of the wave
// is past its budget pay for that correction, and the first kSafePlanes do not
// look for one.
template <int NW, int STRIDE, int P, bool NEXT_W, typename F>
__device__ __forceinline__ void decode_plane(BlockReader<NW, STRIDE>& rd, PlaneCursor& c, F ahead, uint32_t (&G)[8])
{
    constexpr uint32_t kMaxBits = 32u * NW;
    constexpr bool kWide = kWideState<NW>;
    uint32_t xv;
    uint32_t ones = plane_bits<kWide, NEXT_W>(rd.sec, c, ahead, xv);
    if constexpr (31 - P >= kSafePlanes<NW>) {
        const uint32_t at = state_value<kWide>(c.S);
        if constexpr (P == kSafeCutPlane && kCanCut<NW>)
            rd.cut = rd.cut && at >= state_at(kMaxBits + 1u);
        rd.past = kWide ? __ballot(at >= state_at(kMaxBits)) : lanes_from_u16(c.S, state_at(kMaxBits));
        if (__builtin_expect(rd.past != 0, 0)) { // a branch, not selects on every plane
            // the implied 1 of coefficient 15 moves back to where the run
            // stood when the budget ended (ex = zeros read past the end; ex
            // <= 15 wherever that 1 is set)
            const uint32_t ex = __builtin_elementwise_sub_sat(at >> kPosShift, kMaxBits - 2u);
            const uint32_t m = ones & 0x80000000u;
            ones ^= m ^ (m >> (ex & 31u));
            // a lane past the end reads only zero bits: its plane word is
            // zero; it goes on from the end, with nothing significant (which
            // no longer matters), where the words it may have read are zero
            c.S = __builtin_elementwise_min(at, state_at(kMaxBits));
        }
    }
    store_plane<P>(G, ones, xv);
}

// Planes P..LAST of a half.  When every lane of the wave is past its budget
// the planes left are zero.
// An odd plane reads 64 bits from its position and leaves the even plane below
// it its window, so that a pair waits for the stream once; the even plane reads
// on only where its section takes more than one lookup.  (65536^2 at rate 8:
// 2.94 ms (before the transposes shifted two registers at once, 2.86 now);
// 3.00 with the 32 bits ahead read in every plane, which takes 6
// cycles more a plane; 3.06 with every plane's window read in turn.)
template <int NW, int STRIDE, int P, int LAST>
__device__ __forceinline__ void decode_planes_from(BlockReader<NW, STRIDE>& rd, PlaneCursor& c, uint32_t (&G)[8])
{
    if constexpr (P >= LAST) {
        if constexpr (31 - P > kSafePlanes<NW> || kSafePlanes<NW> == 0) {
            if (rd.past == __builtin_amdgcn_read_exec()) {
                clear_planes<P>(G);
                return;
            }
        }
        if constexpr (P & 1) {
            const uint32_t* p = state_word<STRIDE>(rd.lw, rd.sec, c.S);
            const uint32_t lo = p[0], hi = p[STRIDE], more = p[2 * STRIDE];
            c.w = funnel(hi, lo, c.S >> kPosShift);
            const uint32_t ahead = funnel(more, hi, c.S >> kPosShift);
            decode_plane<NW, STRIDE, P, true>(rd, c, [ahead](uint32_t) { return ahead; }, G);
        } else {
            decode_plane<NW, STRIDE, P, false>(
                rd, c, [&rd](uint32_t S) { return bits_ahead<STRIDE>(rd.lw, rd.sec, S); }, G);
        }
        decode_planes_from<NW, STRIDE, P - 1, LAST>(rd, c, G);
    }
}

// Words a lane's staged block occupies in LDS: NW words of the block, then
// zeros, which the decoder reads past the end of the bit budget.  bits_ahead
// takes the two words after a position that stays below 32 bits past the end
// (a lane past it goes back to it after each plane, or stands in a zero block
// and moves one bit a plane; a plane never spans more than 31 bits: nsig
// verbatim bits and at most 1 + 2 (15 - nsig) section bits, or 16 verbatim
// bits), so word NW + 2 is the last one read.
template <int NW>
constexpr int kStagedWords = NW + 3;

// Planes 31 and 30, the first from the block's first words (w0, w1, w2): every
// lane is at bit 9 with nothing significant.  Plane 31 is empty in all blocks
// but those with a coefficient below -(2^31 - 1) / 3, so when no lane of the
// wave opens a run in it, it is one bit to pass.
template <int NW, int STRIDE>
__device__ __forceinline__ void decode_top_planes(BlockReader<NW, STRIDE>& rd, uint32_t w0, uint32_t w1, uint32_t w2,
                                                  bool nz, PlaneCursor& c, uint32_t (&H)[8])
{
    static_assert(kSafePlanes<NW> >= 2, "no block ends within its first two planes");
    c.w = nz ? funnel(w1, w0, 7u) : 0u;
    uint32_t ahead = nz ? funnel(w2, w1, 7u) : 0u;
    if (__any((c.w & 4u) != 0u)) {
        decode_plane<NW, STRIDE, 31, true>(rd, c, [ahead](uint32_t) { return ahead; }, H);
        decode_planes_from<NW, STRIDE, 30, 30>(rd, c, H);
    } else {
        H[7] = 0u;
        c.S += 1u << kPosShift;
        c.w = funnel(ahead, c.w, 1u);
        ahead >>= 1; // plane 30 has nothing verbatim: 31 bits are enough
        decode_plane<NW, STRIDE, 30, false>(rd, c, [ahead](uint32_t) { return ahead; }, H);
    }
}

// Decode the coefficients of the block staged at lw[q * STRIDE], q =
// 0..NW-1 (lw[q * STRIDE] == 0 for q = NW..NW+2); w: its words again, in
// registers (the first three are used).  Outputs the 16 transform coefficients (two's
// complement, at their block positions 4r + c, before the inverse
// transform).  Returns false for an all-zero block (then cf[] is all 0).
// Every bit pattern decodes (the function is total).
// `cut`: the budget ended above plane kSafeCutPlane (then only the exact
// integer lift reproduces the decoded block; see lin_inv_lift).
// `planes_read` is called once the code's bits have all been read: a caller
// loads the next block's words there, with the transposes and its own work
// on the coefficients still to come.
template <int NW, int STRIDE, typename F>
__device__ __forceinline__ bool decode_block_coeffs(const uint32_t* lw, const SectionReader& sec,
                                                    const uint32_t (&w)[NW], uint32_t (&cf)[16], bool& cut,
                                                    F planes_read)
{
    const bool nz = (w[0] & 1u) != 0;
    // a zero block is exact; others are cut until plane kSafeCutPlane is read
    BlockReader<NW, STRIDE> rd{lw, sec, 0, kCanCut<NW> && nz};
    PlaneCursor c;
    c.S = nz ? state_at(9u) : state_at(32u * NW);
    uint32_t H[8], L[8]; // every word is written by a plane or by the early exit
    const uint32_t w1 = NW > 1 ? w[NW > 1 ? 1 : 0] : 0u, w2 = NW > 2 ? w[NW > 2 ? 2 : 0] : 0u;
    if constexpr (kSafePlanes<NW> >= 2) {
        decode_top_planes<NW, STRIDE>(rd, w[0], w1, w2, nz, c, H);
        decode_planes_from<NW, STRIDE, 29, 16>(rd, c, H);
    } else {
        rd.past = __ballot(!nz);
        decode_planes_from<NW, STRIDE, 31, 16>(rd, c, H);
    }
    const bool low = rd.past != __builtin_amdgcn_read_exec(); // some lane has planes below 16
    if (low)
        decode_planes_from<NW, STRIDE, 15, 0>(rd, c, L);
    cut = rd.cut;
    planes_read();
    complement_odd_planes(H);
    transpose_half(H);
    if (low) {
        complement_odd_planes(L);
        transpose_half(L);
    } else {
        const uint32_t none = vgpr_const(kNega);
#pragma unroll
        for (int q = 0; q < 8; ++q)
            L[q] = none;
    }
    assemble_coeffs(H, L, cf);
    return nz;
}

// The binade exponent of the block whose first word is w0.
__device__ __forceinline__ int block_emax(uint32_t w0) { return (int)((w0 >> 1) & 0xFFu) - 127; }

// The decoded block: its coefficients through the inverse transform, as
// integers (value = iv * 2^(emax - 30)).
template <int NW, int STRIDE, typename F>
__device__ __forceinline__ bool decode_block_ints(const uint32_t* lw, const SectionReader& sec,
                                                  const uint32_t (&w)[NW], uint32_t (&iv)[16], F planes_read)
{
    bool cut;
    const bool nz = decode_block_coeffs<NW, STRIDE>(lw, sec, w, iv, cut, planes_read);
    inv_xform(iv);
    return nz;
}

template <int NW, int STRIDE>
__device__ __forceinline__ bool decode_block_ints(const uint32_t* lw, const uint32_t* tab, uint32_t w0, int& emax,
                                                  uint32_t (&iv)[16])
{
    uint32_t w[NW];
#pragma unroll
    for (int k = 0; k < NW; ++k)
        w[k] = lw[k * STRIDE];
    emax = block_emax(w0);
    return decode_block_ints<NW, STRIDE>(lw, section_reader<kWideState<NW>>(tab), w, iv, [] {});
}

// The inverse lift without its two floor halvings is a linear map B (the
// inverse of the forward lift's matrix (1/16) [[4,4,4,4],[5,1,-1,-5],
// [-4,4,4,-4],[-2,6,-6,2]]):
//   B = [[1, 3/2, -1, -1/4], [1, 1/2, 1, 5/4], [1, -1/2, 1, -5/4], [1, -3/2, -1, 1/4]]
// and the 2-D inverse transform of a coefficient block C is B C B^T up to
// those halvings (at most a few units of the block's last integer bit).
// Hence a block's row sums against u are B (C (B^T u)): B^T u is a per-
// column-block quantity, and B, being the same for every block, can be
// applied once to a row group's accumulated sums.  This holds while the
// integer lift stays inside int32; a block cut by the bit budget above plane
// kSafeCutPlane can leave it (the exact lift wraps modulo 2^32), so such
// blocks take the exact path: their decoded integers' row sums z, carried
// back to coefficient space as L z (L = B^-1, the forward lift's linear part).
template <typename T>
__device__ __forceinline__ void lin_inv_lift(T& x, T& y, T& z, T& w)
{
    y += w * T(0.5);
    w -= y * T(0.5);
    T t = y;
    y += w;
    w -= t;
    t = z;
    z += x;
    x -= t;
    t = y;
    y += z;
    z -= t;
    t = w;
    w += x;
    x -= t;
}

// B^T u for one block column (u0..u3 its four u values).
template <typename T>
__device__ __forceinline__ void lin_bt_u(T u0, T u1, T u2, T u3, T (&ut)[4])
{
    const T s03 = u0 + u3, d03 = u0 - u3, s12 = u1 + u2, d12 = u1 - u2;
    ut[0] = s03 + s12;
    ut[1] = T(1.5) * d03 + T(0.5) * d12;
    ut[2] = s12 - s03;
    ut[3] = T(1.25) * d12 - T(0.25) * d03;
}

// --------------------------------------------------------------- encoding
// The coefficients' planes, from the decoder's transpose run the other way: a
// half's registers are put together from the coefficients' bytes, and the same
// three exchange stages give the planes.
__device__ __forceinline__ void coeff_planes(const uint32_t (&n)[16], bool high, uint32_t (&G)[8])
{
#pragma unroll
    for (int t = 0; t < 8; ++t) // bytes 2 and 3 (high) or 0 and 1 of coefficients t and t + 8, alternating
        G[t] = __builtin_amdgcn_perm(n[t + 8], n[t], high ? 0x07030602u : 0x05010400u);
    transpose_half(G);
}

// A section's code comes 8 coefficients at a time from a table: the tokens of
// the bits c (each one of c: a 1 that opens its run, the run's zeros, the 1),
// in bits 0..15, how many bits they are in bits 16..20, and the coefficients
// they pass in bits 24..27.
struct EncodeTable {
    uint32_t e[256];
    constexpr EncodeTable() : e()
    {
        for (int c = 0; c < 256; ++c) {
            uint32_t code = 0, len = 0, adv = 0;
            for (uint32_t i = 0; i < 8; ++i) {
                if ((c >> i & 1) == 0)
                    continue;
                code |= 1u << len | 1u << (len + 1u + (i - adv));
                len += 2u + (i - adv);
                adv = i + 1u;
            }
            e[c] = code | len << 16 | adv << 24;
        }
    }
};

// A block's code as it is written: the next free bit, and how many
// coefficients are significant.
struct EncodeState {
    uint32_t pos, nsig;
};

// Code of one plane word x (at most 31 bits: the nsig verbatim bits, then the
// section's tokens and the 0 that ends it unless every coefficient is
// significant) into `sink`.
template <int NW, typename Sink>
__device__ __forceinline__ void encode_plane(uint32_t x, const uint32_t* tab, EncodeState& st, Sink& sink)
{
    const uint32_t r = x >> st.nsig;
    uint32_t e = tab[r & 0xFFu];
    uint32_t code = e & 0xFFFFu, len = __builtin_amdgcn_ubfe(e, 16u, 5u), adv = e >> 24;
    if (__any(r > 0xFFu)) {
        if (r > 0xFFu) {
            // the next token's run starts with the zeros left of the first 8
            e = tab[r >> 8];
            const uint32_t z = 8u - adv;
            code |= (1u | ((e & 0xFFFFu) >> 1) << (1u + z)) << len;
            len += __builtin_amdgcn_ubfe(e, 16u, 5u) + z;
            adv = 8u + (e >> 24);
        }
    }
    const uint32_t sig = st.nsig + adv;
    // coefficient 15's 1 is implied; anything less ends with a 0
    len = sig == 16u ? __builtin_elementwise_sub_sat(len, 1u) : len + 1u;
    const uint32_t bits = __builtin_amdgcn_ubfe(x, 0u, st.nsig) | __builtin_amdgcn_ubfe(code, 0u, len) << (st.nsig & 31u);
    sink.put(st.pos, bits);
    // past the budget everything goes to the two words after the block
    st.pos = __builtin_elementwise_min(st.pos + st.nsig + len, 32u * NW);
    st.nsig = sig;
}

// Planes of a half from P = p0 + 15 down; stops when the wave's blocks are full.
template <int NW, int P, int LAST, typename Sink>
__device__ __forceinline__ bool encode_planes(const uint32_t (&G)[8], const uint32_t* tab, EncodeState& st, Sink& sink)
{
    if constexpr (P >= LAST) {
        if (!__any(st.pos < 32u * NW))
            return false;
        encode_plane<NW>(P & 8 ? G[P & 7] >> 16 : G[P & 7] & 0xFFFFu, tab, st, sink);
        return encode_planes<NW, P - 1, LAST>(G, tab, st, sink);
    } else {
        return true;
    }
}

// Encode 16 values (local index 4r + c) into `sink`, whose words are zero:
// put(pos, bits) ORs bits in at bit pos, pos <= 32 * NW, up to 31 bits on.
// Returns false if a value is NaN or Inf (the block is then a zero block).
template <int NW, typename Sink>
__device__ __forceinline__ bool encode_block(const float (&f)[16], const uint32_t* tab, Sink& sink)
{
    // the largest magnitude's bit pattern: its exponent field F gives emax =
    // F - 126 (|f| in [2^(emax-1), 2^emax); a subnormal has F = 0, emax = -126)
    uint32_t m = 0u;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
        const uint32_t a = __float_as_uint(f[v]) & 0x7FFFFFFFu;
        m = a > m ? a : m;
    }
    const bool finite = m < 0x7F800000u, live = finite && m != 0u;
    const int emax = (int)(m >> 23) - 126;
    uint32_t n[16];
    {
        uint32_t iv[16];
#pragma unroll
        for (int v = 0; v < 16; ++v)
            iv[v] = finite ? (uint32_t)(int32_t)__builtin_ldexpf(f[v], 30 - emax) : 0u; // truncates
        fwd_xform(iv);
#pragma unroll
        for (int s = 0; s < 16; ++s)
            n[s] = (iv[order_of(s)] + kNega) ^ kNega;
    }
    EncodeState st{live ? 9u : 32u * NW, 0u};
    if (live)
        sink.put(0u, 1u | (uint32_t)(emax + 127) << 1);
    uint32_t G[8];
    coeff_planes(n, true, G);
    if (encode_planes<NW, 31, 16>(G, tab, st, sink) && __any(st.pos < 32u * NW)) {
        coeff_planes(n, false, G);
        (void)encode_planes<NW, 15, 0>(G, tab, st, sink);
    }
    return finite;
}

// The same into an array of NW words.
template <int NW>
__device__ __forceinline__ bool encode_block(const float (&f)[16], uint32_t (&out)[NW])
{
    static constexpr EncodeTable tab{};
    struct Words {
        uint32_t w[NW + 2] = {};
        __device__ void put(uint32_t pos, uint32_t bits)
        {
            const uint64_t v = (uint64_t)bits << (pos & 31u);
            w[pos >> 5] |= (uint32_t)v;
            w[(pos >> 5) + 1] |= (uint32_t)(v >> 32);
        }
    } sink;
    const bool finite = encode_block<NW>(f, tab.e, sink);
    for (int k = 0; k < NW; ++k)
        out[k] = sink.w[k];
    return finite;
}

} // namespace wh
