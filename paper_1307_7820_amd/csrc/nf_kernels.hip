// HIP kernels for gfx950: the two-vector Four-Russians fill of the Nussinov
// table (Section 3.1, Eq. 3) swept as a tile wavefront (Sections 4-5).
//
// Work of one wavefront step (tile diagonal d):
//   * k_between: for a tile (A, B = A+d) and a range of intermediate tiles C,
//     the best split over every q-group of posts inside those tiles, one R
//     lookup per group (Eq. 3).  Only tiles of diagonals < d are read.
//   * k_tile: the finish of tile (A, B): folds in the partial maxima, the
//     groups of the two tiles next to the diagonal ends (C = A+1, C = B-1),
//     the pairing term and the splits that fall inside tiles A and B
//     (the "residual" split points of Section 3.1), row by row from the
//     bottom, each row held as the bits of its differences; then writes the
//     dense int16 cells and the packed row/column words (and, at q = 8, the
//     marks by which k_between skips groups).
//   * k_diag: the tiles (A, A) on the main diagonal, where every split point
//     is inside the tile.
// Max is idempotent and order-free, so the result does not depend on how the
// between-group work is split into partial slots.
#include "nf_internal.h"

#include <hip/hip_ext.h>

#include <type_traits>

namespace nf {

namespace {

// Address-space views of generic pointers.  The between-group lookups read
// row words wave-uniformly through the scalar cache (constant address
// space); column words are per-lane global loads.  The scalar cache is not
// kept coherent with vector stores inside a launch, so the invariant is: no
// row word that a launch reads through the scalar cache is written by that
// same launch.  It holds because a between chunk of tile (A, A+d) reads only
// tiles of diagonals 2 .. d-2, a staged between launch writes no packed
// words (the finishes of diagonal d-1 that may run beside it on another
// stream write only that diagonal), and the fused step that runs it
// (d = s+1) writes only the words of diagonal s.  Packed blocks of different
// tiles never share a cache line (each block is a multiple of 256 bytes).
// A tile finish at q < 4 reads the end tiles' row words this way too, also of
// earlier diagonals only.
#define NF_GLOBAL __attribute__((address_space(1)))
#define NF_CONST __attribute__((address_space(4)))
template <class T>
__device__ __forceinline__ const NF_GLOBAL T* as_global(const T* p)
{
    return (const NF_GLOBAL T*)p;
}
template <class T>
__device__ __forceinline__ const NF_CONST T* as_const(const T* p)
{
    return (const NF_CONST T*)p;
}

// R index of a row word held in a scalar register and a column word: bits
// 31..16 of each, one VALU instruction (SDWA selects both high halves; an
// ALU operation, not a load).
__device__ __forceinline__ uint32_t r_index_s(uint32_t rw, uint32_t cw)
{
    uint32_t idx;
    __asm__("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:WORD_1"
            : "=v"(idx)
            : "s"(rw), "v"(cw));
    return idx;
}

// The same with both words in vector registers.
__device__ __forceinline__ uint32_t r_index_v(uint32_t rw, uint32_t cw)
{
    uint32_t idx;
    __asm__("v_add_u32_sdwa %0, %1, %2 dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:WORD_1"
            : "=v"(idx)
            : "v"(rw), "v"(cw));
    return idx;
}

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// max of the low 16 bits of a, b and c as unsigned numbers, one VALU
// instruction (the high halves of the operands are ignored).
__device__ __forceinline__ uint32_t max3_u16(uint32_t a, uint32_t b, uint32_t c)
{
    uint32_t d;
    __asm__("v_max3_u16 %0, %1, %2, %3" : "=v"(d) : "v"(a), "v"(b), "v"(c));
    return d;
}

// Copy the q-dependent R table (RSZ bytes) into LDS.  From 1 KB on by DMA
// (global -> LDS, no registers and no LDS store; a wave moves 1 KB and RSZ is
// a multiple of it, so no lane reads past R or writes past Rl), which the
// caller waits for (vector memory counter); below that through registers.
// The caller's barrier follows.
template <int RSZ>
__device__ __forceinline__ void issue_R(uint8_t* Rl, const uint8_t* __restrict__ Rg, int nthr)
{
    if constexpr (RSZ >= 1024) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
        for (int base = wave * 1024; base < RSZ; base += nthr * 16)  // wave-uniform
            __builtin_amdgcn_global_load_lds((const NF_GLOBAL void*)(Rg + base + lane * 16),
                                             (__attribute__((address_space(3))) void*)(Rl + base), 16, 0, 0);
    } else if constexpr (RSZ >= 16) {
        for (int x = threadIdx.x * 16; x < RSZ; x += nthr * 16)
            *reinterpret_cast<uint4*>(Rl + x) = *reinterpret_cast<const uint4*>(Rg + x);
    } else {
        if (threadIdx.x < RSZ) Rl[threadIdx.x] = Rg[threadIdx.x];
    }
}
template <int RSZ>
__device__ __forceinline__ void load_R(uint8_t* Rl, const uint8_t* __restrict__ Rg, int nthr)
{
    issue_R<RSZ>(Rl, Rg, nthr);
    if constexpr (RSZ >= 1024) __builtin_amdgcn_s_waitcnt(0);
}

// Between-group maxima for the RPW rows r0..r0+RPW-1 (wave-uniform) and column j
// (the lane) of tile (A, B), over the groups of tiles C in [c0, c1).
// For group k of tile C the row word comes from tile (A, C) and the column
// word from tile (C, B); Eq. 3 turns the q split points of the group into
//     F(a, Cq') + F(Cq', b) + R[h][c].
// With NS > 1 the caller's share is every NS-th group of the flattened
// (C, k) sequence, starting at group h.
//
// A lookup is two and a half VALU instructions: the R index (one SDWA add of
// the high halves of the scalar row word and the column word), one 3-input
// add of the whole row word, the whole column word and R (the low halves
// hold the two bases, so the low half of the sum is the split's value, see
// the packed words), and half of a 16-bit 3-input max over two groups.  acc
// holds its maxima in the low 16 bits.
template <int Q, int RPW, int NS>
__device__ __forceinline__ void between_accumulate(int (&acc)[RPW], const uint8_t* Rl,
                                                   const uint32_t* __restrict__ RS,
                                                   const uint32_t* __restrict__ CS, int NT, int A,
                                                   int B, int c0, int c1, int r0, int j, int h)
{
    constexpr int G = groups_per_tile(Q);
    constexpr int SW = state_words(Q);
    constexpr int RW = row_words(Q);
    if constexpr (G % NS == 0) {
        // every tile gives this wave the same KPT groups k = h, h+NS, ...,
        // taken KB at a time (KB * RPW row words fit the scalar registers):
        // all the row words (scalar loads) and column words of a batch are
        // loaded before its first lookup, so the wait for the scalar loads,
        // which also waits for the LDS gathers in flight, comes once per
        // batch; the next batch's column words are loaded while this batch's
        // lookups run
        constexpr int KPT = G / NS;
        constexpr int KB = KPT % 4 == 0 ? 4 : (KPT % 2 == 0 ? 2 : 1);
        constexpr int NBT = KPT / KB;  // batches per tile
        uint32_t cwn[KB];
        auto load_cw = [&](int C, int u0) {
            const NF_GLOBAL uint32_t* cs = as_global(CS + tile_index(NT, C, B - C) * SW + j);
#pragma unroll
            for (int v = 0; v < KB; ++v) cwn[v] = cs[(h + (u0 + v) * NS) * 64];
        };
        if (c0 < c1) load_cw(c0, 0);
        for (int C = c0; C < c1; ++C) {
            const NF_CONST uint32_t* rs = as_const(RS + tile_index(NT, A, C - A) * RW + r0);
#pragma unroll
            for (int bt = 0; bt < NBT; ++bt) {
                const int u0 = bt * KB;
                uint32_t cw[KB], rw[KB][RPW];
#pragma unroll
                for (int v = 0; v < KB; ++v) cw[v] = cwn[v];
#pragma unroll
                for (int v = 0; v < KB; ++v)
#pragma unroll
                    for (int r = 0; r < RPW; ++r) rw[v][r] = rs[(h + (u0 + v) * NS) * 64 + r];
                if (bt + 1 < NBT)
                    load_cw(C, u0 + KB);
                else if (C + 1 < c1)
                    load_cw(C + 1, 0);
#pragma unroll
                for (int v = 0; v < KB; v += 2) {
#pragma unroll
                    for (int r = 0; r < RPW; ++r) {
                        const uint32_t t0 = rw[v][r] + cw[v] + Rl[r_index_s(rw[v][r], cw[v])];
                        const uint32_t t1 =
                            v + 1 < KB ? rw[v + 1][r] + cw[v + 1] + Rl[r_index_s(rw[v + 1][r], cw[v + 1])] : 0u;
                        acc[r] = (int)max3_u16((uint32_t)acc[r], t0, t1);
                    }
                }
            }
        }
    } else {
        for (int C = c0; C < c1; ++C) {
            const NF_CONST uint32_t* rs = as_const(RS + tile_index(NT, A, C - A) * RW + r0);
            const NF_GLOBAL uint32_t* cs = as_global(CS + tile_index(NT, C, B - C) * SW + j);
            const int k0 = ((h - (C - c0) * G) % NS + NS) % NS;
#pragma unroll 2
            for (int k = k0; k < G; k += NS) {
                const uint32_t cw = cs[k * 64];
#pragma unroll
                for (int r = 0; r < RPW; ++r) {
                    const uint32_t rw = rs[k * 64 + r];
                    const uint32_t t = rw + cw + Rl[r_index_s(rw, cw)];
                    acc[r] = (int)max3_u16((uint32_t)acc[r], t, 0u);
                }
            }
        }
    }
#pragma unroll
    for (int r = 0; r < RPW; ++r) acc[r] &= 0xffff;
}

__global__ void k_precompute_R(int q, uint8_t* __restrict__ R)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < 1 << (2 * (q - 1))) R[e] = r_entry(q, e);
}

__global__ void k_copy_codes(const uint8_t* __restrict__ src, int n, uint8_t* __restrict__ dst, int padded)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < padded) dst[e] = e < n ? (src[e] & 3) : 0;
}

// ---- Rows in bits.
//
// A row of the table differs from the row below it by 0 or 1 in every column
// (Lemma 1), so a tile is finished row by row, bottom-up, as one bit per cell:
// delta(i, j) = X(i, j) - X(i+1, j).  With U(j', j) = F(BT+j', BT+j) (tile
// (B, B)) let
//     E(j', j) = X(i+1, j) - X(i+1, j') - U(j', j)            (j' < j)
// be the slack of the split at j' on the row below: >= 0, since j' is a split
// of Eq. 1.  A split at j' gives delta(i, j) = 1 exactly when delta(i, j') = 1
// and E(j', j) = 0, a pairing (i, j) exactly when E(j-1, j) = 0 (then
// X(i+1, j-1) + 1 > X(i+1, j)).  Eq. 1 makes F superadditive, so "E = 0" is
// transitive and one pass closes a set of columns that rise by themselves
// over all splits:  delta(j) = s(j) or (some j' in s with E(j', j) = 0).
// Afterwards E(j', j) += delta(i, j) - delta(i, j').
// The splits inside tile A are the same thing along the column: the slack
//     V(i', j) = X(i+1, j) - X(i', j) - L(i+1, i'),   L(i, i') = F(AT+i, AT+i'),
// gives delta(i, j) = 1 when V = 0 and dL(i, i') = L(i, i') - L(i+1, i') = 1,
// and moves by delta(i, j) - dL(i, i').
//
// The slacks are bit-sliced: bit b of word p_k of a lane is bit k of the slack
// at split point b (slacks are at most 63, so six words), and the +1/-1/0 of
// a row is a ripple through the six words, two instructions each, for 32
// split points at once.  A row therefore costs about 30 VALU instructions
// per 32 split points and 64 lanes and no LDS access on its chain, where the
// max-plus closure over 8 wavefronts it replaces took 27 instructions in each
// of the 8, an LDS round trip and a barrier.

// f(a, b, c) bit by bit, one instruction: kTable = f(0xF0, 0xCC, 0xAA).
template <int kTable>
__device__ __forceinline__ uint32_t bits3(uint32_t a, uint32_t b, uint32_t c)
{
    return __builtin_amdgcn_bitop3_b32(a, b, c, kTable & 0xff);
}
constexpr int kA = 0xF0, kB = 0xCC, kC = 0xAA;  // the three operands in a table

// Slacks of 32 split points (one per bit) in one lane.  A row's change (+ 1 at
// the bits of c where up is all ones, - 1 where it is 0) is taken in two
// parts: mark() moves the set of zero slacks, which the next row waits for,
// and ripple() the words, which it does not.  A block of at most four rows
// that starts with every slack below 12 needs the four low words only: no
// slack passes 15 or leaves 0 downwards there.
struct Slack {
    uint32_t p[6];
    uint32_t zero, one;  // the split points of slack 0 and 1

    template <int kWords>
    __device__ __forceinline__ void find_one()
    {
        uint32_t hi = bits3<kA | kB | kC>(p[1], p[2], p[3]);
        if constexpr (kWords == 6) hi = bits3<kA | kB | kC>(hi, p[4], p[5]);
        one = p[0] & ~hi;
    }
    __device__ __forceinline__ void begin()
    {
        zero = ~(bits3<kA | kB | kC>(p[0], p[1], p[2]) | bits3<kA | kB | kC>(p[3], p[4], p[5]));
        find_one<6>();
    }
    __device__ __forceinline__ void mark(uint32_t c, uint32_t up)
    {
        zero = bits3<(kA & kB) | (~kA & kC)>(c, one & ~up, zero);
    }
    template <int kWords>
    __device__ __forceinline__ void ripple(uint32_t c, uint32_t up)
    {
#pragma unroll
        for (int k = 0; k < kWords - 1; ++k) {
            const uint32_t carry = bits3<kA & ~(kB ^ kC)>(c, p[k], up);
            p[k] ^= c;
            c = carry;
        }
        p[kWords - 1] ^= c;
        find_one<kWords>();
    }
    // nonzero at the slacks of 12 and more
    __device__ __forceinline__ uint32_t large() const { return bits3<kA | (kB & kC)>(p[4], p[3], p[2]) | p[5]; }
};

// bit `pos` of x as a mask (all ones or 0), one instruction
__device__ __forceinline__ uint32_t bit_mask(uint32_t x, uint32_t pos)
{
    return (uint32_t)__builtin_amdgcn_sbfe((int)x, pos, 1u);
}

// lane kLane of `old` replaced by the scalar v
template <int kLane>
__device__ __forceinline__ uint32_t with_lane(uint32_t old, uint32_t v)
{
    __asm__("v_writelane_b32 %0, %1, %2" : "+v"(old) : "s"(v), "n"(kLane));
    return old;
}

// f(r), f(r-1), ..., f(0), each with its number as a constant
template <int r, class F>
__device__ __forceinline__ void rows_down(F&& f)
{
    f(std::integral_constant<int, r>{});
    if constexpr (r > 0) rows_down<r - 1>(f);
}

// For each of the 64 rows of a lane's code (S_{a+1} of row `lane`), the rows
// whose base pairs with cb: bit i of the result.
__device__ __forceinline__ unsigned long long pair_rows(int code, int cb)
{
    const unsigned long long m0 = __ballot(code == 0), m1 = __ballot(code == 1), m2 = __ballot(code == 2),
                             m3 = __ballot(code == 3);
    return cb == 0 ? m3 : (cb == 1 ? m2 : (cb == 2 ? m1 : m0));
}

// What a main-diagonal tile (B, B) keeps in the fold's blocks of packed words
// (which hold no words for it): the slack words of tile column B, written by
// the finish of (A+1, B) and read and updated by the finish of (A, B) one
// step later, and the bits dL(i, .) of its own rows.  Three words of slack
// and one half of every row's bits lie in the row block, the others in the
// column block: 448 words in each, what a block holds at q = 9.
//   word k of column j, split points 32h .. 32h+31: [(k % 3) * 128 + 2j + h]
//   dL(i, i' < 32) in the row block at [384 + i], dL(i, i' >= 32) in the column block
constexpr int kRowBits = 384;
static_assert(row_words(9) >= kRowBits + 64 && state_words(9) >= kRowBits + 64, "the main-diagonal blocks hold the slacks");

// Main-diagonal tiles (A, A): every split point lies inside the tile.  One
// wavefront (lane j = column j) fills the tile by rows in bits (Eq. 1 needs
// only the pairings and the splits E), the others wait for the emit.
struct DiagLds {
    unsigned long long cm[64];  // bit i of cm[j] = delta(i, j)
    uint2 rows[64];             // rows[i] = dL(i, .)
};

//
// Admission (staged != null and it.pad2 != 0, the serving engine's newly
// admitted folds): the fold's padded codes are read from staged + it.pad1
// instead of its own block, and the tile also does the fold's set-up: it
// copies its T codes (the last tile also the padding after them) into the
// fold's block and clears its two accumulator blocks (it.acc, one per
// diagonal parity), so that admitting a fold takes no copy or fill of its
// own.  Nothing else reads the fold's block before this launch has ended.
//
// Direct codes (n >= 0, with staged == null: a single fold on device codes): the n codes are read from the caller's buffer, taken mod 4,
// and copied padded into the fold's block in the same way.
template <int Q>
__device__ __forceinline__ void diag_body(const TileWork& it, DiagLds& s, int tid, int nthr, const uint8_t* staged,
                                          const uint8_t* codes, int n)
{
    constexpr int T = tile_size(Q);
    const FoldDesc& f = it.f;
    const int aT = it.A * T;
    const bool admit = staged != nullptr && it.pad2 != 0;
    const bool direct = n >= 0;
    const uint8_t* src = direct ? codes : (admit ? staged + it.pad1 : f.codes);
    auto code = [&](int e) -> int { return direct ? (e < n ? src[e] & 3 : 0) : (int)src[e]; };
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;

    if (admit || direct) {
        uint8_t* dst = const_cast<uint8_t*>(f.codes);
        const int hi = it.A == f.NT - 1 ? f.NT * T + 64 : aT + T;
        for (int e = aT + tid; e < hi; e += nthr) dst[e] = (uint8_t)code(e);
    }
    if (admit) {
        int4* a0 = reinterpret_cast<int4*>(it.acc + (size_t)it.A * kTileCells);
        int4* a1 = reinterpret_cast<int4*>(it.acc + (size_t)(f.NT + it.A) * kTileCells);
        for (int e = tid; e < kTileCells / 4; e += nthr) a0[e] = a1[e] = make_int4(0, 0, 0, 0);
    }
    if (wave == 0) {
        const int j = lane;
        const int ca = code(aT + j);                              // S_{a+1} for a = aT + lane
        const int cb = (aT + j - 1 >= 0) ? code(aT + j - 1) : 0;  // S_b for b = aT + j
        // split points below j; pairing rows i <= j - 2
        const unsigned long long below = j < T ? (1ull << j) - 1 : 0ull;
        unsigned long long pm = pair_rows(ca, cb) & (below >> 1);
        const unsigned long long left = j > 0 ? 1ull << (j - 1) : 0ull;  // the slack a pairing needs
        const uint32_t blo = (uint32_t)left, bhi = (uint32_t)(left >> 32);
        const uint32_t vlo = (uint32_t)below, vhi = (uint32_t)(below >> 32);
        Slack lo{}, hi{};
        lo.p[5] = ~vlo;  // never 0 at split points that are not left of j
        hi.p[5] = ~vhi;
        lo.begin();
        hi.begin();
        unsigned long long cm = 0;
        for (int b = 7; b >= 0; --b) {
            const uint32_t pmb = (uint32_t)(pm >> (8 * b));
            const unsigned long long pts = ~((256ull << (8 * b)) - 1);  // the split points of the blocks below
            uint32_t rlo = 0, rhi = 0;  // lane r: dL(8b + r, .)
            rows_down<7>([&](auto rc) {
                constexpr int r = rc;
                if (T < 64 && 8 * b + r >= T) return;
                const uint32_t pb = bit_mask(pmb, r);
                const unsigned long long st =
                    __ballot((bits3<(kA & kB) | kC>(lo.zero, blo, hi.zero & bhi) & pb) != 0);
                const unsigned long long cl =
                    __ballot(bits3<(kA & kB) | kC>(lo.zero, (uint32_t)st, hi.zero & (uint32_t)(st >> 32)) != 0);
                const unsigned long long dl = st | cl;
                const uint32_t up = (dl >> j) & 1 ? ~0u : 0u;
                // split points i < j' < j move; j' = i joins with slack 0
                const unsigned long long rm = pts | ((0xffull & (0xfeull << r)) << (8 * b));
                const uint32_t cl_lo = bits3<(kA ^ kB) & kC>(up, (uint32_t)dl, vlo & (uint32_t)rm);
                const uint32_t cl_hi = bits3<(kA ^ kB) & kC>(up, (uint32_t)(dl >> 32), vhi & (uint32_t)(rm >> 32));
                lo.mark(cl_lo, up);
                hi.mark(cl_hi, up);
                lo.ripple<6>(cl_lo, up);
                hi.ripple<6>(cl_hi, up);
                cm = (cm << 1) | (up & 1u);
                rlo = with_lane<r>(rlo, (uint32_t)dl);
                rhi = with_lane<r>(rhi, (uint32_t)(dl >> 32));
            });
            if (lane < 8) s.rows[8 * b + lane] = make_uint2(rlo, rhi);
        }
        s.cm[j] = cm;
        uint32_t* rs = f.RS + tile_index(f.NT, it.A, 0) * row_words(Q);
        uint32_t* cs = f.CS + tile_index(f.NT, it.A, 0) * state_words(Q);
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            uint32_t* o = (k < 3 ? rs : cs) + (k % 3) * 128 + 2 * j;
            *reinterpret_cast<uint2*>(o) = make_uint2(lo.p[k], hi.p[k]);
        }
        const uint2 rw = s.rows[j];
        rs[kRowBits + j] = rw.x;
        cs[kRowBits + j] = rw.y;
    }
    __syncthreads();

    int16_t* F = f.F;
    const long long ld = f.ld;
    if (lane < T) {
        const unsigned long long cm = s.cm[lane];
        for (int i = wave; i < T; i += nthr / 64) F[(aT + i) * ld + aT + lane] = (int16_t)__popcll(cm >> i);
    }
}

template <int Q>
__global__ __launch_bounds__(kThreads) void k_diag(const TileWork* __restrict__ items, const uint8_t* staged,
                                                   const uint8_t* codes, int n)
{
    __shared__ DiagLds s;
    diag_body<Q>(items[blockIdx.x], s, threadIdx.x, kThreads, staged, codes, n);
}

// A workgroup barrier for LDS alone.  __syncthreads() also waits for the
// wavefront's global accesses, which would put the latency of the finished
// cells' stores into every block of the pipeline.
__device__ __forceinline__ void lds_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// One between item: rows r0 .. r0+RPW-1 and column j (the lane) of the tile's
// 64x64 maxima, written to its accumulator.  Wavefront w takes the row block
// w % (64/RPW); with NS = 2 the two wavefronts of a row block split the
// groups and merge their maxima through red (64x64 ints of LDS).  Every
// thread of the workgroup must call this.
template <int Q, int RPW, int NS>
__device__ __forceinline__ void between_body(const BetweenWork& it, const uint8_t* Rl,
                                             const uint32_t* RS, const uint32_t* CS, int wave, int j,
                                             uint16_t* red)
{
    constexpr int NB = 64 / RPW;
    static_assert(NS == 1 || NS == 2, "one or two wavefronts per row block");
    const int h = wave / NB;
    const int r0 = (wave - h * NB) * RPW;
    int acc[RPW];
#pragma unroll
    for (int r = 0; r < RPW; ++r) acc[r] = 0;
    between_accumulate<Q, RPW, NS>(acc, Rl, RS, CS, it.f.NT, it.A, it.A + it.d, it.c0, it.c1, r0, j, h);
    if constexpr (NS == 2) {
        if (h == 1) {
#pragma unroll
            for (int r = 0; r < RPW; ++r) red[(r0 + r) * 64 + j] = (uint16_t)acc[r];  // maxima < 2^15
        }
        __syncthreads();
        if (h == 1) return;
#pragma unroll
        for (int r = 0; r < RPW; ++r) acc[r] = max(acc[r], (int)red[(r0 + r) * 64 + j]);
    }

    int32_t* out = it.acc + r0 * 64 + j;
    if (it.atomic) {  // several items share the tile's accumulator
#pragma unroll
        for (int r = 0; r < RPW; ++r) atomicMax(out + r * 64, acc[r]);
    } else {
#pragma unroll
        for (int r = 0; r < RPW; ++r) out[r * 64] = acc[r];
    }
}

// The between items where the finish marks the groups that can matter
// (sparse_between).
//
// A split at m can only raise cell (a, b) over the one below it if base a+1
// pairs with base m in it: else F(a, m) = F(a+1, m) or a split m' < m of
// (a, m), which reaches b as well, does the same.  So of the groups of row a
// only those count that hold a post m whose cell (a, m) rises by its pairing
// alone (the left halves that the sparse folding algorithms call candidates;
// Frid and Gusfield apply the idea to the Four-Russians lookup in "An
// improved Four-Russians method and sparsified Four-Russians algorithm for
// RNA folding").  On iid sequences of 3000 to 6000 bases 18% of the groups
// are left, on repeats at most a third.  The maxima over them are not the
// maxima over all groups, but every cell comes out the same.
//
// Lane = column; kH tells how an item is cut.  kH = 1: one workgroup, eight
// rows a wavefront, four group tiles C at a time.  kH = 2 (the wide shape of
// the fused step): two workgroups with 32 rows each, four rows a wavefront,
// eight tiles at a time.  The tiles' column words go to LDS, a wavefront's row
// words into registers by row (lane 8q + k of word r holds row r, tile q,
// group k), and each row's marks into a scalar word whose set bits are walked
// in batches: the lane read of the row word, the column word's address, the R
// index, the sum, half a max: 4.5 VALU instructions against 2.5 for a group of
// the dense walk, on a fifth of the groups.  A batch is two dependent LDS
// round trips (about 350 cycles), so few and full batches count: with kH = 2 a
// row has 11 marks a turn against 5 to 6, which serves long items (MI355X,
// n = 16000 7.69 -> 7.16 ms); short ones lose with twice the workgroups (4096
// folds of 50..2000 bases 9.11 -> 9.62 ms).
template <int Q, int kH>
struct SparseLds {
    alignas(16) uint32_t col[32 * kH * 64];  // column word of group 8q + k, column j
    // per wavefront: row word of row r, group g at [r][g ^ swizzle(r)] (the
    // transposed stores hit every bank once)
    alignas(16) uint32_t row[8][256];
};

template <int Q, int kH>
__device__ __forceinline__ void between_sparse(const BetweenWork& it, int half, uint8_t* Rl,
                                               const uint8_t* __restrict__ Rg, SparseLds<Q, kH>& s)
{
    static_assert(Q == 8 && (kH == 1 || kH == 2), "eight groups a tile, 64 posts");
    constexpr int RSZ = 1 << (2 * (Q - 1));
    constexpr int SW = state_words(Q);
    constexpr int RW = row_words(Q);
    constexpr int NR = 8 / kH;   // rows a wavefront
    constexpr int NC = 4 * kH;   // tiles at a time
    constexpr int NG = 32 * kH;  // their groups
    using Marks = typename std::conditional<kH == 2, unsigned long long, uint32_t>::type;
    auto swizzle = [](int r) { return kH == 2 ? 16 * r : 8 * (r >> 1); };
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int NT = it.f.NT, A = it.A, B = A + it.d, c1 = it.c1;
    const int r0 = 32 * half + NR * wave;
    const NF_GLOBAL char* RSr = (const NF_GLOBAL char*)it.f.RS;
    const NF_GLOBAL char* CSr = (const NF_GLOBAL char*)it.f.CS;
    const NF_GLOBAL char* LV = (const NF_GLOBAL char*)(it.f.F + mark_row(NT, A) * it.f.ld);
    issue_R<RSZ>(Rl, Rg, kBetweenThreads);

    // The words of the tiles C .. C+NC-1.  Tile numbers and byte offsets fit 32
    // bits (at most 524800 blocks of 2 KB), so an address is the fold's base, a
    // scalar offset and a lane's.  From c1 on nothing is loaded: no mark uses it.
    static_assert(SW == 512 && RW == 512, "2 KB blocks");
    auto index = [&](int a, int d) { return (uint32_t)(d * NT - d * (d - 1) / 2 + a); };
    auto lane_index = [&](int d) { return (uint32_t)(__mul24(d, NT) - (__mul24(d, d - 1) >> 1) + A); };  // of (A, A+d)
    // a row word's lane: tile kH p + rq, row rr, group lane & 7; a mark's: tile mq, row mr
    const int rq = kH == 2 ? lane >> 5 : 0, rr0 = (lane >> 3) & (NR - 1);
    const uint32_t roff = (uint32_t)((lane & 7) * 64 + r0 + rr0) * 4u;
    const int mq = lane & (NC - 1);
    const uint32_t moff = (uint32_t)(r0 + ((lane / NC) & (NR - 1)));
    u32x4 colw[kH];
    uint32_t roww[4], mark;
    auto load = [&](int C) {
#pragma unroll
        for (int i = 0; i < kH; ++i) {
            const int id = kH * wave + i;  // half a tile's column words
            const int cc = C + (id >> 1);
            if (cc < c1)
                colw[i] = *(const NF_GLOBAL u32x4*)(CSr + (index(cc, B - cc) * 2048u + (uint32_t)(id & 1) * 1024u +
                                                           (uint32_t)lane * 16u));
        }
#pragma unroll
        for (int p = 0; p < 4; ++p) {
            const int d = min(C + kH * p + rq, c1 - 1) - A;
            if (C + kH * p < c1)
                roww[p] = *(const NF_GLOBAL uint32_t*)(RSr + ((kH == 2 ? lane_index(d) : index(A, d)) * 2048u + roff));
        }
        mark = *(const NF_GLOBAL uint8_t*)(LV + ((uint32_t)(min(C + mq, c1 - 1) - A) * 64u + moff));
    };
    uint32_t acc[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) acc[r] = 0;
#pragma unroll
    for (int i = 0; i < kH; ++i) colw[i] = u32x4{0u, 0u, 0u, 0u};
#pragma unroll
    for (int p = 0; p < 4; ++p) roww[p] = 0;
    load(it.c0);
    __builtin_amdgcn_s_waitcnt(0);  // the R transfer (and the first words)
    for (int C = it.c0; C < c1; C += NC) {
        __syncthreads();  // the lookups of the tiles before are done
#pragma unroll
        for (int i = 0; i < kH; ++i) *reinterpret_cast<u32x4*>(&s.col[(kH * wave + i) * 256 + 4 * lane]) = colw[i];
        uint32_t* rowl = s.row[wave];
#pragma unroll
        for (int p = 0; p < 4; ++p) rowl[rr0 * NG + (((kH * p + rq) * 8 + (lane & 7)) ^ swizzle(rr0))] = roww[p];
        uint32_t m4 = C + mq < c1 ? mark << (8 * (mq & 3)) : 0u;
        m4 |= (uint32_t)__builtin_amdgcn_mov_dpp((int)m4, 0xB1, 0xF, 0xF, true);  // quad_perm [1,0,3,2]
        m4 |= (uint32_t)__builtin_amdgcn_mov_dpp((int)m4, 0x4E, 0xF, 0xF, true);  // quad_perm [2,3,0,1]
        Marks marks[NR];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            marks[r] = (uint32_t)__builtin_amdgcn_readlane((int)m4, NC * r);
            if constexpr (kH == 2)
                marks[r] |= (Marks)(uint32_t)__builtin_amdgcn_readlane((int)m4, NC * r + 4) << 32;
        }
        if (C + NC < c1) load(C + NC);
        lds_barrier();
        uint32_t vr[NR];  // lane g: row word of row r, group g
#pragma unroll
        for (int r = 0; r < NR; ++r) vr[r] = rowl[r * NG + ((lane & (NG - 1)) ^ swizzle(r))];
#pragma unroll
        for (int r = 0; r < NR; ++r) {
            Marks m = marks[r];
            auto take = [&](auto cnt) {
                constexpr int N = cnt;
                uint32_t rw[N], cw[N], rr[N];
#pragma unroll
                for (int u = 0; u < N; ++u) {
                    int g;
                    if constexpr (kH == 2) {
                        g = __builtin_ctzll(m);
                        __asm__("s_bitset0_b64 %0, %1" : "+s"(m) : "s"(g));
                    } else {
                        g = __builtin_ctz(m);
                        __asm__("s_bitset0_b32 %0, %1" : "+s"(m) : "s"(g));
                    }
                    rw[u] = (uint32_t)__builtin_amdgcn_readlane((int)vr[r], g);
                    cw[u] = s.col[g * 64 + lane];
                }
#pragma unroll
                for (int u = 0; u < N; ++u) rr[u] = Rl[r_index_s(rw[u], cw[u])];
#pragma unroll
                for (int u = 0; u < N; u += 2) {
                    const uint32_t t0 = rw[u] + cw[u] + rr[u];
                    const uint32_t t1 = u + 1 < N ? rw[u + 1] + cw[u + 1] + rr[u + 1] : t0;
                    acc[r] = max3_u16(acc[r], t0, t1);
                }
            };
            constexpr int kMost = 4 * kH;
            int n = kH == 2 ? __builtin_popcountll(m) : __builtin_popcount((uint32_t)m);
            for (; n >= kMost; n -= kMost) take(std::integral_constant<int, kMost>{});
            if constexpr (kH == 2) {
                if (n & 4) take(std::integral_constant<int, 4>{});
            }
            if (n & 2) take(std::integral_constant<int, 2>{});
            if (n & 1) take(std::integral_constant<int, 1>{});
        }
    }
    int32_t* out = it.acc + r0 * 64 + lane;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
        const int v = (int)(acc[r] & 0xffffu);
        if (it.atomic) atomicMax(out + r * 64, v);  // several items share the tile's accumulator
        else out[r * 64] = v;
    }
}

template <int Q>
__global__ __launch_bounds__(kBetweenThreads) void k_between(const BetweenWork* __restrict__ items,
                                                      const uint8_t* __restrict__ Rg)
{
    constexpr int RSZ = 1 << (2 * (Q - 1));
    __shared__ __align__(16) uint8_t Rl[RSZ < 16 ? 16 : RSZ];
    if constexpr (sparse_between(Q)) {
        __shared__ SparseLds<Q, 1> s;
        between_sparse<Q, 1>(items[blockIdx.x], 0, Rl, Rg, s);
    } else {
        const BetweenWork& it = items[blockIdx.x];
        __shared__ uint16_t red[kBetweenSplit == 2 ? 64 * 64 : 1];
        load_R<RSZ>(Rl, Rg, kBetweenThreads);
        __syncthreads();
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        between_body<Q, kRowsPerWave, kBetweenSplit>(it, Rl, it.f.RS, it.f.CS, wave, threadIdx.x & 63, red);
    }
}

// Finish of an off-diagonal tile (A, B), B > A, by 8 wavefronts (512 threads).
//
// Cell X(i, j) = F(AT+i, BT+j) is the maximum of P(i, j), the best split in
// the tiles strictly between A and B (the between maxima of acc and the
// groups of the two end tiles C = A+1, C = B-1), the pairing term, and the
// splits inside tiles A and B.  The rows go bottom-up in bits, as above: a
// cell rises over the one below when P does, when a pairing or a split inside
// the tile says so.  The row below row T-1 is row 0 of tile (A+1, B), finished
// one step ago (or of the main-diagonal tile), and the slacks E carry over from
// there, so no step rebuilds them; V starts empty at the tile's last row.
// (MI355X, against the max-plus closure by all eight wavefronts: n = 6000
// 1.90 -> 1.37 ms, 4096 folds of 50..2000 bases 16.9 -> 10.7 ms.)
//
// The wavefronts form a pipeline over blocks of four rows, one barrier a block:
//   waves 2, 3, 6, 7  look up the end tiles' groups of a block (Eq. 3, one row
//               each) and write its P, two blocks ahead of wave 0.  A row is
//               three LDS round trips, about 570 cycles; with two rows on each
//               of two wavefronts the lookups bounded the pipeline;
//   waves 0, 1  take the rows, columns 0..31 and 32..63: lane 32h + c of wave
//               w holds column 32w + c and the split points 32h .. 32h+31 of
//               both kinds.  Wave 1 needs of wave 0 only the rows' delta bits
//               and follows two blocks behind, so that everything a block
//               reads from LDS is loaded a block ahead and no LDS round trip
//               sits on the rows' chain;
//   waves 4, 5  write the finished block: dense cells and column words, row
//               words.
// A block of the rows is 190 instructions (about 850 cycles: a wavefront
// issues one in four cycles, and the ballots' waits are filled); a fold of few
// tiles a step is bound by the 16 + 3 blocks of this chain.  (MI355X: against
// four wavefronts of 16 columns with all lookups ahead of the rows and all
// writing behind, n = 6000 1.487 -> 1.373 ms, n = 500 119 -> 103 us, q = 5
// n = 3001 926 -> 762 us.)
//
// Staged steps hold hundreds to thousands of finishes, four to a CU, and are
// bound by the VALU (over 70% busy) and not by this chain.  There, at q = 8, the
// lookup wavefronts walk the marked groups as between_sparse does (kWalk): 8
// LDS reads and 18 VALU instructions for up to four groups against 20 and 40
// for all sixteen; and every other workgroup gives the rows to wavefronts 2 and
// 3, so that the rows, the longest role, do not all sit on the first two SIMDs
// (workgroups go to the 8 XCDs in turn, and there to its CUs, so the parity is
// that of the bits above the third).  4096 folds of 50..2000 bases: 9.20 ->
// 9.07 ms by the roles, -> 8.78 ms with the walk.  A fused step keeps the
// plain lookups: rows of many marks take two or three rounds there, longer than
// a block of the rows (n = 3300, planted stems: 680 against 708 us).
constexpr int kTileThreads = 512;
static_assert(kTileThreads == 512, "the tile finish assigns roles to 8 wavefronts");

template <int Q, int kMarks>
struct TileLds {
    static constexpr int G = groups_per_tile(Q);
    // the end tiles' words of a row fit the registers of a wavefront; for
    // other q all of P is looked up before the rows start
    static constexpr bool kPipe = G <= 16;
    static constexpr int NE = 2 * G;                          // end-tile groups
    static constexpr int kES = kPipe ? (NE + 3) / 4 * 4 + 4 : 4;  // 16-byte rows, banks spread
    // rows of bits: [0], [1]: delta(i, .) of the columns 0..31 and 32..63 once
    // finished; [2]: delta of the column left of the tile in bit 31; [3]: zero;
    // [4], [5]: dL(i, .) of the split points 0..31 and 32..63; [6], [7]: the
    // split points below row i among them
    alignas(16) uint32_t W[8][64];
    // the finish marks the groups that a between-group lookup may skip (see mark_row)
    static constexpr bool kSparse = kMarks > 0, kWalk = kMarks > 1;
    uint32_t K[kSparse ? 2 : 1][kSparse ? 64 : 1];  // the columns of row i that rise by their pairing alone
    alignas(16) uint16_t P[16][64][4];            // P(i, j) at [i / 4][j][i % 4]
    alignas(16) uint32_t EB[kPipe ? 64 : 1][kES];  // EB[i][e*G + k]: row word of row i, group k of end tile e
    uint32_t CW[kWalk ? NE + 1 : 1][kWalk ? 64 : 1];  // end-tile column words [e*G + k][column], then zeros
};

// max(0, P - x) of the P in the low or high half of pair, nonzero when P > x
// (one SDWA instruction; both are below 2^15)
template <int kHalf>
__device__ __forceinline__ uint32_t above(uint32_t pair, uint32_t x)
{
    uint32_t d;
    if constexpr (kHalf == 0)
        __asm__("v_sub_u16_sdwa %0, %1, %2 clamp dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_0 src1_sel:WORD_0"
                : "=v"(d)
                : "v"(pair), "v"(x));
    else
        __asm__("v_sub_u16_sdwa %0, %1, %2 clamp dst_sel:DWORD dst_unused:UNUSED_PAD src0_sel:WORD_1 src1_sel:WORD_0"
                : "=v"(d)
                : "v"(pair), "v"(x));
    return d;
}

// The finish of one tile by kTileThreads threads.  R is copied from Rg
// (global) into Rl.  kMarks: 1 writes the marks, 2 also has the lookup
// wavefronts walk the marked groups only (kWalk).
// flip (0 or 1): the roles of wavefronts w and w ^ 2 change places.
template <int Q, int kMarks>
__device__ __forceinline__ void tile_body(const TileWork& it, int flip, uint8_t* Rl, const uint8_t* __restrict__ Rg,
                                          TileLds<Q, kMarks>& s)
{
    using Lds = TileLds<Q, kMarks>;
    constexpr bool kWalk = Lds::kWalk;
    constexpr int M = Q - 1;
    constexpr int G = groups_per_tile(Q);
    constexpr int T = tile_size(Q);
    constexpr int SW = state_words(Q);
    constexpr int RW = row_words(Q);
    constexpr int RSZ = 1 << (2 * M);
    constexpr int NE = Lds::kPipe ? Lds::NE : 4;
    constexpr int NE4 = (NE + 3) / 4 * 4;

    const FoldDesc& f = it.f;
    const int A = it.A, d = it.d, B = A + d;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane((tid >> 6) ^ (2 * flip));
    const int lane = tid & 63;
    const long long ld = f.ld;
    const int aT = A * T, bT = B * T;
    const NF_GLOBAL int16_t* F = (const NF_GLOBAL int16_t*)f.F;
    const NF_GLOBAL uint8_t* codes = (const NF_GLOBAL uint8_t*)f.codes;
    const NF_GLOBAL uint32_t* RSr = (const NF_GLOBAL uint32_t*)f.RS;
    const NF_GLOBAL uint32_t* CSr = (const NF_GLOBAL uint32_t*)f.CS;
    NF_GLOBAL uint32_t* rsB = (NF_GLOBAL uint32_t*)f.RS + tile_index(f.NT, B, 0) * RW;
    NF_GLOBAL uint32_t* csB = (NF_GLOBAL uint32_t*)f.CS + tile_index(f.NT, B, 0) * SW;
    NF_GLOBAL int32_t* acc = (NF_GLOBAL int32_t*)it.acc;
    const bool between = it.nslot > 0;

    // ---- set-up.  Every global load goes out before the first LDS store of
    // loaded data (which waits for it), so that the tile pays about one memory
    // round trip here.
    issue_R<RSZ>(Rl, Rg, kTileThreads);
    constexpr int kLines = Lds::kPipe ? (NE + 7) / 8 : 1;
    uint32_t line[kLines];  // row words of end-tile group wave + 8u, row `lane` (0 where the end tile does not exist)
    if constexpr (Lds::kPipe) {
#pragma unroll
        for (int u = 0; u < kLines; ++u) {
            const int x = wave + 8 * u;
            const int e = x >= G ? 1 : 0, k = x - e * G;
            line[u] = 0;
            if (x < NE && d >= 2 + e) line[u] = (RSr + tile_index(f.NT, A, e == 0 ? 1 : d - 1) * RW + k * 64)[(unsigned)lane];
        }
    }
    auto store_lines = [&] {
        if constexpr (Lds::kPipe) {
#pragma unroll
            for (int u = 0; u < kLines; ++u)
                if (wave + 8 * u < NE4) s.EB[lane][wave + 8 * u] = line[u];
            if constexpr (NE4 > 8 * kLines) {
                if (wave < NE4 - 8 * kLines) s.EB[lane][8 * kLines + wave] = 0;
            }
        }
    };
    // the end of the set-up: R and the LDS stores are complete
    auto set_up_done = [&] {
        if constexpr (RSZ >= 1024) __builtin_amdgcn_s_waitcnt(0);
        __syncthreads();
    };
    if constexpr (!Lds::kPipe) {
        // all of P, rows 8 wave .. 8 wave + 7
        set_up_done();
        int pr[8];
        const int r0 = 8 * wave;
#pragma unroll
        for (int r = 0; r < 8; ++r) pr[r] = between ? (acc + (r0 + r) * 64)[(unsigned)lane] : 0;
        if (d >= 2) between_accumulate<Q, 8, 1>(pr, Rl, f.RS, f.CS, f.NT, A, B, A + 1, A + 2, r0, lane, 0);
        if (d >= 3) between_accumulate<Q, 8, 1>(pr, Rl, f.RS, f.CS, f.NT, A, B, B - 1, B, r0, lane, 0);
#pragma unroll
        for (int r = 0; r < 8; ++r) {
            if (between) (acc + (r0 + r) * 64)[(unsigned)lane] = 0;
            s.P[2 * wave + (r >> 2)][lane][r & 3] = (T == 64 || lane < T) ? (uint16_t)pr[r] : (uint16_t)0;
        }
    }
    // Phase p of the pipeline: wave 0 takes block 15 - p, wave 1 block
    // 15 - (p - 2), the lookups run for block 15 - (p + 2), the writing for
    // block 15 - (p - 3).  Every wavefront passes the same barriers: one after
    // the set-up, one after the first two blocks' P, one after each phase but
    // the last.
    constexpr int kPhases = 19;
    const int h = lane >> 5, c = lane & 31;

    if (wave < 2) {
        // ---- the rows
        const int j = 32 * wave + c;
        Slack E{}, V{};
        uint32_t left = 0, x = 0;
        const uint32_t* src = s.W[3];   // delta bits of the columns to the left
        const uint32_t* dsrc = s.W[3];  // dL
        const uint32_t* vsrc = s.W[3];  // the split points of tile A below the row
        // the split points of this lane left of column j
        const uint32_t below = j >= T ? 0u : (j >= 32 * h + 32 ? ~0u : (j > 32 * h ? (1u << (j - 32 * h)) - 1 : 0u));
        uint32_t vrE = below;
        const uint32_t own = h == wave ? ~0u : 0u, ownb = own & below;
#pragma unroll
        for (int k = 0; k < 6; ++k) E.p[k] = (k < 3 ? rsB : csB)[(k % 3) * 128 + 2 * j + h] & below;
        unsigned long long pm = pair_rows(lane < T ? (int)codes[aT + lane] : 4, (int)codes[bT + j - 1]);
        if (j < T) {
            if (j > 0 && ((j - 1) >> 5) == h) left = 1u << ((j - 1) & 31);
            x = (uint32_t)(int)F[(aT + T) * ld + bT + j];
            if (h < wave) src = s.W[0];
            dsrc = s.W[4 + h];
            vsrc = s.W[6 + h];
            if (j == 0 && h == 1) {
                // column 0: the column left of the tile is its split point -1,
                // bit 31 here, with slack X(T, 0) - X(T, -1)
                const int xl = d == 1 ? (int)x : (int)F[(aT + T) * ld + bT - 1];
                E.p[0] = ((int)x > xl) ? 1u << 31 : 0u;
                vrE = left = 1u << 31;
                src = s.W[2];
            }
        } else {
            pm = 0;
        }
        E.begin();
        V.begin();
        store_lines();
        set_up_done();
        lds_barrier();
        // what a block reads from LDS, loaded at the end of the block before it
        uint2 pw;
        uint4 dw, sw, vw;
        auto fetch = [&](int b) {
            pw = *reinterpret_cast<const uint2*>(&s.P[b][j][0]);
            dw = *reinterpret_cast<const uint4*>(dsrc + 4 * b);
            sw = *reinterpret_cast<const uint4*>(src + 4 * b);
            vw = *reinterpret_cast<const uint4*>(vsrc + 4 * b);
        };
        if (wave == 1) {  // two phases behind
            lds_barrier();
            lds_barrier();
        }
        fetch(15);
        // One row: 40 instructions.  Its chain goes twice through a ballot
        // (VALU to scalar and back, 16 idle cycles each); the ripples of the
        // row before fill those.  With four words the blocks run until a slack
        // of 12 or more shows up, and the rest of the tile with six.
        int b = 15;
        bool small = __ballot((E.large() | V.large()) != 0) == 0;
        auto blocks = [&](auto words) {
            constexpr int W = words;
            while (b >= 0 && (W == 6 || small)) {
                const uint32_t pmb = (uint32_t)(pm >> (4 * b));
                uint32_t rows = 0;    // lane r: delta(4b + r, .) of this wavefront's columns
                uint32_t firsts = 0;  // lane r: the columns that rise by their pairing alone
                uint32_t cE = 0, cV = 0, up = 0;
                const uint32_t ps[2] = {pw.x, pw.y};
                const uint32_t ds[4] = {dw.x, dw.y, dw.z, dw.w};
                const uint32_t ss[4] = {sw.x, sw.y, sw.z, sw.w};
                const uint32_t vs[4] = {vw.x, vw.y, vw.z, vw.w};
                rows_down<3>([&](auto rc) {
                    constexpr int r = rc;
                    if (T == 64 || 4 * b + r < T) {
                        const uint32_t up_p = above<r & 1>(ps[r >> 1], x);
                        const uint32_t pair = bit_mask(pmb, r) & left;
                        const uint32_t v = bits3<(kA & kB) | kC>(V.zero, ds[r], up_p);
                        const uint32_t split = bits3<(kA & kB) | kC>(E.zero, ss[r], v);
                        unsigned long long bs = 0;
                        if constexpr (Lds::kSparse) bs = __ballot(split != 0);
                        const unsigned long long b1 = __ballot(bits3<(kA & kB) | kC>(E.zero, pair, split) != 0);
                        __builtin_amdgcn_sched_barrier(0);
                        if (r < 3) E.ripple<W>(cE, up);
                        __builtin_amdgcn_sched_barrier(0);
                        const uint32_t st = (uint32_t)b1 | (uint32_t)(b1 >> 32);
                        const unsigned long long b2 = __ballot(bits3<kA & kB & kC>(E.zero, st, ownb) != 0);
                        __builtin_amdgcn_sched_barrier(0);
                        if (r < 3) V.ripple<W>(cV, up);
                        __builtin_amdgcn_sched_barrier(0);
                        const uint32_t cl = (uint32_t)b2 | (uint32_t)(b2 >> 32);
                        const uint32_t dl = st | cl;
                        if constexpr (Lds::kSparse)
                            firsts = with_lane<r>(firsts, st & ~((uint32_t)bs | (uint32_t)(bs >> 32) | cl));
                        up = bit_mask(dl, c);
                        cE = bits3<(kA ^ kB) & kC>(up, bits3<kA | (kB & kC)>(ss[r], dl, own), vrE);
                        cV = bits3<(kA ^ kB) & kC>(up, ds[r], vs[r]);
                        E.mark(cE, up);
                        V.mark(cV, up);
                        x -= up;
                        rows = with_lane<r>(rows, dl);
                    }
                });
                if (lane < 4) {
                    s.W[wave][4 * b + lane] = rows;
                    if constexpr (Lds::kSparse) s.K[wave][4 * b + lane] = firsts;
                }
                // The barrier below waits for the stores of W and K, not for the
                // loads behind them: LDS accesses of a wavefront complete in
                // order, and fetch() is four of them.  So these must stay
                // behind the stores (the next line: no memory access may cross
                // it) and be four on every way to the barrier (those of the
                // last block are used after the blocks).  A test looks at the
                // built code.
                __asm__ volatile("" ::: "memory");
                --b;
                fetch(b >= 0 ? b : 0);
                __builtin_amdgcn_sched_barrier(0);
                E.ripple<W>(cE, up);
                V.ripple<W>(cV, up);
                if (W == 4) small = __ballot((E.large() | V.large()) != 0) == 0;
                __asm__ volatile("s_waitcnt lgkmcnt(4)\n\ts_barrier" ::: "memory");
            }
        };
        blocks(std::integral_constant<int, 4>{});
        blocks(std::integral_constant<int, 6>{});
        __asm__ volatile("" ::"v"(pw.x), "v"(dw.x), "v"(sw.x), "v"(vw.x));  // (see above)
        // the slacks for the next step's tile of this column
#pragma unroll
        for (int k = 0; k < 6; ++k) (k < 3 ? rsB : csB)[(k % 3) * 128 + 2 * j + h] = E.p[k];
        for (int p = 16 + 2 * wave; p < kPhases - 1; ++p) lds_barrier();
    } else if ((wave & 2) != 0) {
        // ---- the lookups: P of row 4b + r0, column `lane`
        const int r0 = (wave & 1) + ((wave >> 1) & 2);
        // the end tiles' column words (kWalk: this wavefront's share, for LDS);
        // group x = e*G + k is of tile (A+1, B) or (B-1, B)
        constexpr int kCW = kWalk ? NE4 / 4 : NE4;
        uint32_t cw[kCW];
        uint32_t marks = 0;  // kWalk: the marked groups of row `lane`
        uint32_t words = 0;  // kWalk: row word of group `lane` of the row to come
        uint32_t m0 = 0, m1 = 0, m2 = 0;
        auto maximum = [&](int b) -> uint32_t {
            return between ? (uint32_t)(acc + (4 * b + r0) * 64)[(unsigned)lane] : 0u;
        };
        if constexpr (Lds::kPipe) {
#pragma unroll
            for (int u = 0; u < kCW; ++u) {
                const int x = kWalk ? kCW * r0 + u : u;
                const int e = x >= G ? 1 : 0, k = x - e * G;
                cw[u] = 0;
                if (x < NE && d >= 2 + e)
                    cw[u] = (CSr + tile_index(f.NT, e == 0 ? A + 1 : B - 1, e == 0 ? d - 1 : 1) * SW + k * 64)[(unsigned)lane];
            }
            if constexpr (kWalk) {
                const NF_GLOBAL uint8_t* LV = (const NF_GLOBAL uint8_t*)(F + mark_row(f.NT, A) * ld);
                const uint32_t k0 = d >= 2 ? (LV + 64)[(unsigned)lane] : 0u;
                const uint32_t k1 = d >= 3 ? (LV + (d - 1) * 64)[(unsigned)lane] : 0u;
                marks = k0 | (k1 << G);
            }
            m0 = maximum(15);
            m1 = maximum(14);
            m2 = maximum(13);
        }
        [[maybe_unused]] auto fetch_words = [&](int b) { words = s.EB[4 * b + r0][lane < NE ? lane : NE]; };
        auto look_up = [&](int b, uint32_t m) {
            if constexpr (kWalk) {
                uint32_t left = (uint32_t)__builtin_amdgcn_readlane((int)marks, 4 * b + r0);
                while (left != 0) {
                    uint32_t rw[4], w[4], rr[4];
#pragma unroll
                    for (int u = 0; u < 4; ++u) {
                        const uint32_t x = (uint32_t)__builtin_ctz(left | (1u << NE));  // NE: the zero words
                        left &= ~(1u << x);
                        rw[u] = (uint32_t)__builtin_amdgcn_readlane((int)words, (int)x);
                        w[u] = s.CW[x][lane];
                    }
#pragma unroll
                    for (int u = 0; u < 4; ++u) rr[u] = Rl[r_index_s(rw[u], w[u])];
#pragma unroll
                    for (int u = 0; u < 4; u += 2)
                        m = max3_u16(m, rw[u] + w[u] + rr[u], rw[u + 1] + w[u + 1] + rr[u + 1]);
                }
                s.P[b][lane][r0] = (uint16_t)m;
                if (b > 0) fetch_words(b - 1);
            } else {
                const uint32_t* eb = s.EB[4 * b + r0];
                uint32_t rw[NE4], rr[NE4];
#pragma unroll
                for (int u = 0; u < NE4; u += 4) {
                    const uint4 w = *reinterpret_cast<const uint4*>(eb + u);
                    rw[u] = w.x;
                    rw[u + 1] = w.y;
                    rw[u + 2] = w.z;
                    rw[u + 3] = w.w;
                }
#pragma unroll
                for (int u = 0; u < NE4; ++u) rr[u] = Rl[r_index_v(rw[u], cw[u])];
                __builtin_amdgcn_sched_barrier(0);  // every gather is out before the first sum waits
#pragma unroll
                for (int u = 0; u < NE4; u += 2)
                    m = max3_u16(m, rw[u] + cw[u] + rr[u], rw[u + 1] + cw[u + 1] + rr[u + 1]);
                s.P[b][lane][r0] = (T == 64 || lane < T) ? (uint16_t)m : (uint16_t)0;
            }
        };
        if constexpr (kWalk) {
#pragma unroll
            for (int x = 0; x < kCW; ++x) s.CW[kCW * r0 + x][lane] = cw[x];
            if (r0 == 0) s.CW[NE][lane] = 0;
            if (r0 == 1) s.EB[lane][NE] = 0;
        }
        store_lines();
        set_up_done();
        if constexpr (Lds::kPipe) {
            if constexpr (kWalk) fetch_words(15);
            look_up(15, m0);
            look_up(14, m1);
        }
        lds_barrier();
        m0 = m2;
        for (int b = 13; b > 0; b -= 2) {  // (two registers in turn: one would be copied, and waited for, each time)
            if constexpr (Lds::kPipe) {
                m1 = maximum(b - 1);
                look_up(b, m0);
            }
            lds_barrier();
            if constexpr (Lds::kPipe) {
                m0 = maximum(b > 1 ? b - 2 : 0);
                look_up(b - 1, m1);
            }
            lds_barrier();
        }
        if (Lds::kPipe && between) {  // the accumulator is handed back zeroed for its next use
#pragma unroll
            for (int b = 0; b < 16; ++b) (acc + (4 * b + r0) * 64)[(unsigned)lane] = 0;
        }
        for (int p = 14; p < kPhases - 1; ++p) lds_barrier();
    } else {
        // ---- the tables of the rows (the rows' bits of tile (A, A), the
        // halo), then the finished blocks' cells and words
        const long long t_idx = tile_index(f.NT, A, d);
        int top = lane < T ? (int)F[(aT + T) * ld + bT + lane] : 0;  // X of the row below
        if (wave == 4) {
            const uint32_t lo = (RSr + tile_index(f.NT, A, 0) * RW)[kRowBits + lane];
            const uint32_t hi = (CSr + tile_index(f.NT, A, 0) * SW)[kRowBits + lane];
            s.W[3][lane] = 0;
            s.W[4][lane] = lane < T ? lo : 0u;
            s.W[5][lane] = lane < T ? hi : 0u;
        } else {
            uint32_t m = 0;
            if (lane < T) {
                // nothing lies below row T-1 left of tile (B, B)
                const int up = F[(aT + lane) * ld + bT - 1];
                const int dn = (d == 1 && lane == T - 1) ? 0 : (int)F[(aT + lane + 1) * ld + bT - 1];
                if (up > dn) m = 1u << 31;
            }
            const unsigned long long pts = ((T == 64 ? ~0ull : (1ull << T) - 1) >> lane >> 1) << lane << 1;
            s.W[2][lane] = m;
            s.W[6][lane] = (uint32_t)pts;
            s.W[7][lane] = (uint32_t)(pts >> 32);
        }
        store_lines();
        set_up_done();
        for (int p = -1; p < 3; ++p) lds_barrier();
        if (wave == 4) {
            NF_GLOBAL int16_t* Fw = (NF_GLOBAL int16_t*)f.F;
            NF_GLOBAL uint32_t* CSw = (NF_GLOBAL uint32_t*)(f.CS + t_idx * SW);
            uint32_t cbits = 0;  // the rows' bits at this column, the last row in bit 0
            [[maybe_unused]] NF_GLOBAL uint32_t* LVw = (NF_GLOBAL uint32_t*)(Fw + mark_row(f.NT, A) * ld) + d * 16;
#pragma unroll 2
            for (int b = 15; b >= 0; --b) {
                if constexpr (Lds::kSparse) {
                    // lane 8r + k: group k of row 4b + r
                    const uint32_t kw = s.K[(lane >> 2) & 1][4 * b + ((lane >> 3) & 3)];
                    const unsigned long long live = __ballot(((kw >> (8 * (lane & 3))) & 0xffu) != 0);
                    if (lane == 0) LVw[b] = (uint32_t)live;
                }
                const uint4 w = *reinterpret_cast<const uint4*>(&s.W[h][4 * b]);
                const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
                rows_down<3>([&](auto rc) {
                    constexpr int r = rc;
                    const int i = 4 * b + r;
                    if (T == 64 || i < T) {
                        const uint32_t bit = (ws[r] >> c) & 1u;
                        top += (int)bit;
                        cbits = (cbits << 1) | bit;
                        if (T == 64 || lane < T) (Fw + (long long)(aT + i) * ld + bT)[(unsigned)lane] = (int16_t)top;
                        // the rows of group i / Q are complete (columns >= T: all zero)
                        if (i % Q == 0)
                            CSw[i / Q * 64 + lane] = ((cbits & ((1u << M) - 1u)) << 16) | (uint32_t)top;
                    }
                });
                if (b > 0) lds_barrier();
            }
        } else {
            NF_GLOBAL uint32_t* RSw = (NF_GLOBAL uint32_t*)(f.RS + t_idx * RW);
            unsigned long long H = __ballot(top > __shfl_up(top, 1));  // differences along the row (column 0's is not used)
#pragma unroll 2
            for (int b = 15; b >= 0; --b) {
                const uint4 w = *reinterpret_cast<const uint4*>(&s.W[h][4 * b]);
                const uint32_t ws[4] = {w.x, w.y, w.z, w.w};
                // four rows of a group's row words are 16 bytes.  Padding rows
                // get zero words: readers load whole 64-row lines and zero
                // keeps their sums bounded and R in range
                uint32_t rw[4] = {0u, 0u, 0u, 0u};
                rows_down<3>([&](auto rc) {
                    constexpr int r = rc;
                    if (T == 64 || 4 * b + r < T) {
                        const unsigned long long dl =
                            (unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)ws[r], 0) |
                            ((unsigned long long)(uint32_t)__builtin_amdgcn_readlane((int)ws[r], 32) << 32);
                        H ^= dl ^ (dl << 1);
                        top += (int)((ws[r] >> c) & 1u);
                        const uint32_t hb = (uint32_t)((H >> lane) >> 1) & ((1u << M) - 1u);
                        rw[r] = ((hb << M) << 16) | (uint32_t)top;
                    }
                });
                if (lane % Q == 0 && lane < T)
                    *(NF_GLOBAL u32x4*)(RSw + lane / Q * 64 + 4 * b) = u32x4{rw[0], rw[1], rw[2], rw[3]};
                if (b > 0) lds_barrier();
            }
        }
    }
}

// Tile finishes alone (staged steps).
template <int Q>
__global__ __launch_bounds__(kTileThreads) void k_tile(const TileWork* __restrict__ items, const uint8_t* __restrict__ Rg)
{
    constexpr int RSZ = 1 << (2 * (Q - 1));
    __shared__ __align__(16) uint8_t Rl[RSZ < 16 ? 16 : RSZ];
    constexpr int kMarks = sparse_between(Q) ? 2 : 0;
    __shared__ __align__(16) TileLds<Q, kMarks> s;
    tile_body<Q, kMarks>(items[blockIdx.x], __builtin_popcount(blockIdx.x >> 3) & 1, Rl, Rg, s);
}

// One wavefront step in one launch: workgroups [0, ntile) finish the tiles
// of diagonal s, the rest run the between chunks of diagonal s+1 (which only
// read diagonals <= s-1 and write the other half of the accumulators), one
// workgroup each, or two in the wide shape (kH = 1 or 2 of between_sparse, q =
// 8).  kH = 0: without marks, every group looked up.
template <int Q, int kH>
__global__ __launch_bounds__(kTileThreads) void k_stage(const TileWork* __restrict__ titems, int ntile,
                                                        const BetweenWork* __restrict__ bitems,
                                                        const uint8_t* __restrict__ Rg)
{
    constexpr int RSZ = 1 << (2 * (Q - 1));
    __shared__ __align__(16) uint8_t Rl[RSZ < 16 ? 16 : RSZ];
    const int b = blockIdx.x;
    if constexpr (kH > 0) {
        __shared__ union Lds {
            TileLds<Q, 1> tile;
            SparseLds<Q, kH> between;
        } s;
        if (b < ntile)
            tile_body<Q, 1>(titems[b], 0, Rl, Rg, s.tile);
        else
            between_sparse<Q, kH>(bitems[(b - ntile) / kH], (b - ntile) % kH, Rl, Rg, s.between);
    } else {
        __shared__ __align__(16) TileLds<Q, 0> s;
        if (b < ntile) {
            tile_body<Q, 0>(titems[b], 0, Rl, Rg, s);
        } else {
            load_R<RSZ>(Rl, Rg, kTileThreads);
            __syncthreads();
            const BetweenWork& it = bitems[b - ntile];
            const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
            between_body<Q, 16, kTileThreads / 64 / 4>(it, Rl, it.f.RS, it.f.CS, wave, threadIdx.x & 63,
                                                       &s.P[0][0][0]);
        }
    }
}

__global__ void k_scores(const FoldDesc* __restrict__ folds, int nfolds, int32_t* __restrict__ scores)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < nfolds) scores[e] = folds[e].F[folds[e].n];  // F(0, n) = D(1, n)
}

// The same, each score to scores[fold.pad] (the serving engine's slots in
// mapped host memory).
__global__ void k_scores_to_slots(const FoldDesc* __restrict__ folds, int nfolds, int32_t* __restrict__ scores)
{
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e < nfolds) scores[folds[e].pad] = folds[e].F[folds[e].n];
}

// S[i*n + j] = D(i+1, j+1) = F(i, j+1) for i <= j, 0 below the diagonal, and
// the score F(0, n) where asked for.  A thread writes 8 consecutive entries of
// S (two rows' at a row's end): with kVec as one 16-byte store (S is 16-byte
// aligned; a row of S need not be), the entries of F by 16-byte loads at their
// 2-byte alignment where the 8 lie in one row.  The copy moves 2 n^2 bytes out
// and n^2 in and is bound by memory; 2-byte stores at an 8-byte stride took
// twice as long (MI355X, n = 16000: 335 us).
struct __attribute__((packed, aligned(2))) Row8 {
    int16_t v[8];
};
template <bool kVec>
__global__ __launch_bounds__(256) void k_expand(const int16_t* __restrict__ F, int ld, int n,
                                                int16_t* __restrict__ S, int32_t* __restrict__ score)
{
    const uint32_t e0 = (blockIdx.x * 256u + threadIdx.x) * 8u, end = (uint32_t)n * (uint32_t)n;
    if (score != nullptr && blockIdx.x == 0 && threadIdx.x == 0) *score = F[n];
    if (e0 >= end) return;
    uint32_t i = e0 / (uint32_t)n, j = e0 - i * (uint32_t)n;
    Row8 o;
    if (j + 8 <= (uint32_t)n) {
        if (j + 7 < i) {
#pragma unroll
            for (int u = 0; u < 8; ++u) o.v[u] = 0;
        } else {
            // (columns j+1 .. j+8 <= n of row i: inside the table)
            o = *reinterpret_cast<const Row8*>(F + (long long)i * ld + 1 + j);
#pragma unroll
            for (int u = 0; u < 8; ++u)
                if (j + u < i) o.v[u] = 0;
        }
    } else {
#pragma unroll
        for (int u = 0; u < 8; ++u) {
            o.v[u] = (e0 + u < end && j >= i) ? F[(long long)i * ld + 1 + j] : (int16_t)0;
            if (++j == (uint32_t)n) {
                j = 0;
                ++i;
            }
        }
    }
    if (kVec && e0 + 8 <= end) {
        *reinterpret_cast<uint4*>(S + e0) = __builtin_bit_cast(uint4, o);
    } else {
#pragma unroll
        for (int u = 0; u < 8; ++u)
            if (e0 + u < end) S[e0 + u] = o.v[u];
    }
}

// Launch on stream s; with events, the dispatch itself records e0 when the
// kernel starts and e1 when it ends (kernel-only durations for profiling).
template <class K, class... Args>
hipError_t launch_k(K kernel, dim3 grid, dim3 block, hipStream_t s, hipEvent_t e0, hipEvent_t e1, Args... args)
{
    if (e0 || e1)
        hipExtLaunchKernelGGL(kernel, grid, block, 0, s, e0, e1, 0, args...);
    else
        hipLaunchKernelGGL(kernel, grid, block, 0, s, args...);
    return hipGetLastError();
}

template <int Q>
hipError_t launch_q(int which, const void* items, int nitems, const uint8_t* R, hipStream_t s, hipEvent_t e0,
                    hipEvent_t e1)
{
    if (nitems <= 0) return hipSuccess;
    dim3 grid(nitems);
    // (for the main-diagonal tiles R carries the staged codes of admission, or null)
    if (which == 0)
        return launch_k(k_diag<Q>, grid, dim3(kThreads), s, e0, e1, (const TileWork*)items, R, (const uint8_t*)nullptr, -1);
    if (which == 1) return launch_k(k_tile<Q>, grid, dim3(kTileThreads), s, e0, e1, (const TileWork*)items, R);
    return launch_k(k_between<Q>, grid, dim3(kBetweenThreads), s, e0, e1, (const BetweenWork*)items, R);
}

hipError_t dispatch(int q, int which, const void* items, int nitems, const uint8_t* R, hipStream_t s, hipEvent_t e0,
                    hipEvent_t e1)
{
    switch (q) {
    case 1: return launch_q<1>(which, items, nitems, R, s, e0, e1);
    case 2: return launch_q<2>(which, items, nitems, R, s, e0, e1);
    case 3: return launch_q<3>(which, items, nitems, R, s, e0, e1);
    case 4: return launch_q<4>(which, items, nitems, R, s, e0, e1);
    case 5: return launch_q<5>(which, items, nitems, R, s, e0, e1);
    case 6: return launch_q<6>(which, items, nitems, R, s, e0, e1);
    case 7: return launch_q<7>(which, items, nitems, R, s, e0, e1);
    case 8: return launch_q<8>(which, items, nitems, R, s, e0, e1);
    case 9: return launch_q<9>(which, items, nitems, R, s, e0, e1);
    default: return hipErrorInvalidValue;
    }
}

}  // namespace

hipError_t launch_precompute_R(int q, uint8_t* R, hipStream_t s)
{
    if (q < 1 || q > 9) return hipErrorInvalidValue;
    const int entries = 1 << (2 * (q - 1));
    hipLaunchKernelGGL(k_precompute_R, dim3((entries + 255) / 256), dim3(256), 0, s, q, R);
    return hipGetLastError();
}

hipError_t launch_copy_codes(const uint8_t* src, int n, uint8_t* dst, int padded, hipStream_t s)
{
    if (padded <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_copy_codes, dim3((padded + 255) / 256), dim3(256), 0, s, src, n, dst, padded);
    return hipGetLastError();
}

hipError_t launch_diag(int q, const TileWork* items, int nitems, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    return dispatch(q, 0, items, nitems, nullptr, s, e0, e1);
}

namespace {
template <int Q>
hipError_t diag_codes_q(const TileWork* items, int nitems, const uint8_t* codes, int n, hipStream_t s)
{
    return launch_k(k_diag<Q>, dim3(nitems), dim3(kThreads), s, nullptr, nullptr, items, (const uint8_t*)nullptr, codes, n);
}
}  // namespace

hipError_t launch_diag_codes(int q, const TileWork* items, int nitems, const uint8_t* codes, int n, hipStream_t s)
{
    if (nitems <= 0) return hipSuccess;
    switch (q) {
    case 1: return diag_codes_q<1>(items, nitems, codes, n, s);
    case 2: return diag_codes_q<2>(items, nitems, codes, n, s);
    case 3: return diag_codes_q<3>(items, nitems, codes, n, s);
    case 4: return diag_codes_q<4>(items, nitems, codes, n, s);
    case 5: return diag_codes_q<5>(items, nitems, codes, n, s);
    case 6: return diag_codes_q<6>(items, nitems, codes, n, s);
    case 7: return diag_codes_q<7>(items, nitems, codes, n, s);
    case 8: return diag_codes_q<8>(items, nitems, codes, n, s);
    case 9: return diag_codes_q<9>(items, nitems, codes, n, s);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_diag_admit(int q, const TileWork* items, int nitems, const uint8_t* staged, hipStream_t s)
{
    return dispatch(q, 0, items, nitems, staged, s, nullptr, nullptr);
}

hipError_t launch_tile(int q, const TileWork* items, int nitems, const uint8_t* R, hipStream_t s, hipEvent_t e0,
                       hipEvent_t e1)
{
    return dispatch(q, 1, items, nitems, R, s, e0, e1);
}

hipError_t launch_between(int q, const BetweenWork* items, int nitems, const uint8_t* R, hipStream_t s, hipEvent_t e0,
                          hipEvent_t e1)
{
    return dispatch(q, 2, items, nitems, R, s, e0, e1);
}

hipError_t launch_scores(const FoldDesc* folds, int nfolds, int32_t* scores, hipStream_t s)
{
    if (nfolds <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_scores, dim3((nfolds + 255) / 256), dim3(256), 0, s, folds, nfolds, scores);
    return hipGetLastError();
}

hipError_t launch_scores_to_slots(const FoldDesc* folds, int nfolds, int32_t* scores, hipStream_t s)
{
    if (nfolds <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_scores_to_slots, dim3((nfolds + 255) / 256), dim3(256), 0, s, folds, nfolds, scores);
    return hipGetLastError();
}

namespace {
template <int Q>
hipError_t stage_q(const TileWork* t, int nt, const BetweenWork* b, int nb, const uint8_t* R, hipStream_t s,
                   hipEvent_t e0, hipEvent_t e1)
{
    return launch_k(k_stage<Q, 0>, dim3(nt + nb), dim3(kTileThreads), s, e0, e1, t, nt, b, R);
}
}  // namespace

hipError_t launch_stage(int q, int shape, const TileWork* titems, int ntile, const BetweenWork* bitems, int nbtw,
                        const uint8_t* R, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    if (ntile + nbtw <= 0) return hipSuccess;
    if (shape == kStageMarks && q == 8)
        return launch_k(k_stage<8, 1>, dim3(ntile + nbtw), dim3(kTileThreads), s, e0, e1, titems, ntile, bitems, R);
    if (shape == kStageWide && q == 8)
        return launch_k(k_stage<8, 2>, dim3(ntile + 2 * nbtw), dim3(kTileThreads), s, e0, e1, titems, ntile, bitems, R);
    switch (q) {
    case 1: return stage_q<1>(titems, ntile, bitems, nbtw, R, s, e0, e1);
    case 2: return stage_q<2>(titems, ntile, bitems, nbtw, R, s, e0, e1);
    case 3: return stage_q<3>(titems, ntile, bitems, nbtw, R, s, e0, e1);
    case 4: return stage_q<4>(titems, ntile, bitems, nbtw, R, s, e0, e1);
    case 5: return stage_q<5>(titems, ntile, bitems, nbtw, R, s, e0, e1);
    case 6: return stage_q<6>(titems, ntile, bitems, nbtw, R, s, e0, e1);
    case 7: return stage_q<7>(titems, ntile, bitems, nbtw, R, s, e0, e1);
    case 8: return stage_q<8>(titems, ntile, bitems, nbtw, R, s, e0, e1);
    case 9: return stage_q<9>(titems, ntile, bitems, nbtw, R, s, e0, e1);
    default: return hipErrorInvalidValue;
    }
}

hipError_t launch_expand(const int16_t* F, int ld, int n, int16_t* S, hipStream_t s, int32_t* score)
{
    if (n <= 0) return hipSuccess;
    const uint32_t end = (uint32_t)n * (uint32_t)n;  // n <= 65534: below 2^32
    const dim3 grid((end - 1) / 2048 + 1);
    if (((uintptr_t)S & 15) == 0)
        hipLaunchKernelGGL(k_expand<true>, grid, dim3(256), 0, s, F, ld, n, S, score);
    else
        hipLaunchKernelGGL(k_expand<false>, grid, dim3(256), 0, s, F, ld, n, S, score);
    return hipGetLastError();
}

}  // namespace nf
