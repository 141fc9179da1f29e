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
//     (the "residual" split points of Section 3.1), cell by cell along the
//     tile's own anti-diagonals; then writes the dense int16 cells and the
//     packed row/column words.
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
// The tile finish reads every packed word through vector loads.
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
// a multiple of it, so no lane reads past R or writes past Rl), waited for
// here; below that through registers.  The caller's barrier follows.
template <int RSZ>
__device__ __forceinline__ void load_R(uint8_t* Rl, const uint8_t* __restrict__ Rg, int nthr)
{
    if constexpr (RSZ >= 1024) {
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
        for (int base = wave * 1024; base < RSZ; base += nthr * 16)  // wave-uniform
            __builtin_amdgcn_global_load_lds((const NF_GLOBAL void*)(Rg + base + lane * 16),
                                             (__attribute__((address_space(3))) void*)(Rl + base), 16, 0, 0);
        __builtin_amdgcn_s_waitcnt(0);
    } else if constexpr (RSZ >= 16) {
        for (int x = threadIdx.x * 16; x < RSZ; x += nthr * 16)
            *reinterpret_cast<uint4*>(Rl + x) = *reinterpret_cast<const uint4*>(Rg + x);
    } else {
        if (threadIdx.x < RSZ) Rl[threadIdx.x] = Rg[threadIdx.x];
    }
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
    const int m = q - 1;
    const int size = 1 << m;
    const int e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= size * size) return;
    const int h = e >> m;
    const int c = e & (size - 1);
    int tot = 0, best = 0;  // running total of v + v-bar, starting at k = 0 with 0
    for (int p = 1; p <= m; ++p) {
        tot += ((h >> (p - 1)) & 1) - ((c >> (p - 1)) & 1);
        best = max(best, tot);
    }
    R[e] = (uint8_t)best;
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

// Slacks of 32 split points (one per bit) in one lane.
struct Slack {
    uint32_t p[6];
    uint32_t nz;  // the OR of p: bit b is 0 where the slack is 0

    __device__ __forceinline__ void test()
    {
        nz = bits3<kA | kB | kC>(bits3<kA | kB | kC>(p[0], p[1], p[2]), bits3<kA | kB | kC>(p[3], p[4], p[5]), 0u);
    }
    // at the bits of c: + 1 where up is all ones, - 1 where it is 0
    __device__ __forceinline__ void step(uint32_t c, uint32_t up)
    {
#pragma unroll
        for (int k = 0; k < 5; ++k) {
            const uint32_t carry = bits3<kA & ~(kB ^ kC)>(c, p[k], up);
            p[k] ^= c;
            c = carry;
        }
        p[5] ^= c;
        test();
    }
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

// f(7), f(6), ..., f(0), each with its number as a constant
template <int r = 7, class F>
__device__ __forceinline__ void rows8(F&& f)
{
    f(std::integral_constant<int, r>{});
    if constexpr (r > 0) rows8<r - 1>(f);
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
template <int Q>
__device__ __forceinline__ void diag_body(const TileWork& it, DiagLds& s, int tid, int nthr, const uint8_t* staged)
{
    constexpr int T = tile_size(Q);
    const FoldDesc& f = it.f;
    const int aT = it.A * T;
    const bool admit = staged != nullptr && it.pad2 != 0;
    const uint8_t* src = admit ? staged + it.pad1 : f.codes;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;

    if (admit) {
        uint8_t* dst = const_cast<uint8_t*>(f.codes);
        const int hi = it.A == f.NT - 1 ? f.NT * T + 64 : aT + T;
        for (int e = aT + tid; e < hi; e += nthr) dst[e] = src[e];
        int4* a0 = reinterpret_cast<int4*>(it.acc + (size_t)it.A * kTileCells);
        int4* a1 = reinterpret_cast<int4*>(it.acc + (size_t)(f.NT + it.A) * kTileCells);
        for (int e = tid; e < kTileCells / 4; e += nthr) a0[e] = a1[e] = make_int4(0, 0, 0, 0);
    }
    if (wave == 0) {
        const int j = lane;
        const int ca = src[aT + j];                              // S_{a+1} for a = aT + lane
        const int cb = (aT + j - 1 >= 0) ? src[aT + j - 1] : 0;  // S_b for b = aT + j
        // split points below j; pairing rows i <= j - 2
        const unsigned long long below = j < T ? (1ull << j) - 1 : 0ull;
        unsigned long long pm = pair_rows(ca, cb) & (below >> 1);
        const unsigned long long left = j > 0 ? 1ull << (j - 1) : 0ull;  // the slack a pairing needs
        const uint32_t blo = (uint32_t)left, bhi = (uint32_t)(left >> 32);
        const uint32_t vlo = (uint32_t)below, vhi = (uint32_t)(below >> 32);
        Slack lo{}, hi{};
        lo.p[5] = ~vlo;  // never 0 at split points that are not left of j
        hi.p[5] = ~vhi;
        lo.test();
        hi.test();
        unsigned long long cm = 0;
        for (int b = 7; b >= 0; --b) {
            const uint32_t pmb = (uint32_t)(pm >> (8 * b));
            const unsigned long long pts = ~((256ull << (8 * b)) - 1);  // the split points of the blocks below
            uint32_t rlo = 0, rhi = 0;  // lane r: dL(8b + r, .)
            rows8([&](auto rc) {
                constexpr int r = rc;
                if (T < 64 && 8 * b + r >= T) return;
                const uint32_t pb = bit_mask(pmb, r);
                const unsigned long long st =
                    __ballot(((bits3<~kA & kB>(lo.nz, blo, 0u) | bits3<~kA & kB>(hi.nz, bhi, 0u)) & pb) != 0);
                const unsigned long long cl =
                    __ballot((bits3<~kA & kB>(lo.nz, (uint32_t)st, 0u) | bits3<~kA & kB>(hi.nz, (uint32_t)(st >> 32), 0u)) != 0);
                const unsigned long long dl = st | cl;
                const uint32_t up = (dl >> j) & 1 ? ~0u : 0u;
                // split points i < j' < j move; j' = i joins with slack 0
                const unsigned long long rm = pts | ((0xffull & (0xfeull << r)) << (8 * b));
                lo.step(bits3<(kA ^ kB) & kC>(up, (uint32_t)dl, vlo & (uint32_t)rm), up);
                hi.step(bits3<(kA ^ kB) & kC>(up, (uint32_t)(dl >> 32), vhi & (uint32_t)(rm >> 32)), up);
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
__global__ __launch_bounds__(kThreads) void k_diag(const TileWork* __restrict__ items, const uint8_t* staged)
{
    __shared__ DiagLds s;
    diag_body<Q>(items[blockIdx.x], s, threadIdx.x, kThreads, staged);
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

template <int Q>
__global__ __launch_bounds__(kBetweenThreads) void k_between(const BetweenWork* __restrict__ items,
                                                      const uint8_t* __restrict__ Rg)
{
    constexpr int RSZ = 1 << (2 * (Q - 1));
    __shared__ __align__(16) uint8_t Rl[RSZ < 16 ? 16 : RSZ];
    __shared__ uint16_t red[kBetweenSplit == 2 ? 64 * 64 : 1];

    const BetweenWork& it = items[blockIdx.x];
    load_R<RSZ>(Rl, Rg, kBetweenThreads);
    __syncthreads();
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    between_body<Q, kRowsPerWave, kBetweenSplit>(it, Rl, it.f.RS, it.f.CS, wave, threadIdx.x & 63, red);
}

// Finish of an off-diagonal tile (A, B), B > A, by 8 wavefronts (512 threads).
//
// Cell X(i, j) = F(AT+i, BT+j) is the maximum of P(i, j), the best split in
// the tiles strictly between A and B (the between maxima of acc and the
// groups of the two end tiles C = A+1, C = B-1), the pairing term, and the
// splits inside tiles A and B.  P is computed first (8 rows per wavefront,
// Eq. 3 lookups); the rows then go bottom-up in bits, as above: a cell rises
// over the one below when P does, when a pairing or a split inside the tile
// says so.  The row below row T-1 is row 0 of tile (A+1, B), finished one
// step ago (or of the main-diagonal tile), and the slacks E carry over from
// there, so no step rebuilds them; V starts empty at the tile's last row.
//
// The rows are taken by four wavefronts, 16 columns each.  Lane 16h + c of
// wavefront w holds column 16w + c and the split points 16h .. 16h+15 of both
// kinds: E in the low half of its slack words, V in the high half, so that one
// ripple moves both.  A wavefront works 8 rows (a block) behind its left
// neighbour, from which it needs the rows' delta bits only; a barrier
// separates the blocks.  (MI355X, against the max-plus closure by all eight
// wavefronts: n = 6000 1.90 -> 1.49 ms, 4096 folds of 50..2000 bases
// 16.9 -> 11.2 ms.)
constexpr int kTileThreads = 512;
constexpr int kChainWaves = 4;
static_assert(kTileThreads == 512, "the tile finish maps 8 wavefronts onto 8 row blocks");

template <int Q>
struct TileLds {
    // M[h][i]: bits 31..16 = dL(i, 16h .. 16h+15); bits 15..0 = delta(i, .) of
    // the columns 16h .. 16h+15 once finished (h = 3 first holds, in bit 15,
    // delta of the column left of the tile, for column 0)
    alignas(16) uint32_t M[4][64];
    alignas(16) uint16_t P[8][64][8];  // P(i, j) at [i / 8][j][i % 8]
    uint32_t cm[2][64];                // delta(32 u + b, j): bit b of cm[u][j]
    int32_t top[64];                   // X(T, j): the row below row T-1
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
// (global) into Rl.
template <int Q>
__device__ __forceinline__ void tile_body(const TileWork& it, uint8_t* Rl, const uint8_t* __restrict__ Rg,
                                          TileLds<Q>& s)
{
    constexpr int M = Q - 1;
    constexpr int G = groups_per_tile(Q);
    constexpr int T = tile_size(Q);
    constexpr int SW = state_words(Q);
    constexpr int RW = row_words(Q);
    constexpr int RSZ = 1 << (2 * M);

    const FoldDesc& f = it.f;
    const int A = it.A, d = it.d, B = A + d;
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lane = tid & 63;
    const long long ld = f.ld;
    const int aT = A * T, bT = B * T;
    const NF_GLOBAL int16_t* F = (const NF_GLOBAL int16_t*)f.F;
    const NF_GLOBAL uint8_t* codes = (const NF_GLOBAL uint8_t*)f.codes;
    const NF_GLOBAL uint32_t* rsA = (const NF_GLOBAL uint32_t*)f.RS + tile_index(f.NT, A, 0) * RW;
    const NF_GLOBAL uint32_t* csA = (const NF_GLOBAL uint32_t*)f.CS + tile_index(f.NT, A, 0) * SW;
    NF_GLOBAL uint32_t* rsB = (NF_GLOBAL uint32_t*)f.RS + tile_index(f.NT, B, 0) * RW;
    NF_GLOBAL uint32_t* csB = (NF_GLOBAL uint32_t*)f.CS + tile_index(f.NT, B, 0) * SW;

    // ---- set-up: R, the rows' bits of tile (A, A), the row below, the halo
    load_R<RSZ>(Rl, Rg, kTileThreads);
    if (tid < 256) {
        const int h = wave, i = lane;
        uint32_t m = (h < 2 ? rsA : csA)[kRowBits + i];
        m = (h & 1) ? (m & 0xffff0000u) : (m << 16);
        if (i >= T) m = 0;
        if (h == 3 && i < T) {
            // delta(i, -1); nothing lies below row T-1 left of tile (B, B)
            const int up = F[(aT + i) * ld + bT - 1];
            const int dn = (d == 1 && i == T - 1) ? 0 : (int)F[(aT + i + 1) * ld + bT - 1];
            if (up > dn) m |= 1u << 15;
        }
        s.M[h][i] = m;
    } else if (wave == 4) {
        s.top[lane] = lane < T ? (int)F[(aT + T) * ld + bT + lane] : 0;
    }

    // the row wavefronts' own state
    const int h = lane >> 4, c = lane & 15;
    const int j = 16 * (wave & 3) + c;
    Slack sl{};
    uint32_t vr = 0, own = 0, left = 0;
    unsigned long long pm = 0;
    uint32_t x = 0;
    if (wave < kChainWaves) {
        typedef const NF_GLOBAL uint16_t* half_ptr;
        // the split points of this lane left of column j
        const uint32_t below = j >= T ? 0u : (j >= 16 * h + 16 ? 0xffffu : (j > 16 * h ? (1u << (j - 16 * h)) - 1 : 0u));
#pragma unroll
        for (int k = 0; k < 6; ++k)
            sl.p[k] = ((half_ptr)(k < 3 ? rsB : csB))[(k % 3) * 256 + 4 * j + h] & below;
        vr = below;
        own = h == wave ? 0xffffu : 0u;
        left = (j > 0 && ((j - 1) >> 4) == h) ? 1u << ((j - 1) & 15) : 0u;
        pm = pair_rows(lane < T ? (int)codes[aT + lane] : 4, (int)codes[bT + j - 1]);
        if (j >= T) pm = 0;
        x = j < T ? (uint32_t)(int)F[(aT + T) * ld + bT + j] : 0u;
        if (j == 0 && h == 3) {
            // column 0: the column left of the tile is its split point -1, bit
            // 15 here, with slack X(T, 0) - X(T, -1)
            const int xl = d == 1 ? (int)x : (int)F[(aT + T) * ld + bT - 1];
            sl.p[0] = ((int)x > xl) ? 1u << 15 : 0u;
            vr = left = 1u << 15;
        }
        sl.p[5] |= 0xffffu & ~vr;      // never 0 where there is no split point
        if (j >= T) sl.p[5] = ~0u;
        sl.test();
    }

    // ---- P for the rows 8 wave .. 8 wave + 7, column `lane`
    {
        int acc[8];
        const int r0 = 8 * wave;
        NF_GLOBAL int32_t* accb = (NF_GLOBAL int32_t*)it.acc + r0 * 64;
        if (it.nslot > 0) {
#pragma unroll
            for (int r = 0; r < 8; ++r) acc[r] = (accb + r * 64)[(unsigned)lane];
        } else {
#pragma unroll
            for (int r = 0; r < 8; ++r) acc[r] = 0;
        }
        __syncthreads();  // R
        if (d >= 2) between_accumulate<Q, 8, 1>(acc, Rl, f.RS, f.CS, f.NT, A, B, A + 1, A + 2, r0, lane, 0);
        if (d >= 3) between_accumulate<Q, 8, 1>(acc, Rl, f.RS, f.CS, f.NT, A, B, B - 1, B, r0, lane, 0);
        if (it.nslot > 0) {  // hand the accumulator back zeroed for its next use
#pragma unroll
            for (int r = 0; r < 8; ++r) (accb + r * 64)[(unsigned)lane] = 0;
        }
        uint4 pk = make_uint4((uint32_t)acc[0] | ((uint32_t)acc[1] << 16), (uint32_t)acc[2] | ((uint32_t)acc[3] << 16),
                              (uint32_t)acc[4] | ((uint32_t)acc[5] << 16), (uint32_t)acc[6] | ((uint32_t)acc[7] << 16));
        if (lane >= T) pk = make_uint4(0u, 0u, 0u, 0u);
        *reinterpret_cast<uint4*>(&s.P[wave][lane][0]) = pk;
    }
    __syncthreads();

    // ---- rows bottom-up, block b = 7 - (phase - wave) of 8 rows
    uint32_t cml = 0, cmh = 0;
    for (int phase = 0; phase < 8 + kChainWaves - 1; ++phase) {
        const int b = 7 - (phase - wave);
        if (wave < kChainWaves && b >= 0 && b < 8) {
            const uint4 pk = *reinterpret_cast<const uint4*>(&s.P[b][j][0]);
            const uint4 ma = *reinterpret_cast<const uint4*>(&s.M[h][8 * b]);
            const uint4 mb = *reinterpret_cast<const uint4*>(&s.M[h][8 * b + 4]);
            const uint32_t ps[4] = {pk.x, pk.y, pk.z, pk.w};
            const uint32_t ms[8] = {ma.x, ma.y, ma.z, ma.w, mb.x, mb.y, mb.z, mb.w};
            const uint32_t pmb = (uint32_t)(pm >> (8 * b));
            const uint32_t rmask = (h == (b >> 1) && j < T) ? ~0u : 0u;  // lanes that hold the split points of this block
            uint32_t bit = 1u << (16 + (b & 1) * 8 + 7);
            uint32_t rows = 0;  // lane r: delta(8b + r, .) of this wavefront's columns
            uint32_t cm8 = 0;
            rows8([&](auto rc) {
                constexpr int r = rc;
                if (T == 64 || 8 * b + r < T) {
                    const uint32_t up_p = above<r & 1>(ps[r >> 1], x);
                    const uint32_t cand = bits3<kA | (kB & kC)>(ms[r], bit_mask(pmb, r), left);
                    const unsigned long long b1 = __ballot(bits3<(~kA & kB) | kC>(sl.nz, cand, up_p) != 0);
                    const uint32_t t1 = (uint32_t)b1 | (uint32_t)(b1 >> 32);
                    const uint32_t st = t1 | (t1 >> 16);
                    const unsigned long long b2 = __ballot(bits3<~kA & kB & kC>(sl.nz, st, own) != 0);
                    const uint32_t dl = st | (uint32_t)(b2 >> (16 * wave));
                    const uint32_t up = bit_mask(dl, c);
                    const uint32_t mv = bits3<kA | (kB & kC)>(ms[r], dl, own);
                    sl.step(bits3<(kA ^ kB) & kC>(up, mv, vr), up);
                    vr = bits3<kA | (kB & kC)>(vr, rmask, bit);
                    x -= up;
                    cm8 = __builtin_amdgcn_alignbit(cm8, up, 31);
                    rows = with_lane<r>(rows, dl);
                }
                bit >>= 1;
            });
            cmh = __builtin_amdgcn_alignbit(cmh, cml, 24);
            cml = (cml << 8) | cm8;
            // the block's bits for the wavefronts to the right and the emit
            if (lane < 8) reinterpret_cast<uint16_t*>(&s.M[wave][8 * b + lane])[0] = (uint16_t)rows;
        }
        __syncthreads();
    }
    if (wave < kChainWaves) {
        if (h == 0) {
            s.cm[0][j] = cml;
            s.cm[1][j] = cmh;
        }
        typedef NF_GLOBAL uint16_t* half_out;
#pragma unroll
        for (int k = 0; k < 6; ++k) ((half_out)(k < 3 ? rsB : csB))[(k % 3) * 256 + 4 * j + h] = (uint16_t)sl.p[k];
    }
    __syncthreads();

    // ---- emit: dense cells, row words, column words; wavefront w takes the
    // rows 8w .. 8w+7, lane = column
    const long long t_idx = tile_index(f.NT, A, d);
    NF_GLOBAL int16_t* Fw = (NF_GLOBAL int16_t*)f.F;
    NF_GLOBAL uint32_t* RSw = (NF_GLOBAL uint32_t*)(f.RS + t_idx * RW);
    NF_GLOBAL uint32_t* CSw = (NF_GLOBAL uint32_t*)(f.CS + t_idx * SW);
    const unsigned long long cm = ((unsigned long long)s.cm[1][lane] << 32) | s.cm[0][lane];
    const int top = s.top[lane];
    {
        const int r0 = 8 * wave;
        const uint32_t cm8 = (uint32_t)(cm >> r0);
        int v = top + __popcll((cm >> r0) >> 8);  // X(r0 + 8, lane)
        unsigned long long H = __ballot(v > __shfl_up(v, 1));  // horizontal differences (column 0's is not used)
#pragma unroll
        for (int r = 7; r >= 0; --r) {
            const int i = r0 + r;
            const uint32_t bit = (cm8 >> r) & 1u;
            const unsigned long long dl = __ballot(bit);
            v += (int)bit;
            H ^= dl ^ (dl << 1);
            if (T == 64 || i < T) {
                if (T == 64 || lane < T) (Fw + (long long)(aT + i) * ld + bT)[(unsigned)lane] = (int16_t)v;
                if ((T == 64 || lane < T) && (lane % Q) == 0) {
                    uint32_t hb = 0;
                    if constexpr (M > 0) hb = (uint32_t)((H >> lane) >> 1) & ((1u << M) - 1u);
                    RSw[(lane / Q) * 64 + i] = ((hb << M) << 16) | (uint32_t)v;
                }
            } else if (lane < G) {
                // padding row (T < 64): readers load whole 64-row lines, so
                // give it words that keep their sums bounded and R in range
                RSw[lane * 64 + i] = 0;
            }
        }
    }
    for (int k = wave; k < G; k += kTileThreads / 64) {
        const unsigned long long u = cm >> (k * Q);  // the group's rows are its low bits
        uint32_t cw = 0;  // padding column, as for padding rows
        if (T == 64 || lane < T)
            cw = (((uint32_t)u & ((1u << M) - 1u)) << 16) | (uint32_t)(top + __popcll(u));
        CSw[k * 64 + lane] = cw;
    }
}

template <int Q, bool kWide>
constexpr int kStageWavesPerSimd = (Q == 8 && kWide) ? 6 : 1;

// Tile finishes alone (staged steps).  kWide: the lean finish at six
// wavefronts per SIMD, three workgroups per CU (q = 8), as in the fused step.
template <int Q, bool kWide>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(kStageWavesPerSimd<Q, kWide>)))
void k_tile(const TileWork* __restrict__ items, const uint8_t* __restrict__ Rg)
{
    constexpr int RSZ = 1 << (2 * (Q - 1));
    __shared__ __align__(16) uint8_t Rl[RSZ < 16 ? 16 : RSZ];
    __shared__ __align__(16) TileLds<Q> s;
    tile_body<Q>(items[blockIdx.x], Rl, Rg, s);
}

// One wavefront step in one launch: workgroups [0, ntile) finish the tiles
// of diagonal s, the rest run the between chunks of diagonal s+1 (which only
// read diagonals <= s-1 and write the other half of the accumulators).
//
// Two shapes of the same code.  The default leaves the register count to the
// compiler (two workgroups per CU at q = 8: the finish's registers and LDS
// bound it), which keeps the finish, the fold's critical path, fastest.  The
// wide shape (q = 8 only) holds each workgroup to 80 VGPRs (the compiler
// spills a few registers to scratch) so that a CU takes three, six
// wavefronts per SIMD: the between chunks, which bound long folds, then run
// faster while each finish runs slower.  (Measured on MI355X: n = 16000
// 13.2 -> 12.2 ms, n = 6000 2.21 -> 2.34 ms.)
template <int Q, bool kWide>
__global__ __launch_bounds__(kTileThreads) __attribute__((amdgpu_waves_per_eu(kStageWavesPerSimd<Q, kWide>)))
void k_stage(const TileWork* __restrict__ titems, int ntile,
                                                        const BetweenWork* __restrict__ bitems,
                                                        const uint8_t* __restrict__ Rg)
{
    constexpr int RSZ = 1 << (2 * (Q - 1));
    __shared__ __align__(16) uint8_t Rl[RSZ < 16 ? 16 : RSZ];
    __shared__ __align__(16) TileLds<Q> s;
    const int b = blockIdx.x;
    if (b < ntile) {
        tile_body<Q>(titems[b], Rl, Rg, s);
    } else {
        load_R<RSZ>(Rl, Rg, kTileThreads);
        __syncthreads();
        const BetweenWork& it = bitems[b - ntile];
        const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
        between_body<Q, 16, kTileThreads / 64 / 4>(it, Rl, it.f.RS, it.f.CS, wave, threadIdx.x & 63,
                                                   &s.P[0][0][0]);
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

// S[i*n + j] = D(i+1, j+1) = F(i, j+1) for i <= j, 0 below the diagonal.
__global__ void k_expand(const int16_t* __restrict__ F, int ld, int n, int16_t* __restrict__ S)
{
    const int i = blockIdx.y;
    const int j0 = (blockIdx.x * blockDim.x + threadIdx.x) * 4;
    const int16_t* src = F + (long long)i * ld + 1;
    int16_t* dst = S + (long long)i * n;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
        const int j = j0 + u;
        if (j < n) dst[j] = j >= i ? src[j] : (int16_t)0;
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
    if (which == 0) return launch_k(k_diag<Q>, grid, dim3(kThreads), s, e0, e1, (const TileWork*)items, R);
    if (which == 1) return launch_k(k_tile<Q, false>, grid, dim3(kTileThreads), s, e0, e1, (const TileWork*)items, R);
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

hipError_t launch_diag_admit(int q, const TileWork* items, int nitems, const uint8_t* staged, hipStream_t s)
{
    return dispatch(q, 0, items, nitems, staged, s, nullptr, nullptr);
}

hipError_t launch_tile(int q, const TileWork* items, int nitems, const uint8_t* R, hipStream_t s, hipEvent_t e0,
                       hipEvent_t e1, bool wide)
{
    if (wide && q == 8 && nitems > 0)
        return launch_k(k_tile<8, true>, dim3(nitems), dim3(kTileThreads), s, e0, e1, items, R);
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
    return launch_k(k_stage<Q, false>, dim3(nt + nb), dim3(kTileThreads), s, e0, e1, t, nt, b, R);
}
}  // namespace

hipError_t launch_stage(int q, bool wide, const TileWork* titems, int ntile, const BetweenWork* bitems, int nbtw,
                        const uint8_t* R, hipStream_t s, hipEvent_t e0, hipEvent_t e1)
{
    if (ntile + nbtw <= 0) return hipSuccess;
    if (wide && q == 8)
        return launch_k(k_stage<8, true>, dim3(ntile + nbtw), dim3(kTileThreads), s, e0, e1, titems, ntile, bitems, R);
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

hipError_t launch_expand(const int16_t* F, int ld, int n, int16_t* S, hipStream_t s)
{
    if (n <= 0) return hipSuccess;
    dim3 grid((n + 1023) / 1024, n);
    hipLaunchKernelGGL(k_expand, grid, dim3(256), 0, s, F, ld, n, S);
    return hipGetLastError();
}

}  // namespace nf
