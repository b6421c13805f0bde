// MFMA kernel template (bf16 / fp16 inputs, fp32 accumulation, 16x16x32 atoms) for MatMul / BatchMatMul operators whose
// extents are no multiples of 16, so that no member of their spaces has wave tiles of whole atoms and rows at 16-byte
// offsets: every such member used to run on the scalar template, which reads two LDS words per multiply-add.
//
// A workgroup owns the member's BM x BN tile, whatever its extents.  The tile is rounded up to whole atoms and dealt to
// WM x WN waves of MI x NI atoms (the host picks the division; a member's own wave tiles, factors of 125 or 27, would each
// be rounded up by themselves).  What the atoms compute past the tile is not stored.  The reduction is walked in NSL slabs
// of KS (the member's slab rounded up to whole MFMA steps), the last one filled up with zeros in both operands.
//
// Measured (bf16): 1000^3 in tiles of 20 x 100 168 us on the scalar template (20 waves, the best there), 15.6 us with every piece's place worked out
// for every slab, 12.5 us here (160 TFLOP/s); 120 x 280 x 3650 in 60 x 56 39.7 -> 19.5; 220 x 280 x 950 in 44 x 56 12.3 -> 6.4.  119 drawn and random
// members against the template before that and before the order of the workgroups followed the XCDs: 1.29x in the geometric mean.
// What bounds it: at these tiles the way of the loads.  1000^3, counters over the cycles in which a compute unit is busy (22 900, 9.9 us; the rest is the
// launch): the load unit 72 %, the unit that returns its data 84 %, 38 cycles a wave load of 1 KiB (rows of 200 bytes in pieces of 16 that begin at multiples of 8), LDS
// 54 % (a third of it bank conflicts), matrix pipes 18 %.  Deeper prefetch gains nothing there.
// Every operand travels in 16-byte pieces of 8 consecutive elements,
// loaded at the 2-byte alignment an odd row length leaves.  A piece that would reach past its row is loaded from as far left as
// it must be to end with the row, and shifted down when it is stored: no load leaves its operand's rows.
//   * A [M][K]: pieces along k.  LDS As[row][KS + 8]: a fragment is one 16-byte read; the odd number of pieces per row spreads 16 rows
//     over all banks.
//   * B [K][N] (and a first operand stored [K][M]): pieces along n.  LDS Bs[k][LDX] as memory has it, fragments read with the
//     transposing LDS load (two per fragment).  LDX is an odd multiple of 32 bytes and every 8 rows lie 128 bytes
//     further, so the 4 rows x 32 bytes that two groups of 16 lanes read together (8 rows apart) fall into 8 different groups of banks.
// NSTG = 2: the pieces of the next DEPTH slabs are in registers while slab s is multiplied; the next one's are stored to the other stage afterwards
// (one barrier per slab).  NSTG = 1: load, barrier, store, barrier, multiply.
//
// KWAVES: another way, for long reductions on grids that leave a compute unit to one workgroup.  Every wave has the whole tile as its wave tile and a
// contiguous part of the reduction, in steps of 32 positions through a part of the LDS of its own, so that nothing waits at a barrier until the sums
// meet at the end and each operand is read from the LDS once.  The last step begins early enough to be full and leaves out what has been
// added; a tile at the end of a row begins far enough left for whole pieces, its surplus columns are not stored: no load reaches past an operand and the loop
// has one form.  What bounds it: the load unit (16 bytes a lane: 19 cycles a wave from L1 at 4-byte alignment, 68 at 2-byte), then the LDS stores.
// The sums are written to LDS as rows, so that consecutive threads store consecutive columns.

#if IN_DTYPE == 1
typedef __attribute__((ext_vector_type(8))) __bf16 frag_t;
#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0)
#else
typedef __attribute__((ext_vector_type(8))) _Float16 frag_t;
#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0)
#endif
#if !defined(KWAVES) && !KEEP   // nothing of a plan for two slabs under way, or for a second workgroup's registers, holds
#undef DEPTH
#define DEPTH 1
#undef MINW
#define MINW ((NT / 64 + 3) / 4)
#endif
// Two stages without kept places (and not FRESH), mostly pieces of k rows: each is placed where it is loaded and where it is stored.  With the choice between
// two places per piece and the shift decided before, which serve kept ones, the compiler made several branches of every such piece (420 x 2295 x 2400 in 70 x 459,
// eight waves of 5 x 6 atoms, 134 us against 127; 312 x 950 x 1875 in 26 x 950, 1 x 15 atoms, 94 against 85; with 7 x 2 and 13 x 2 atoms 65 against 79, 46 against 50).
#if !KEEP && NSTG == 2 && !defined(FRESH) && NI > MI && !A_TRANS
#define RECALC 1
#else
#define RECALC 0
#endif
typedef u32x4 __attribute__((aligned(2))) u32x4_a2;
typedef __attribute__((ext_vector_type(4))) short v4s;

constexpr int odd16(int n) { return ((n + 15) / 16 | 1) * 16; }
__device__ __forceinline__ constexpr int kr_off(int ld, int k) { return k * ld + (k >> 3) * 64; }   // LDS element of k row k
constexpr int CM = (BM + 7) / 8, CN = (BN + 7) / 8;   // pieces of a k row
#ifndef KWAVES
constexpr int KPART = K / KSPLIT;                 // reduction length of this workgroup
static_assert(NSL * KS >= KPART && (NSL - 1) * KS < KPART && KS % 32 == 0 && KPART >= 8, "decoder and template disagree");
static_assert(WM * MI * 16 >= BM && WN * NI * 16 >= BN && NT == 64 * WM * WN, "decoder and template disagree");
constexpr bool K_TAIL = KPART % KS != 0;          // the last slab is not full
constexpr int LDK = KS + 8;                       // elements per LDS row of a k-contiguous operand
constexpr int LDM = odd16(WM * MI * 16), LDN = odd16(WN * NI * 16);
constexpr int A_STAGE = A_TRANS ? KS * LDM + (KS / 8) * 64 : WM * MI * 16 * LDK;
constexpr int B_STAGE = KS * LDN + (KS / 8) * 64;
static_assert(NSTG * (A_STAGE + B_STAGE) * 2 <= LDS_BYTES, "stages exceed the LDS the host asks for");
constexpr int CK = KS / 8;                        // pieces of a k-contiguous row
constexpr int A_PIECES = A_TRANS ? KS * CM : BM * CK, B_PIECES = KS * CN;
constexpr int NA = (A_PIECES + NT - 1) / NT, NB = (B_PIECES + NT - 1) / NT;

struct Slab { u32x4 a[NA], b[NB]; };
#endif

// v shifted down by sh elements (0 .. 7), zeros from above; sh >= 8: zeros
__device__ __forceinline__ u32x4 shift_down(u32x4 v, int sh)
{
    u32 w0 = v.x, w1 = v.y, w2 = v.z, w3 = v.w;
    if (sh & 1) { w0 = (w0 >> 16) | (w1 << 16); w1 = (w1 >> 16) | (w2 << 16); w2 = (w2 >> 16) | (w3 << 16); w3 >>= 16; }
    if (sh & 2) { w0 = w1; w1 = w2; w2 = w3; w3 = 0; }
    if (sh & 4) { w0 = w2; w1 = w3; w2 = 0; w3 = 0; }
    if (sh >= 8) w0 = w1 = w2 = w3 = 0;
    const u32x4 r = {w0, w1, w2, w3};
    return r;
}

// Fragment of k rows, an atom whose first row / column is x0, from the LDS rows of one MFMA step: in each group of 16 lanes, lane s addresses 4
// consecutive elements of k row s / 4, and lane i receives the 4 values of element i
template <int LD>
__device__ __forceinline__ frag_t kr_frag(const u16 *S, int x0, int lane)
{
    const int s = lane & 15;
    const u16 *p = S + kr_off(LD, 8 * (lane >> 4)) + (s >> 2) * LD + x0 + 4 * (s & 3);
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)p);
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)(p + 4 * LD));
    return __builtin_bit_cast(frag_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// ---------------------------------------------------------------- waves that share the reduction (KWAVES)
#ifdef KWAVES
constexpr int KC = 32;                               // reduction positions of a step
constexpr int MA = (BM + 15) / 16, NATOM = (BN + 15) / 16;
constexpr int NSTEP = (K + KC - 1) / KC, DUP = NSTEP * KC - K;   // the last step begins DUP positions early and leaves them out
constexpr int LA = A_TRANS ? odd16(MA * 16) : KC + 8, LB = odd16(NATOM * 16);
constexpr int KR_GAPS = (KC / 8 - 1) * 64;
constexpr int A_PART = A_TRANS ? KC * LA + KR_GAPS : MA * 16 * LA, B_PART = KC * LB + KR_GAPS, PART = A_PART + B_PART;
constexpr int PA = A_TRANS ? KC * CM : BM * (KC / 8), PB = KC * CN;
constexpr int QA = (PA + 63) / 64, QB = (PB + 63) / 64;
// partial sums: P[wave][row][LC]; four rows further on is a quarter of the banks further on
constexpr int LC = NATOM * 16 + 4;
constexpr int RED_ROWS = MA * 16;
static_assert(K >= KC && NT == 64 * KWAVES && KWAVES <= NSTEP && KSPLIT == 1, "decoder and template disagree");
static_assert(KWAVES * (PART * 2 > RED_ROWS * LC * 4 ? PART * 2 : RED_ROWS * LC * 4) == LDS_BYTES, "decoder and template disagree");

#define GLOBAL __attribute__((address_space(1)))
typedef GLOBAL u32x4_a2 g_u32x4;
typedef GLOBAL u16 g_u16;
// base (in scalar registers, and left there) + a lane's byte offset
template <typename T>
__device__ __forceinline__ auto load_at(const u16 *base, u32 off)
{
    const GLOBAL char *p = (const GLOBAL char *)base;
    asm("" : "+s"(p));
    return *(const T *)(p + off);
}
// Operands of k rows with pieces that begin at odd elements.  A 16-byte load that is not 4-byte aligned takes the load unit 68 cycles a wave instead of 19
// (8-byte aligned: 19 - 22, measured from L1 and L2), so such a piece is loaded from one element to the left, its last element by a load of its own (9
// cycles), and shifted by half a word when it is stored: 100 x 5439 x 1056 in 50 x 21 15.5 -> 11.1 us.  Not the k-contiguous rows of four pieces, where the
// single elements cost as much as they spare (162 x 2100 x 2079 in 54 x 60 10.2 us without and 12.8 with, 200 x 6880 x 2275 in 50 x 32 32.5 and 39.7).
constexpr bool ODD_A = A_TRANS && (M % 2 != 0 || (BM % 2 != 0 && M > BM)), ODD_B = N % 2 != 0 || (BN % 2 != 0 && N > BN);
template <int Q, bool ODD> struct Pieces16 { u32x4 v[Q]; u32 e[ODD ? Q : 1]; };
struct Step { Pieces16<QA, ODD_A> a; Pieces16<QB, ODD_B> b; };
// a lane's pieces: element offset from the step's first position (ODD: plus the parity of that position), LDS element
struct Places { u32 ga[QA], gb[QB], sa[QA], sb[QB]; };

__device__ __forceinline__ void place_kr(u32 &g, u32 &s, int q, int pieces, int c, int len, int ld)
{
    if (q >= pieces) q = 0;
    g = (u32)(q / c * len + q % c * 8);
    s = (u32)(kr_off(ld, q / c) + q % c * 8);
}
// Operand's pieces from element `from` of it on.  back: in the step that ends with the operand, the last piece of an operand as wide as the tile, no multiple of
// 8, would reach that far past its end: it is loaded from further left and shifted.
template <int Q, bool ODD>
__device__ __forceinline__ void load_pieces(Pieces16<Q, ODD> &r, const u32 (&g)[Q], const u16 *operand, long from, int last_lane, int back)
{
    const u32 odd = ODD ? (u32)from & 1u : 0u;
    const u16 *base = operand + (from - odd);
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        u32 at = g[i] + odd;
        if (back > 0 && i == Q - 1 && last_lane >= 0) at -= (int)(threadIdx.x & 63) == last_lane ? back : 0;
        r.v[i] = load_at<g_u32x4>(base, 2u * (ODD ? at & ~1u : at));
        if (ODD) r.e[i] = load_at<g_u16>(base, 2u * at + 14u);
    }
}
template <int Q, bool ODD>
__device__ __forceinline__ void store_pieces(const Pieces16<Q, ODD> &r, const u32 (&g)[Q], const u32 (&s)[Q], u16 *S, int pieces, long from, int lane, int last_lane, int back)
{
#pragma unroll
    for (int i = 0; i < Q; ++i) {
        u32x4 v = r.v[i];
        int shift_by = 0;
        if (back > 0 && i == Q - 1 && last_lane >= 0) shift_by = lane == last_lane ? back : 0;
        if (ODD) {
            const u32 sh = ((g[i] + (u32)from - shift_by) & 1u) << 4;
            v.x = __builtin_amdgcn_alignbit(v.y, v.x, sh); v.y = __builtin_amdgcn_alignbit(v.z, v.y, sh);
            v.z = __builtin_amdgcn_alignbit(v.w, v.z, sh); v.w = __builtin_amdgcn_alignbit(r.e[i], v.w, sh);
        }
        if (back > 0 && i == Q - 1 && last_lane >= 0) v = shift_down(v, shift_by);
        if ((i + 1) * 64 <= pieces || lane + i * 64 < pieces) *(u32x4 *)(S + s[i]) = v;
    }
}
// the first reduction position of step s, and how far the last piece of its operands reaches past their ends
constexpr int BACK_A = A_TRANS && M < 8 * CM ? 8 * CM - M : 0, BACK_B = N < 8 * CN ? 8 * CN - N : 0;
struct From { long a, b; int end_a, end_b; };
__device__ __forceinline__ From from_of(long a0, long b0, int s)
{
    const bool last = s == NSTEP - 1;
    const long k0 = last ? K - KC : s * KC;
    const From f = {a0 + (A_TRANS ? k0 * M : k0), b0 + k0 * N, last ? (PA - 1) % 64 : -1, last ? (PB - 1) % 64 : -1};
    return f;
}
__device__ __forceinline__ void load_step(Step &r, const Places &p, const u16 *A, const u16 *B, const From &f)
{
    load_pieces<QA, ODD_A>(r.a, p.ga, A, f.a, f.end_a, BACK_A);
    load_pieces<QB, ODD_B>(r.b, p.gb, B, f.b, f.end_b, BACK_B);
}
__device__ __forceinline__ void store_step(const Step &r, const Places &p, u16 *As, u16 *Bs, const From &f, int lane)
{
    store_pieces<QA, ODD_A>(r.a, p.ga, p.sa, As, PA, f.a, lane, f.end_a, BACK_A);
    store_pieces<QB, ODD_B>(r.b, p.gb, p.sb, Bs, PB, f.b, lane, f.end_b, BACK_B);
}
// The lanes of a wave exchange operands through LDS that is the wave's own.  Its accesses to the LDS take effect in the order of the code; this keeps the
// compiler from moving one lane's reads before another's writes, or its next writes before those reads.  No instruction comes of it.
__device__ __forceinline__ void exchange()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
template <bool MASK>
__device__ __forceinline__ void multiply_step(f32x4 (&acc)[MA][NATOM], const u16 *As, const u16 *Bs, int lane)
{
    u32x4 keep;                                      // (the last step) which of the lane's 8 positions have not been added yet
#pragma unroll
    for (int d = 0; d < 4; ++d) keep[d] = (lane / 16 * 8 + 2 * d >= DUP ? 0xffffu : 0u) | (lane / 16 * 8 + 2 * d + 1 >= DUP ? 0xffff0000u : 0u);
    auto masked = [&](frag_t f) { return MASK ? __builtin_bit_cast(frag_t, __builtin_bit_cast(u32x4, f) & keep) : f; };
    frag_t af[MA];
#pragma unroll
    for (int i = 0; i < MA; ++i)
#if A_TRANS
        af[i] = masked(kr_frag<LA>(As, i * 16, lane));
#else
        af[i] = masked(__builtin_bit_cast(frag_t, *(const u32x4 *)(As + (i * 16 + lane % 16) * LA + lane / 16 * 8)));
#endif
#pragma unroll
    for (int j = 0; j < NATOM; ++j) {
        const frag_t bf = masked(kr_frag<LB>(Bs, j * 16, lane));
#pragma unroll
        for (int i = 0; i < MA; ++i) acc[i][j] = MFMA(af[i], bf, acc[i][j]);
    }
}

extern "C" __global__ __launch_bounds__(NT, MINW)
void KERNEL_NAME(const u16 *__restrict__ A, const u16 *__restrict__ B, float *__restrict__ C,
                 unsigned long long *ctl /* unused: members of this template are never folded */)
{
    extern __shared__ __attribute__((aligned(16))) u16 smem[];
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    u16 *const As = smem + wave * PART, *const Bs = As + A_PART;
    const BlockId bid = block_id();
    // a tile whose pieces would reach past the row's end begins further left; its first columns are computed and not stored
    const int m0 = bid.m * BM, n0 = bid.n * BN;
    const int ms = A_TRANS && M >= 8 * CM ? min(m0, M - 8 * CM) : m0, ns = N >= 8 * CN ? min(n0, N - 8 * CN) : n0;
    const int s0 = NSTEP * wave / KWAVES, s1 = NSTEP * (wave + 1) / KWAVES;
    Places p;
#pragma unroll
    for (int i = 0; i < QA; ++i) {
#if A_TRANS
        place_kr(p.ga[i], p.sa[i], lane + i * 64, PA, CM, M, LA);
#else
        const int q = lane + i * 64 < PA ? lane + i * 64 : 0;
        p.ga[i] = (u32)(q / (KC / 8) * K + q % (KC / 8) * 8);
        p.sa[i] = (u32)(q / (KC / 8) * LA + q % (KC / 8) * 8);
#endif
    }
#pragma unroll
    for (int i = 0; i < QB; ++i) place_kr(p.gb[i], p.sb[i], lane + i * 64, PB, CN, N, LB);

    for (int bi = 0; bi < BATCH_INNER; ++bi) {
        const long batch = (long)bid.b * BATCH_INNER + bi;
        const long a0 = batch * M * K + (A_TRANS ? (long)ms : (long)m0 * K), b0 = batch * K * N + ns;
        float *Cb = C + batch * M * N + (long)m0 * N + n0;
        f32x4 acc[MA][NATOM];
#pragma unroll
        for (int i = 0; i < MA; ++i)
#pragma unroll
            for (int j = 0; j < NATOM; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;
        Step step;
        load_step(step, p, A, B, from_of(a0, b0, s0));
        // (a loop-carried value that is a load on every way in becomes a load at its use)
#pragma unroll
        for (int i = 0; i < QA; ++i) { asm volatile("" : "+v"(step.a.v[i])); if (ODD_A) asm volatile("" : "+v"(step.a.e[ODD_A ? i : 0])); }
#pragma unroll
        for (int i = 0; i < QB; ++i) { asm volatile("" : "+v"(step.b.v[i])); if (ODD_B) asm volatile("" : "+v"(step.b.e[ODD_B ? i : 0])); }
        if (bi > 0) __syncthreads();                  // the previous batch's sums have been read
#pragma unroll 1
        for (int s = s0; s < s1 - 1; ++s) {
            store_step(step, p, As, Bs, from_of(a0, b0, s), lane);
            exchange();
            load_step(step, p, A, B, from_of(a0, b0, s + 1));
            __builtin_amdgcn_sched_barrier(0);
            multiply_step<false>(acc, As, Bs, lane);
            exchange();
        }
        store_step(step, p, As, Bs, from_of(a0, b0, s1 - 1), lane);
        exchange();
        if (DUP > 0 && wave == KWAVES - 1) multiply_step<true>(acc, As, Bs, lane);
        else multiply_step<false>(acc, As, Bs, lane);

        // The waves' sums meet in LDS, every wave's as rows of the tile; then the threads walk the tile's rows.
        __syncthreads();
        float *const red = (float *)smem;
        {
            float *const mine = red + wave * (RED_ROWS * LC) + lane / 16 * 4 * LC + lane % 16;
#pragma unroll
            for (int i = 0; i < MA; ++i)
#pragma unroll
                for (int j = 0; j < NATOM; ++j)
#pragma unroll
                    for (int r = 0; r < 4; ++r) mine[(i * 16 + r) * LC + j * 16] = acc[i][j][r];
        }
        __syncthreads();
        const float *const from = red + (m0 - ms) * LC + (n0 - ns);
#pragma unroll 2
        for (int e = tid; e < BM * BN; e += NT) {
            const int row = e / BN, col = e % BN;
            float sum = from[row * LC + col];
#pragma unroll
            for (int w = 1; w < KWAVES; ++w) sum += from[w * (RED_ROWS * LC) + row * LC + col];
            Cb[(long)row * N + col] = sum;
        }
    }
}
#else
// Where a thread's pieces come from and go to, worked out once: recomputed for every slab, the places cost more vector instructions
// than the slab has of all other kinds (1000^3 in tiles of 20 x 100: 210 of 230 in its loop).
//   g: byte offset from the operand at the slab's first reduction position.
//   t: the same for the last slab where it is not full (from 8 positions further left for a k-contiguous operand, if there is a slab before it): no load
//      reaches past the operand's rows.
//   s: LDS element.
constexpr int LAST0 = (NSL - 1) * KS, TAIL0 = NSL > 1 ? LAST0 - 8 : 0;
template <int N_>
struct Pieces { u32 g[N_], t[K_TAIL ? N_ : 1], s[N_]; };

__device__ __forceinline__ void plan_kc(Pieces<NA> &p, int tid)
{
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int q = tid + i * NT < A_PIECES ? tid + i * NT : 0, row = q / CK, c = q % CK * 8;
        p.g[i] = 2u * (u32)(row * K + c);
        if (K_TAIL) p.t[i] = 2u * (u32)(row * K + min(LAST0 + c, KPART - 8) - TAIL0);
        p.s[i] = (u32)(row * LDK + c);
    }
}
template <int N_, int PIECES, int LEN, int C, int LD>
__device__ __forceinline__ void plan_kr(Pieces<N_> &p, int x0, int tid)
{
#pragma unroll
    for (int i = 0; i < N_; ++i) {
        const int q = tid + i * NT < PIECES ? tid + i * NT : 0, kr = q / C, x = q % C * 8, at = min(x0 + x, LEN - 8);
        p.g[i] = 2u * (u32)(kr * LEN + at);
        if (K_TAIL) p.t[i] = 2u * (u32)((min(LAST0 + kr, KPART - 1) - LAST0) * LEN + at);
        p.s[i] = (u32)(kr_off(LD, kr) + x);
    }
}

struct Plan {
    Pieces<NA> a;
    Pieces<NB> b;
};
// KEEP = 0: few registers for the places; where they are worked out, and what of them is kept, is left to the compiler, or (FRESH, a kernel that
// spills otherwise) they are worked out for every slab: the thread number is opaque then
__device__ __forceinline__ void plan_slab(Plan &p, int m0, int n0, int tid)
{
#ifdef FRESH
    asm volatile("" : "+v"(tid));
    tid &= 1023;
#endif
#if A_TRANS
    plan_kr<NA, A_PIECES, M, CM, LDM>(p.a, m0, tid);
#else
    plan_kc(p.a, tid);
#endif
    plan_kr<NB, B_PIECES, N, CN, LDN>(p.b, n0, tid);
}

// Pieces of k rows are shifted where they were loaded from further left to end with their row, in tiles that reach the row's end (and, with tiles of 2 and
// 3, also in the ones before it: 8 past the start of a tile is then more than two tiles on; whole multiples of 8 never are).
constexpr bool edge_tile(int tile, int x0, int len) { return tile % 8 != 0 && ((tile + 7) / 8 * 8 > 2 * tile || x0 + tile == len); }

#if RECALC
// k-contiguous operand: piece q of a slab that starts at reduction position k0
__device__ __forceinline__ u32x4 load_kc(const u16 *__restrict__ base, int q, int k0)
{
    const int row = q / CK, k = k0 + q % CK * 8;
    return *(const u32x4_a2 *)(base + (u32)(row * K + (K_TAIL ? min(k, KPART - 8) : k)));
}
__device__ __forceinline__ void store_kc(u16 *S, u32x4 v, int q, int k0, bool last)
{
    const int c = q % CK;
    if (K_TAIL && last) v = shift_down(v, max(k0 + c * 8 - (KPART - 8), 0));
    *(u32x4 *)(S + q / CK * LDK + c * 8) = v;
}
// operand of k rows: LEN elements of a row in memory, of which the tile's begin at x0; C pieces per row
template <int LEN, int C>
__device__ __forceinline__ u32x4 load_kr(const u16 *__restrict__ base, int q, int k0, int x0)
{
    const int k = k0 + q / C;
    return *(const u32x4_a2 *)(base + (u32)((K_TAIL ? min(k, KPART - 1) : k) * LEN + min(x0 + q % C * 8, LEN - 8)));
}
template <int LEN, int C, int LD, int TILE>
__device__ __forceinline__ void store_kr(u16 *S, u32x4 v, int q, int k0, int x0, bool last)
{
    const int kr = q / C, x = q % C * 8;
    if (edge_tile(TILE, x0, LEN)) v = shift_down(v, max(x0 + x - (LEN - 8), 0));
    if (K_TAIL && last && k0 + kr >= KPART) { const u32x4 z = {0u, 0u, 0u, 0u}; v = z; }
    *(u32x4 *)(S + kr_off(LD, kr) + x) = v;
}
__device__ __forceinline__ void load_slab(Slab &s, const Plan &, const u16 *__restrict__ Ab, const u16 *__restrict__ Bb, int j, bool, int m0, int n0, int tid)
{
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int q = tid + i * NT;
        if (A_PIECES % NT == 0 || q < A_PIECES) s.a[i] = load_kc(Ab, q, j * KS);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int q = tid + i * NT;
        if (B_PIECES % NT == 0 || q < B_PIECES) s.b[i] = load_kr<N, CN>(Bb, q, j * KS, n0);
    }
}
__device__ __forceinline__ void store_slab(const Slab &s, int j, u16 *As, u16 *Bs, int m0, int n0, int tid)
{
    const bool last = j == NSL - 1;
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int q = tid + i * NT;
        if (A_PIECES % NT == 0 || q < A_PIECES) store_kc(As, s.a[i], q, j * KS, last);
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int q = tid + i * NT;
        if (B_PIECES % NT == 0 || q < B_PIECES) store_kr<N, CN, LDN, BN>(Bs, s.b[i], q, j * KS, n0, last);
    }
}
#else
// slab j of the operands; last: it is the last one.  (A thread without an i-th piece loads its operand's first.)
__device__ __forceinline__ void load_slab(Slab &s, const Plan &kept, const u16 *__restrict__ Ab, const u16 *__restrict__ Bb, int j, bool last, int m0, int n0, int tid)
{
    Plan fresh;
    if (!KEEP) plan_slab(fresh, m0, n0, tid);
    const Plan &p = KEEP ? kept : fresh;
    const bool tail = last && K_TAIL;
#if A_TRANS
    const char *a = (const char *)(Ab + (long)(tail ? LAST0 : j * KS) * M);
#else
    const char *a = (const char *)(Ab + (tail ? TAIL0 : j * KS));
#endif
    const char *b = (const char *)(Bb + (long)(tail ? LAST0 : j * KS) * N);
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const u32 g = p.a.g[i], t = K_TAIL ? p.a.t[K_TAIL ? i : 0] : g;
        s.a[i] = *(const u32x4_a2 *)(a + (tail ? t : g));
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const u32 g = p.b.g[i], t = K_TAIL ? p.b.t[K_TAIL ? i : 0] : g;
        s.b[i] = *(const u32x4_a2 *)(b + (tail ? t : g));
    }
}

template <int N_, int PIECES, int LEN, int C>
__device__ __forceinline__ void store_kr(u16 *S, const u32x4 (&r)[N_], const Pieces<N_> &p, bool last, bool edge, int x0, int tid)
{
#pragma unroll
    for (int i = 0; i < N_; ++i) {
        const int q = tid + i * NT;
        u32x4 v = r[i];
        if (edge) v = shift_down(v, max(x0 + q % C * 8 - (LEN - 8), 0));
        if (last && K_TAIL && LAST0 + q / C >= KPART) { const u32x4 z = {0u, 0u, 0u, 0u}; v = z; }
        if ((i + 1) * NT <= PIECES || q < PIECES) *(u32x4 *)(S + p.s[i]) = v;
    }
}
__device__ __forceinline__ void store_slab(const Slab &s, const Plan &kept, u16 *As, u16 *Bs, bool last, bool edge_a, bool edge_b, int m0, int n0, int tid)
{
    Plan fresh;
    if (!KEEP) plan_slab(fresh, m0, n0, tid);
    const Plan &p = KEEP ? kept : fresh;
#if A_TRANS
    store_kr<NA, A_PIECES, M, CM>(As, s.a, p.a, last, edge_a, m0, tid);
#else
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int q = tid + i * NT;
        u32x4 v = s.a[i];
        if (last && K_TAIL) v = shift_down(v, max(LAST0 + q % CK * 8 - (KPART - 8), 0));
        if ((i + 1) * NT <= A_PIECES || q < A_PIECES) *(u32x4 *)(As + p.a.s[i]) = v;
    }
#endif
    store_kr<NB, B_PIECES, N, CN>(Bs, s.b, p.b, last, edge_b, n0, tid);
}
#endif

// Fragment of an atom whose first row / column is x0, K step kk.  Lane l supplies row or column l % 16, the 8 reduction
// values from 8 * (l / 16).
__device__ __forceinline__ frag_t frag_kc(const u16 *S, int x0, int kk, int lane)
{
    return __builtin_bit_cast(frag_t, *(const u32x4 *)(S + (x0 + lane % 16) * LDK + kk * 32 + lane / 16 * 8));
}
// (transposing read: in each group of 16 lanes, lane s addresses 4 consecutive elements of k row s / 4, and lane i receives the 4
// values of element i)
template <int LD>
__device__ __forceinline__ frag_t frag_kr(const u16 *S, int x0, int kk, int lane)
{
    const int s = lane & 15;
    const u16 *p = S + kr_off(LD, kk * 32 + 8 * (lane >> 4)) + (s >> 2) * LD + x0 + 4 * (s & 3);
    const v4s lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)p);
    const v4s hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) v4s *)(p + 4 * LD));
    return __builtin_bit_cast(frag_t, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

__device__ __forceinline__ void compute_slab(f32x4 (&acc)[MI][NI], const u16 *As, const u16 *Bs, int wm, int wn, int lane)
{
#pragma unroll
    for (int kk = 0; kk < KS / 32; ++kk) {
        frag_t af[MI], bf[NI];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#if A_TRANS
            af[i] = frag_kr<LDM>(As, (wm * MI + i) * 16, kk, lane);
#else
            af[i] = frag_kc(As, (wm * MI + i) * 16, kk, lane);
#endif
#pragma unroll
        for (int j = 0; j < NI; ++j) bf[j] = frag_kr<LDN>(Bs, (wn * NI + j) * 16, kk, lane);
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) acc[i][j] = MFMA(af[i], bf[j], acc[i][j]);
    }
}

// The whole reduction of one tile.  edge_a, edge_b: its pieces may have to be shifted (constants with KEEP).
__device__ __forceinline__ void walk(f32x4 (&acc)[MI][NI], const Plan &plan, const u16 *__restrict__ Ab, const u16 *__restrict__ Bb, u16 *As, u16 *Bs,
                                     bool edge_a, bool edge_b, int m0, int n0, int wm, int wn, int lane, int tid, int bi)
{
    // slab j of the walk, if there is one, into or from a set of registers
    Slab slab[DEPTH];
    auto load = [&](int j, int d) {
        if (j < NSL) load_slab(slab[d], plan, Ab, Bb, j, j == NSL - 1, m0, n0, tid);
    };
    auto store = [&](int j, int d, int stage) {
#if RECALC
        if (j < NSL) store_slab(slab[d], j, As + stage * A_STAGE, Bs + stage * B_STAGE, m0, n0, tid);
#else
        if (j < NSL) store_slab(slab[d], plan, As + stage * A_STAGE, Bs + stage * B_STAGE, j == NSL - 1, edge_a, edge_b, m0, n0, tid);
#endif
    };
    auto compute = [&](int stage) { compute_slab(acc, As + stage * A_STAGE, Bs + stage * B_STAGE, wm, wn, lane); };
#if NSTG == 2
    if (bi > 0) __syncthreads();                       // the previous batch's last slab has been multiplied
#if KEEP
    // Slab s in stage s & 1, slabs s+1 .. s+DEPTH in registers or on their way there: slab j in set j % DEPTH.  The steps whose slabs
    // may be the last one, or past it, are laid out one by one.
#pragma unroll
    for (int d = 0; d < DEPTH; ++d) load(d, d);
    store(0, 0, 0);
    load(DEPTH, 0);
    __syncthreads();
    constexpr int MAIN = NSL > DEPTH + 2 ? (NSL - DEPTH - 2) / DEPTH * DEPTH : 0;
#pragma unroll 1
    for (int s0 = 0; s0 < MAIN; s0 += DEPTH) {
#pragma unroll
        for (int d = 0; d < DEPTH; ++d) {
            const int s = s0 + d, set = (d + 1) % DEPTH;
            __builtin_amdgcn_sched_barrier(0);
            compute(s & 1);
            __builtin_amdgcn_sched_barrier(0);
            store_slab(slab[set], plan, As + (~s & 1) * A_STAGE, Bs + (~s & 1) * B_STAGE, false, edge_a, edge_b, m0, n0, tid);
            load_slab(slab[set], plan, Ab, Bb, s + 1 + DEPTH, false, m0, n0, tid);
            __syncthreads();
        }
    }
#pragma unroll
    for (int s = MAIN; s < NSL; ++s) {
        __builtin_amdgcn_sched_barrier(0);
        compute(s & 1);
        __builtin_amdgcn_sched_barrier(0);
        store(s + 1, (s + 1) % DEPTH, ~s & 1);
        load(s + 1 + DEPTH, (s + 1) % DEPTH);
        if (s + 1 < NSL) __syncthreads();
    }
#else
    // (large tiles: one loop whose last pass loads and stores the last slab once more, into the stage nobody reads any longer)
    load(0, 0);
    store(0, 0, 0);
    __syncthreads();
#pragma unroll 1
    for (int s = 0; s < NSL; ++s) {
        const int sn = s + 1 < NSL ? s + 1 : NSL - 1;
        load(sn, 0);
        __builtin_amdgcn_sched_barrier(0);
        compute(s & 1);
        __builtin_amdgcn_sched_barrier(0);
        store(sn, 0, ~s & 1);
        __syncthreads();
    }
#endif
#else
    auto step = [&](int s, bool last) {
        load_slab(slab[0], plan, Ab, Bb, s, last, m0, n0, tid);
        __syncthreads();
        store_slab(slab[0], plan, As, Bs, last, edge_a, edge_b, m0, n0, tid);
        __syncthreads();
        compute(0);
    };
#pragma unroll 1
    for (int s = 0; s < NSL - KEEP; ++s) step(s, !KEEP && s == NSL - 1);
    if (KEEP) step(NSL - 1, true);
    __syncthreads();
#endif
}

extern "C" __global__ __launch_bounds__(NT, MINW)
void KERNEL_NAME(const u16 *__restrict__ A, const u16 *__restrict__ B, float *__restrict__ C,
                 unsigned long long *ctl /* unused: members of this template are never folded */)
{
    extern __shared__ __attribute__((aligned(16))) u16 smem[];
    u16 *const As = smem, *const Bs = smem + NSTG * A_STAGE;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave / WN, wn = wave % WN;
    const BlockId bid = block_id();
    const int m0 = bid.m * BM, n0 = bid.n * BN;
    Plan plan;
    if (KEEP) plan_slab(plan, m0, n0, tid);

    for (int bi = 0; bi < BATCH_INNER; ++bi) {
#if KSPLIT > 1   // MatMul, reduction split over grid z: this workgroup owns K range [bid.b * KPART, + KPART)
        const long batch = 0, kb = (long)bid.b * KPART;
#else
        const long batch = (long)bid.b * BATCH_INNER + bi, kb = 0;
#endif
#if A_TRANS
        const u16 *Ab = A + batch * M * K + kb * M;
#else
        const u16 *Ab = A + batch * M * K + (long)m0 * K + kb;
#endif
        const u16 *Bb = B + batch * K * N + kb * N;
        float *Cb = C + batch * M * N;

        f32x4 acc[MI][NI];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int r = 0; r < 4; ++r) acc[i][j][r] = 0.f;

        const bool edge_a = A_TRANS && edge_tile(BM, m0, M), edge_b = edge_tile(BN, n0, N);
        auto run = [&](bool ea, bool eb) { walk(acc, plan, Ab, Bb, As, Bs, ea, eb, m0, n0, wm, wn, lane, tid, bi); };
        if (!KEEP) run(edge_a, edge_b);
        else if (edge_a) { if (edge_b) run(true, true); else run(true, false); }
        else if (edge_b) run(false, true);
        else run(false, false);
        // register r of an atom is row 4 * (l / 16) + r of column l % 16
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const int row = (wm * MI + i) * 16 + 4 * (lane / 16), col = (wn * NI + j) * 16 + lane % 16;
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    if (row + r < BM && col < BN) c_out(&Cb[(long)(m0 + row + r) * N + n0 + col], acc[i][j][r]);
            }
    }
}

#endif
