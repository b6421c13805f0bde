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
// What bounds it: at these tiles the LDS (1000^3: per slab and compute unit some 1500 of its cycles, fragments that every wave reads for itself and bank
// conflicts) and the phases of a slab that follow one another, loads, stores and multiplication in equal parts; deeper prefetch gains nothing there.
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

#if IN_DTYPE == 1
typedef __attribute__((ext_vector_type(8))) __bf16 frag_t;
#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0)
#else
typedef __attribute__((ext_vector_type(8))) _Float16 frag_t;
#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0)
#endif
#if !KEEP   // nothing of a plan for two slabs under way, or for a second workgroup's registers, holds
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

constexpr int KPART = K / KSPLIT;                 // reduction length of this workgroup
static_assert(NSL * KS >= KPART && (NSL - 1) * KS < KPART && KS % 32 == 0 && KPART >= 8, "decoder and template disagree");
static_assert(WM * MI * 16 >= BM && WN * NI * 16 >= BN && NT == 64 * WM * WN, "decoder and template disagree");
constexpr bool K_TAIL = KPART % KS != 0;          // the last slab is not full

constexpr int odd16(int n) { return ((n + 15) / 16 | 1) * 16; }
constexpr int LDK = KS + 8;                       // elements per LDS row of a k-contiguous operand
constexpr int LDM = odd16(WM * MI * 16), LDN = odd16(WN * NI * 16);
__device__ __forceinline__ constexpr int kr_off(int ld, int k) { return k * ld + (k >> 3) * 64; }   // LDS element of k row k
constexpr int A_STAGE = A_TRANS ? KS * LDM + (KS / 8) * 64 : WM * MI * 16 * LDK;
constexpr int B_STAGE = KS * LDN + (KS / 8) * 64;
static_assert(NSTG * (A_STAGE + B_STAGE) * 2 <= LDS_BYTES, "stages exceed the LDS the host asks for");
constexpr int CK = KS / 8;                        // pieces of a k-contiguous row
constexpr int CM = (BM + 7) / 8, CN = (BN + 7) / 8;   // pieces of a k row
constexpr int A_PIECES = A_TRANS ? KS * CM : BM * CK, B_PIECES = KS * CN;
constexpr int NA = (A_PIECES + NT - 1) / NT, NB = (B_PIECES + NT - 1) / NT;

struct Slab { u32x4 a[NA], b[NB]; };

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
