// MFMA kernel template (bf16 / fp16 inputs, fp32 accumulation, 16x16x32 atoms) for MatMul / BatchMatMul operators whose
// extents are no multiples of 16, so that no member of their spaces has wave tiles of whole atoms and rows at 16-byte
// offsets: every such member used to run on the scalar template, which reads two LDS words per multiply-add.
//
// A workgroup owns the member's BM x BN tile, whatever its extents.  The tile is rounded up to whole atoms and dealt to
// WM x WN waves of MI x NI atoms (the host picks the division; a member's own wave tiles, factors of 125 or 27, would each
// be rounded up by themselves).  What the atoms compute past the tile is not stored.  The reduction is walked in NSL slabs
// of KS (the member's slab rounded up to whole MFMA steps), the last one filled up with zeros in both operands.
//
// Measured (bf16): 1000^3 in tiles of 20 x 100 168 us on the scalar template (20 waves, the best there), 15.6 us here (128 TFLOP/s); 105 x 972 x 160 in
// tiles of 15 x 54 60 -> 3.6 us; a batch of 11 x (35 x 36 x 35) 6.2 -> 3.5 us.
// What bounds it: at these tiles the operand stream (1000^3 in tiles of 20 x 100: 0.12 GB through L2) and, with two workgroups per
// compute unit, the chain of 11 slabs (counters: matrix pipes 13 %, LDS 40 % of the busy time, a third of that bank conflicts), so the point
// is to move it in wide pieces whatever the alignment: every operand travels in 16-byte pieces of 8 consecutive elements,
// loaded at the 2-byte alignment an odd row length leaves.  A piece that would reach past its row is loaded from as far left as
// it must be to end with the row, and shifted down when it is stored: no load leaves its operand's rows.
//   * A [M][K]: pieces along k.  LDS As[row][KS + 8]: a fragment is one 16-byte read; the odd number of pieces per row spreads 16 rows
//     over all banks.
//   * B [K][N] (and a first operand stored [K][M]): pieces along n.  LDS Bs[k][LDX] as memory has it, fragments read with the
//     transposing LDS load (two per fragment).  LDX is an odd multiple of 32 bytes and every 8 rows lie 128 bytes
//     further, so the 4 rows x 32 bytes that two groups of 16 lanes read together (8 rows apart) fall into 8 different groups of banks.
// NSTG = 2: the pieces of slab s+1 are in registers while slab s is multiplied and are stored to the other stage afterwards
// (one barrier per slab).  NSTG = 1: load, barrier, store, barrier, multiply.

#if IN_DTYPE == 1
typedef __attribute__((ext_vector_type(8))) __bf16 frag_t;
#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0)
#else
typedef __attribute__((ext_vector_type(8))) _Float16 frag_t;
#define MFMA(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0)
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
    // A last piece can reach past the row's end in the last tile, and with tiles of 2 and 3 also in the ones before it (8 past the
    // start of a tile is then more than two tiles on); whole multiples of 8 never do.
    constexpr bool EARLIER_TOO = (TILE + 7) / 8 * 8 > 2 * TILE;
    if (TILE % 8 != 0 && (EARLIER_TOO || x0 + TILE == LEN)) v = shift_down(v, max(x0 + x - (LEN - 8), 0));
    if (K_TAIL && last && k0 + kr >= KPART) { const u32x4 z = {0u, 0u, 0u, 0u}; v = z; }
    *(u32x4 *)(S + kr_off(LD, kr) + x) = v;
}

__device__ __forceinline__ void load_slab(Slab &s, const u16 *__restrict__ Ab, const u16 *__restrict__ Bb, int m0, int n0, int k0, int tid)
{
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int q = tid + i * NT;
        if (A_PIECES % NT == 0 || q < A_PIECES) {
#if A_TRANS
            s.a[i] = load_kr<M, CM>(Ab, q, k0, m0);
#else
            s.a[i] = load_kc(Ab, q, k0);
#endif
        }
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int q = tid + i * NT;
        if (B_PIECES % NT == 0 || q < B_PIECES) s.b[i] = load_kr<N, CN>(Bb, q, k0, n0);
    }
}

__device__ __forceinline__ void store_slab(const Slab &s, u16 *As, u16 *Bs, int m0, int n0, int k0, bool last, int tid)
{
#pragma unroll
    for (int i = 0; i < NA; ++i) {
        const int q = tid + i * NT;
        if (A_PIECES % NT == 0 || q < A_PIECES) {
#if A_TRANS
            store_kr<M, CM, LDM, BM>(As, s.a[i], q, k0, m0, last);
#else
            store_kc(As, s.a[i], q, k0, last);
#endif
        }
    }
#pragma unroll
    for (int i = 0; i < NB; ++i) {
        const int q = tid + i * NT;
        if (B_PIECES % NT == 0 || q < B_PIECES) store_kr<N, CN, LDN, BN>(Bs, s.b[i], q, k0, n0, last);
    }
}

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

extern "C" __global__ __launch_bounds__(NT)
void KERNEL_NAME(const u16 *__restrict__ A, const u16 *__restrict__ B, float *__restrict__ C,
                 unsigned long long *ctl /* unused: members of this template are never folded */)
{
    extern __shared__ __attribute__((aligned(16))) u16 smem[];
    u16 *const As = smem, *const Bs = smem + NSTG * A_STAGE;
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, wm = wave / WN, wn = wave % WN;
    const BlockId bid = block_id();
    const int m0 = bid.m * BM, n0 = bid.n * BN;

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

        Slab slab;
#if NSTG == 2
        if (bi > 0) __syncthreads();                   // the previous batch's last slab has been multiplied
        load_slab(slab, Ab, Bb, m0, n0, 0, tid);
        store_slab(slab, As, Bs, m0, n0, 0, NSL == 1, tid);
        __syncthreads();
#pragma unroll 1
        for (int s = 0; s < NSL; ++s) {
            const int cur = s & 1, nxt = cur ^ 1;
            // past the last slab: the last once more, into the stage nobody reads any longer
            const int sn = s + 1 < NSL ? s + 1 : NSL - 1;
            load_slab(slab, Ab, Bb, m0, n0, sn * KS, tid);
            __builtin_amdgcn_sched_barrier(0);
            compute_slab(acc, As + cur * A_STAGE, Bs + cur * B_STAGE, wm, wn, lane);
            __builtin_amdgcn_sched_barrier(0);
            store_slab(slab, As + nxt * A_STAGE, Bs + nxt * B_STAGE, m0, n0, sn * KS, sn == NSL - 1, tid);
            __syncthreads();
        }
#else
#pragma unroll 1
        for (int s = 0; s < NSL; ++s) {
            load_slab(slab, Ab, Bb, m0, n0, s * KS, tid);
            __syncthreads();
            store_slab(slab, As, Bs, m0, n0, s * KS, s == NSL - 1, tid);
            __syncthreads();
            compute_slab(acc, As, Bs, wm, wn, lane);
        }
        __syncthreads();
#endif
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
