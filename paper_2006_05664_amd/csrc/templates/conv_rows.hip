// Conv2d kernel template for few input channels (bf16 / fp16 inputs, fp32 accumulation) on gfx950: images of fewer than 16
// channels, whose reduction has no 8 consecutive channels to offer the matrix units.
//
// A workgroup owns BM output channels x a box of NB2 images x BH rows x BW pixels, as on the other templates.  The 8 reduction
// values an MFMA lane supplies are 8 consecutive taps of one kernel row: for an output pixel (y, x) and kernel row (ci, r)
// these are the image values (ci, y*STRIDE + r, x*STRIDE + s .. + 8), consecutive in memory and in LDS.  The reduction is walked as (ci, r, s)
// with every kernel row padded to WKP = 8 or 16 taps (363 -> 528 for 3 channels of 11 x 11; the slabs of 11 taps padded
// to the MFMA step that the register-staged template takes are 1056, and gathered value by value).
//   * The patch: the image rows under the box as the NCHW image has them, all channels and all kernel rows at once,
//     P[image][ci][py][PITCH]; filled with 16-byte pieces at any alignment, without a transposition.  With padding, a piece
//     that would cross an end of its image row is loaded from inside the row and shifted, and positions outside the image are
//     zeros; without, only the tensor's end is kept (no stored pixel uses what then stands past a row).
//     A thread keeps its place in the row from pass to pass: with the piece's number taken apart by every extent, and each crossing
//     piece shifted, 512 x 3 x 227 x 227 below took 233 us; now 205.
//     A fragment is 16 bytes at x*STRIDE elements.  With an odd stride every second pixel starts at an odd element; those read a second copy
//     of the patch that lies one element further left (NCOPY = 2), so that every fragment is at least 4-byte aligned.
//   * Every wave keeps the kernel tensor's fragments of its own output channels for the whole reduction in registers (STEPS x MI of them).  They come
//     through the LDS where that has room (STAGE_A): the workgroup's rows are one run of memory, loaded by consecutive lanes and picked apart
//     there.  Straight from memory every lane of a fragment's load is in a cache line of its own, 68 cycles of the load unit each, for
//     33 of them 60 % of what one box of 11 x 11 taps took (5 x 3 x 64 x 64 * 64 x 3 x 11 x 11, stride 2: 12.9 -> 7.0 us; 99 x 3 x 56 x 56 * 64 x 3 x 5 x 5 35.0 -> 26.5).
//   * Taps past the kernel's width (and kernel rows past its height, where a step takes several) are zeros in the kernel tensor's
//     fragments AND are cleared in the image's: what the patch holds there are other pixels, which may be infinite.
// Measured: 512 x 3 x 227 x 227 * 64 x 3 x 11 x 11, stride 4, bf16 (boxes of 4 images x 55 pixels): 980 us on the register-staged template (73
// TFLOP/s: some ten instructions per gathered value), here 198 - 215 us with the output stored column by column, 173 - 184 us row by row, and
// 161 us with the kernel tensor through the LDS (450 TFLOP/s, 3.4 TB/s).  What bounds it: 396 MB of output in rows of 220 bytes that begin anywhere in a cache line (alone, without fill and
// multiplication, 136 us column by column and 109 row by row; non-temporal stores take 386, a contiguous run of boxes per
// workgroup 249), and that a box's load, multiplication and store follow one another, with two workgroups per compute unit (of 163 us, without
// the stores 116, without the fill 134, without the multiplication 168: that is covered by the other workgroup).
// PERSIST > 0: that many workgroups along the boxes, each taking several; the kernel tensor is then fetched once per workgroup.
// Boxes are dealt so that the workgroups of one XCD (every eighth) walk one contiguous eighth of them: boxes one above the other share
// HK - STRIDE of their image rows, through that XCD's L2.

#if IN_DTYPE == 1
typedef __attribute__((ext_vector_type(8))) __bf16 frag_t;
#define MFMA_32(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0)
#define MFMA_16(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0)
#else
typedef __attribute__((ext_vector_type(8))) _Float16 frag_t;
#define MFMA_32(a, b, c) __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0)
#define MFMA_16(a, b, c) __builtin_amdgcn_mfma_f32_16x16x32_f16(a, b, c, 0, 0, 0)
#endif
#if ATOM == 32
typedef f32x16 acc_t;
#define KA 16
#define NACC 16
#define MFMA(a, b, c) MFMA_32(a, b, c)
#else
typedef f32x4 acc_t;
#define KA 32
#define NACC 4
#define MFMA(a, b, c) MFMA_16(a, b, c)
#endif

typedef u32x4 __attribute__((aligned(2))) u32x4_a2;
typedef u32x4 __attribute__((aligned(STRIDE % 4 == 0 ? 8 : 4))) frag_mem;

constexpr int G = KA / 8;                          // groups of 8 taps in an MFMA step
constexpr int Q = WKP / 8;                         // groups of a kernel row: 1 or 2, so a step takes whole kernel rows
constexpr int RPS = G / Q;                         // kernel rows per step
constexpr int SPC = (HK + RPS - 1) / RPS;          // steps per channel
constexpr int STEPS = CIN * SPC;
constexpr bool ROW_TAIL = SPC * RPS != HK;         // the last step of a channel has kernel rows past the kernel
constexpr int PH = (BH - 1) * STRIDE + HK, PW = (BW - 1) * STRIDE + WK;
constexpr int CPR = (PW + 7) / 8, PITCH = CPR * 8; // pieces and elements per patch row
constexpr int NCOPY = STRIDE % 2 ? 2 : 1;
constexpr int ROWS = NB2 * CIN * PH;
// elements of a copy: the rows, what fragments of its last row may read past them, and (two copies) enough to put the second
// copy on the other half of the banks
constexpr int COPY_MIN = ROWS * PITCH + (SPC * RPS - HK) * PITCH + WKP;
constexpr int COPY = NCOPY == 2 ? (COPY_MIN + 127) / 128 * 128 + 64 : (COPY_MIN + 7) / 8 * 8;
constexpr int A_ROWS = BM * K + 128;               // elements of the workgroup's rows of the kernel tensor in the LDS, and what fragments of the last one may read past them
static_assert(NCOPY * COPY * 2 + BESIDE == LDS_BYTES && (STAGE_A != 1 || A_ROWS * 2 <= LDS_BYTES) && (STAGE_A != 2 || A_ROWS * 2 == BESIDE) && COPY % 8 == 0, "decoder and template disagree");
static_assert(WK <= WKP && (WKP == 8 || WKP == 16) && WIN >= 8 && BM == WM * MI * ATOM && WN * NI * ATOM >= BN && NT == 64 * WM * WN, "decoder and template disagree");
// The fill's split: TPR threads along a patch row, RPP rows at a time, so that a thread keeps its place in the row (XP places if
// the row is longer than the workgroup) and a pass costs it one small division instead of one of every extent.
constexpr int TPR = CPR < NT ? CPR : NT, RPP = NT / TPR, XP = (CPR + NT - 1) / NT;
constexpr int ROW_PASSES = (ROWS + RPP - 1) / RPP, PASSES = NCOPY * XP * ROW_PASSES;
constexpr int BATCH = (PASSES + (PASSES + 17) / 18 - 1) / ((PASSES + 17) / 18);   // pieces a thread has in flight at a time: at most 18, evenly

struct Pass {                                      // pass p: which copy, the rows from which on, the place's offset
    int copy, row, place;
    __device__ __forceinline__ constexpr Pass(int p) : copy(p / (ROW_PASSES * XP)), row(p / XP % ROW_PASSES * RPP), place(p % XP * NT) {}
};
// row / PH for 0 <= row < ROWS + RPP (a 24-bit multiplication where the product stays exact)
__device__ __forceinline__ int div_rows(int row)
{
    if constexpr ((ROWS + RPP) * PH < (1 << 20) && ROWS + RPP <= 4095 && PH > 1) return (int)(((u32)row & 4095u) * ((1u << 20) / PH + 1) >> 20);
    return row / PH;
}

// v shifted by sh elements towards element 0 (sh > 0) or away from it (sh < 0), zeros shifted in; 8 and more: all zeros
__device__ __forceinline__ u32x4 shift_elements(u32x4 v, int sh)
{
    u32 w0 = v.x, w1 = v.y, w2 = v.z, w3 = v.w;
    const int n = sh < 0 ? -sh : sh;
    if (sh > 0) {
        if (n & 1) { w0 = (w0 >> 16) | (w1 << 16); w1 = (w1 >> 16) | (w2 << 16); w2 = (w2 >> 16) | (w3 << 16); w3 >>= 16; }
        if (n & 2) { w0 = w1; w1 = w2; w2 = w3; w3 = 0; }
        if (n & 4) { w0 = w2; w1 = w3; w2 = 0; w3 = 0; }
    } else {
        if (n & 1) { w3 = (w3 << 16) | (w2 >> 16); w2 = (w2 << 16) | (w1 >> 16); w1 = (w1 << 16) | (w0 >> 16); w0 <<= 16; }
        if (n & 2) { w3 = w2; w2 = w1; w1 = w0; w0 = 0; }
        if (n & 4) { w3 = w1; w2 = w0; w1 = 0; w0 = 0; }
    }
    if (n >= 8) w0 = w1 = w2 = w3 = 0;
    const u32x4 r = {w0, w1, w2, w3};
    return r;
}

// Clears the taps past the kernel's width.  Per 4-byte word (two taps): all lanes keep it, none does, all keep half of it,
// or (two groups per kernel row) it depends on the lane's group.
struct TapMask { u32 w[4]; u32 row; };
__device__ __forceinline__ u32x4 keep_taps(u32x4 v, const TapMask &m, bool row_tail)
{
#pragma unroll
    for (int d = 0; d < 4; ++d) {
        if (WKP - 8 + 2 * d + 1 < WK) continue;
        if (2 * d >= WK) v[d] = 0;
        else if (Q == 1) v[d] &= 0xffffu;
        else v[d] &= m.w[d];
    }
    if (row_tail) {
#pragma unroll
        for (int d = 0; d < 4; ++d) v[d] &= m.row;
    }
    return v;
}

extern "C" __global__ __launch_bounds__(NT, 2)
void KERNEL_NAME(const u16 *__restrict__ A, const u16 *__restrict__ B, float *__restrict__ C,
                  unsigned long long *ctl /* unused: members of this template are never folded */)
{
    extern __shared__ __attribute__((aligned(16))) u16 smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6, wm = wave / WN, wn = wave % WN;
    const int lrow = lane % ATOM, kg = lane / ATOM;             // kg: which group of 8 taps of a step the lane supplies
    const BlockId bid = block_id();
    const int m0 = bid.m * BM;

    TapMask mask;
    {
        const int s0 = kg % Q * 8;
#pragma unroll
        for (int d = 0; d < 4; ++d) mask.w[d] = (s0 + 2 * d < WK ? 0xffffu : 0u) | (s0 + 2 * d + 1 < WK ? 0xffff0000u : 0u);
        mask.row = (SPC - 1) * RPS + kg / Q < HK ? ~0u : 0u;
    }
    // the kernel tensor's fragments: lane = output channel, 8 taps from (ci, r, s0)
    frag_t af[MI][STEPS];
#if STAGE_A
    {
#if STAGE_A == 1   // where the patch will be
        u16 *const rows = smem;
#else   // (an array of its own, which the compiler knows to be another than the patch: 15.8 -> 16.1, 10.2 -> 10.4, 5.9 -> 6.0 us behind the patch in the same one)
        __shared__ __attribute__((aligned(16))) u16 rows[A_ROWS];
#endif
        constexpr int PIECES = BM * K / 8, NP = (PIECES + NT - 1) / NT, AT_ONCE = NP < 16 ? NP : 16;
        const u32x4_a2 *const from = (const u32x4_a2 *)(A + (long)m0 * K);
        for (int p0 = 0; p0 < NP; p0 += AT_ONCE) {
            u32x4 v[AT_ONCE];
#pragma unroll
            for (int i = 0; i < AT_ONCE; ++i) v[i] = from[min(tid + (p0 + i) * NT, PIECES - 1)];
#pragma unroll
            for (int i = 0; i < AT_ONCE; ++i)
                if (tid + (p0 + i) * NT < PIECES) ((u32x4 *)rows)[tid + (p0 + i) * NT] = v[i];
        }
        __syncthreads();
        const int r0 = kg / Q, s0 = kg % Q * 8;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            // Words from the one that holds the first tap; where that is the word's upper half, the fragment is half a word further on.  at + step is
            // that word for an even number of taps before a step's, one further for an odd one where the lane's own first tap is odd.
            const int first = ((wm * MI + i) * ATOM + lrow) * K + r0 * WK + s0, odd = first & 1;
            const u32 *const at = (const u32 *)rows + (first >> 1);
#pragma unroll
            for (int t = 0; t < STEPS; ++t) {
                const int step = (t / SPC * HK + t % SPC * RPS) * WK;
                const u32 *const w = (step & 1 ? at + odd : at) + (step >> 1);
                u32x4 v = {w[0], w[1], w[2], w[3]};
                if (K % 2 != 0 || WK % 2 != 0) {
                    const u32 sh = (u32)(odd ^ (step & 1)) << 4;
                    v.x = __builtin_amdgcn_alignbit(v.y, v.x, sh); v.y = __builtin_amdgcn_alignbit(v.z, v.y, sh);
                    v.z = __builtin_amdgcn_alignbit(v.w, v.z, sh); v.w = __builtin_amdgcn_alignbit(w[4], v.w, sh);
                }
                af[i][t] = __builtin_bit_cast(frag_t, keep_taps(v, mask, ROW_TAIL && t % SPC == SPC - 1));
            }
        }
    }
#else
    {
        const int r0 = kg / Q, s0 = kg % Q * 8;
#pragma unroll
        for (int i = 0; i < MI; ++i) {
            const int row0 = (m0 + (wm * MI + i) * ATOM + lrow) * K + r0 * WK + s0;
#pragma unroll
            for (int t = 0; t < STEPS; ++t) {
                const int ci = t / SPC, tr = t % SPC * RPS;
                // (a step whose 8 taps may reach past the end of the tensor, in its last rows: loaded from further left)
                const bool risky = (ci * HK + tr + RPS - 1) * WK + (Q - 1) * 8 + 8 > K;
                const int at = row0 + (ci * HK + tr) * WK;
                const int from = risky ? min(at, M * K - 8) : at;
                u32x4 v = *(const u32x4_a2 *)((const char *)A + 2u * (u32)from);
                if (risky && at != from) v = shift_elements(v, at - from);
                af[i][t] = __builtin_bit_cast(frag_t, keep_taps(v, mask, ROW_TAIL && t % SPC == SPC - 1));
            }
        }
    }
#endif
    // this lane's places in the patch: per column of atoms its output pixel under tap (0, 0), plus its group of taps
    // (columns past the box read its last pixel and are not stored)
    int b_lane[NI];
#pragma unroll
    for (int j = 0; j < NI; ++j) {
        const int ct = (wn * NI + j) * ATOM + lrow, cn = ct < BN ? ct : BN - 1;
        const int b = cn / (BH * BW), y = (cn / BW) % BH, xs = cn % BW * STRIDE, odd = NCOPY == 2 ? xs & 1 : 0;
        b_lane[j] = odd * COPY + (b * CIN * PH + y * STRIDE + kg / Q) * PITCH + xs - odd + kg % Q * 8;
    }

#if PERSIST > 0
    constexpr int PER_XCD = (NBOX + 7) / 8;
    const int last = min(NBOX, ((int)blockIdx.x % 8 + 1) * PER_XCD);
    for (int box = (int)blockIdx.x % 8 * PER_XCD + (int)blockIdx.x / 8; box < last; box += PERSIST / 8) {
#else
    {
        const int box = bid.n;
#endif
        const ColBlock cb = col_block(box);
        const int yin0 = cb.y0 * STRIDE - PAD_CONV, xin0 = cb.x0 * STRIDE - PAD_CONV;
        const u16 *img = B + (long)cb.nb0 * CIN * HIN * WIN;
        // the last element a piece may start at (this box's images start at 0)
        const int end = (int)min(((long)(N / (HOUT * WOUT)) - cb.nb0) * CIN * HIN * WIN - 8, 0x7fffffffL);
        // (the thread number is opaque to the compiler: the places of a thread's pieces would otherwise be kept in registers
        // from box to box and from the loads to the stores, next to the kernel tensor, and spill)
        for (int p0 = 0; p0 < PASSES; p0 += BATCH) {
            u32x4 v[BATCH];
            int ptid = tid;
            asm volatile("" : "+v"(ptid));
            ptid &= 1023;
            const int first = ptid / TPR, place = ptid % TPR;
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                if (p0 + i >= PASSES) break;
                const Pass ps(p0 + i);
                const int row = first + ps.row, c = place + ps.place, x = xin0 + c * 8 + ps.copy;
                const int plane = div_rows(row), r = row - plane * PH, y = yin0 + r;
                const u32x4 zero = {0u, 0u, 0u, 0u};
                v[i] = zero;
                const bool mine = (RPP * TPR == NT || first < RPP) && (ps.row + RPP <= ROWS || row < ROWS) && (XP == 1 || c < CPR);
                if (PAD_CONV == 0) {
                    // nothing a stored pixel uses lies past the image row: what follows it in memory may stand there
                    const int at = (plane * HIN + y) * WIN + x;
                    if (mine) v[i] = *(const u32x4_a2 *)((const char *)img + 2u * (u32)min(at, end));
                } else if (mine && (unsigned)y < (unsigned)HIN)
                    v[i] = *(const u32x4_a2 *)((const char *)img + 2u * (u32)((plane * HIN + y) * WIN + min(max(x, 0), WIN - 8)));
            }
            if (p0 == 0) __syncthreads();                      // the previous box has been multiplied
            asm volatile("" : "+v"(ptid));
            ptid &= 1023;
            const int first2 = ptid / TPR, place2 = ptid % TPR;
#pragma unroll
            for (int i = 0; i < BATCH; ++i) {
                if (p0 + i >= PASSES) break;
                const Pass ps(p0 + i);
                const int row = first2 + ps.row, c = place2 + ps.place, x = xin0 + c * 8 + ps.copy;
                int sh = x - min(max(x, 0), WIN - 8);
                if (PAD_CONV == 0) {
                    const int plane = div_rows(row), at = (plane * HIN + yin0 + row - plane * PH) * WIN + x;
                    sh = max(at - end, 0);
                }
                if (sh != 0) v[i] = shift_elements(v[i], sh);
                if ((RPP * TPR == NT || first2 < RPP) && (ps.row + RPP <= ROWS || row < ROWS) && (XP == 1 || c < CPR))
                    *(u32x4 *)(smem + ps.copy * COPY + row * PITCH + c * 8) = v[i];
            }
        }
        __syncthreads();

        acc_t acc[MI][NI];
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int r = 0; r < NACC; ++r) acc[i][j][r] = 0.f;
        // one set of the image's fragments: each is read again for the next step as soon as its taps are picked out
        u32x4 bf[NI];
#pragma unroll
        for (int j = 0; j < NI; ++j) bf[j] = *(const frag_mem *)(smem + b_lane[j]);
#pragma unroll
        for (int t = 0; t < STEPS; ++t) {
            const int off = ((t + 1) / SPC * PH + (t + 1) % SPC * RPS) * PITCH;
#pragma unroll
            for (int j = 0; j < NI; ++j) {
                const frag_t b = __builtin_bit_cast(frag_t, keep_taps(bf[j], mask, ROW_TAIL && t % SPC == SPC - 1));
                if (t + 1 < STEPS) bf[j] = *(const frag_mem *)(smem + b_lane[j] + off);
#pragma unroll
                for (int i = 0; i < MI; ++i) acc[i][j] = MFMA(af[i][t], b, acc[i][j]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        // an atom's result sits with column (l % ATOM) in lane l; 32x32: register r is row 8*(r/4) + 4*(l/32) + r%4;
        // 16x16: register r is row 4*(l/16) + r
        // Row by row, all of a row's columns one after the other: the atoms of a row share cache lines (rows of 55 pixels begin anywhere in
        // one), and a line that is completed at once is written to memory once (512 x 3 x 227 x 227 above, 396 MB of output: 214 us column by column, 184 so).
        float *const out = C + (((long)cb.nb0 * M + m0 + wm * MI * ATOM) * HOUT + cb.y0) * WOUT + cb.x0;
        out_off at[NI];                                    // byte offsets of the lane's columns, in its first row of an atom
        bool on[NI];
#pragma unroll
        for (int j = 0; j < NI; ++j) {
            const int cn = (wn * NI + j) * ATOM + lrow;
            on[j] = cn < BN;
            at[j] = conv_c_offset(lane / ATOM * 4, cn);
        }
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int r = 0; r < NACC; ++r) {
                char *const row = (char *)(out + (long)(i * ATOM + 8 * (r / 4) + r % 4) * (HOUT * WOUT));
#pragma unroll
                for (int j = 0; j < NI; ++j)
                    if (on[j]) *(float *)(row + at[j]) = acc[i][j][r];
            }
    }
}
