// Conv2d kernel template with an LDS-resident image patch whose wave tiles are rows of pixels (bf16 / fp16 inputs, fp32
// accumulation, unit stride) for gfx950.
//
// Same workgroup tile and operands (image NCHW, kernel tensor OIHW, one launch) as the patch template, and the same walk of the reduction
// in slabs of CS input channels with all their taps.  What differs:
//   * Who multiplies what.  The columns of an MFMA are ATOM consecutive pixels of ONE row of the box (a strip), and a wave owns R rows one
//     above the other.  The fragment of input row y under tap column s then serves output row y - r for every tap row r: a wave reads
//     R + HK - 1 image fragments and HK x MI kernel fragments for HK x R x MI MFMAs, where the patch template, whose columns run across row ends,
//     reads every fragment again for every tap.  The 5x5 convolution below: 18 fragments for 45 MFMAs instead of 4 for 4.  The price are lanes without
//     a pixel (27 of 32); the host takes this template where at least four of five have one, and divides the tile among the waves
//     by a cost of its own.
//   * The patch has no padding: a pixel is CS elements = NCH 16-byte chunks, chunk c of pixel p stored at c ^ swz(p), and the row pitch is a multiple of
//     16 pixels, so that a row further down is a compile-time offset.  A 16-byte read is served in turns of 16 lanes (0-3, 12-15, 20-23, 24-27;
//     the other lanes below 32; the same plus 32): swz spreads the lanes of every turn over 16 different groups of banks, whatever tap shifts them.
//   * The fill.  A task is 8 channels x 2 pixels: eight 4-byte loads, two 16-byte stores.  Neighbouring lanes load neighbouring pixels: with
//     four channels side by side, as the patch template deals them, each lane is a cache line of its own to the
//     load unit (the 14 x 14 convolution 16.5 us so, 13.2 with the pixels first).
// Measured (bf16): 32 x 256 x 14 x 14 * 256 x 256 x 3 x 3 in tiles of 32 channels x one image 16.2 -> 11.7 us (630 TFLOP/s); 512 x 64 x 27 x 27 * 192 x
// 64 x 5 x 5 in tiles of 64 channels x 2 images x 9 rows 300 - 315 -> 234 - 238 us (970 TFLOP/s);
// 85 sampled members 1.23x in the geometric mean, the slowest 0.96x.
// What bounds it: the second by the matrix pipes' power (without any fill and store 171 us: 1.6 PFLOP/s counting the lanes without a pixel) and 287 MB
// of output, 30 us of which the other workgroup does not cover; the first by latency, one workgroup per compute unit: 3.6 us launch, prologue and
// epilogue, then 2.1 us per slab of 64 channels, of which the MFMAs take 0.9.  A second stage there (loads of the next slab during the
// multiplication) was measured: 12.6 instead of 12.4; slabs of 32 or 128 channels 12.2 and 13.0.  Non-temporal stores: 1 % faster on the
// second, 8 % slower on the first.
//
// KW > 1: KW waves share a wave tile and deal the (channel group, tap column) pairs of a slab among themselves; their sums meet in LDS at the end.
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

constexpr int T = HK * WK;                                    // taps
constexpr int PH = BH + HK - 1, PW = BW + WK - 1;             // the patch: input rows and columns under the box
constexpr int SPR = (BW + ATOM - 1) / ATOM;                   // strips of ATOM pixels per row
constexpr int RG = BH / R;                                    // groups of R rows
constexpr int NPIX = NB2 * PH * PWP;
constexpr int NCH = CS / 8;                                   // 16-byte chunks per pixel and per row of the kernel tensor's part
constexpr int KKS = CS / KA;                                  // MFMA steps per tap
constexpr int UNITS = KKS * WK;                               // (channel group, tap column) pairs of a slab, dealt to the KW waves of a tile
constexpr int DUMP = 8 * 64;                                  // 64 chunks that take the stores of pixels outside the patch or the image
constexpr int P_STAGE = NPIX * CS, A_STAGE = T * BM * CS, STAGE = P_STAGE + A_STAGE;   // elements
constexpr int DUMP_AT = STAGE;
constexpr int NWAVES = NT / 64;
static_assert(NCH == 2 || NCH == 4 || NCH == 8 || NCH == 16, "chunks are permuted by exclusive-or");
static_assert(STRIDE == 1 && RG * R == BH && BM == WM * MI * ATOM && WN == NB2 * SPR * RG && NWAVES == WM * WN * KW && PWP >= PW, "decoder and template disagree");
static_assert(CS % KA == 0 && UNITS % KW == 0 && NSTG == 1 && KSTEPS * CS == CIN && PWP % 16 == 0, "decoder and template disagree");
static_assert((DUMP_AT + DUMP) * 2 <= LDS_BYTES && LDS_BYTES <= 160 * 1024, "stages exceed the LDS");

// chunk permutation of pixel (or kernel-tensor row) p
__device__ __forceinline__ constexpr int swz(int p)
{
#if ATOM == 32
    return NCH == 16 ? p & 15 : (p / (16 / NCH)) % NCH;
#else
    return NCH == 16 ? (p & 7) * 2 : ((p / (16 / NCH)) % (NCH / 2)) * 2;
#endif
}

// Patch fill, pairs of pixels (even x, odd x): in images of odd width the loads are only 2-byte aligned and the last pixel of a row is loaded
// from one pixel to the left and shifted (bit 0 of the task's byte offset), so that no load reaches past its row.
constexpr bool ALIGNED = WIN % 2 == 0;
typedef u32 __attribute__((aligned(2))) u32_a2;
// A box as wide (high) as the output covers the whole image: only what lies inside it is filled.
constexpr bool FULL_X = W1 == 1, FULL_Y = H1 == 1;
constexpr int INX = PW - PAD_CONV < WIN ? PW - PAD_CONV : WIN, INY = PH - PAD_CONV < HIN ? PH - PAD_CONV : HIN;
constexpr int NPAIR = FULL_X ? (INX + 1) / 2 : PW / 2 + 1;
constexpr int NROW = FULL_Y ? INY : PH;
constexpr int PAIRS = NPAIR * NROW * NB2;
constexpr int P_TASKS = NCH * PAIRS;
constexpr int NPT = (P_TASKS + NT - 1) / NT;
// Kernel-tensor fill: a task is one output channel x two input channels, 2*T consecutive values; tap t of both makes one 4-byte store.
constexpr int CP = CS / 2;
constexpr int A_TASKS = BM * CP;
constexpr int NAT = (A_TASKS + NT - 1) / NT;

// Both parts' loads in flight at once where the registers hold them beside the accumulators
constexpr bool TOGETHER = MI * R * NACC + 11 * NPT + (T + 2) * NAT + 40 <= 512 / ((NWAVES + 3) / 4 > MINW ? (NWAVES + 3) / 4 : MINW);

struct Fill {
    u32 pg[NPT], pd0[NPT], pd1[NPT];      // image: byte offset of the pair, first channel, slab 0; the chunk each of its pixels goes to
    u32 ag[NAT], ad[NAT];                 // kernel tensor: byte offset of the values, slab 0; the word tap 0 goes to
};
struct PRegs { u32 p[NPT][8]; };
struct ARegs { u32 a[NAT][T]; };

__device__ __forceinline__ void plan_fill(Fill &f, const ColBlock &cb, int m0, int tid)
{
    const int yin0 = cb.y0 - PAD_CONV, xin0 = cb.x0 - PAD_CONV;
    const int xs = xin0 & ~1;
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        const int q = tid + i * NT;
        const int c = q / PAIRS, pr = q % PAIRS;
        const int jp = pr % NPAIR, b = pr / (NPAIR * NROW);
        const int y = (FULL_Y ? 0 : yin0) + (pr / NPAIR) % NROW, py = y - yin0, x = (FULL_X ? 0 : xs) + 2 * jp, px = x - xin0;
        const bool in = (P_TASKS % NT == 0 || q < P_TASKS) && y >= 0 && y < HIN && x >= 0 && x < WIN;
        const bool v0 = in && px >= 0 && px < PW, v1 = in && px + 1 >= 0 && px + 1 < PW && (ALIGNED || x + 1 < WIN);
        const int left = (!ALIGNED && x == WIN - 1) ? 1 : 0;
        const int p = (b * PH + py) * PWP + px, dump = DUMP_AT / 8 + (tid & 63);
        f.pg[i] = (v0 || v1) ? (2u * (u32)((((cb.nb0 + b) * CIN + 8 * c) * HIN + y) * WIN + x - left) | (u32)left) : 0u;
        f.pd0[i] = (u32)(v0 ? p * NCH + (c ^ swz(p)) : dump);
        f.pd1[i] = (u32)(v1 ? (p + 1) * NCH + (c ^ swz(p + 1)) : dump);
    }
#pragma unroll
    for (int i = 0; i < NAT; ++i) {
        const int q = tid + i * NT;
        const int cp = q % CP, m = q / CP;
        const bool on = A_TASKS % NT == 0 || q < A_TASKS;
        f.ag[i] = on ? 2u * (u32)((m0 + m) * K + 2 * cp * T) : 0u;
        f.ad[i] = on ? (u32)(m * (CS / 2) + (((cp >> 2) ^ swz(m)) << 2) + (cp & 3)) : ~0u;
    }
}

__device__ __forceinline__ void load_p(PRegs &r, const Fill &f, const u16 *__restrict__ B, int s)
{
    const char *Bs = (const char *)(B + (long)s * CS * HIN * WIN);
#pragma unroll
    for (int i = 0; i < NPT; ++i)
#pragma unroll
        for (int c = 0; c < 8; ++c) r.p[i][c] = *(const u32_a2 *)(Bs + (long)c * (2 * HIN * WIN) + (ALIGNED ? f.pg[i] : f.pg[i] & ~1u));
}
__device__ __forceinline__ void load_a(ARegs &r, const Fill &f, const u16 *__restrict__ A, int s)
{
    const char *As = (const char *)(A + (long)s * CS * T);
#pragma unroll
    for (int i = 0; i < NAT; ++i)
#pragma unroll
        for (int t = 0; t < T; ++t) r.a[i][t] = *(const u32 *)(As + f.ag[i] + 4 * t);
}
__device__ __forceinline__ void store_p(const PRegs &r, const Fill &f, u16 *S)
{
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
        u32 p[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) p[c] = ALIGNED ? r.p[i][c] : r.p[i][c] >> ((f.pg[i] & 1u) << 4);
        u32x4 w0, w1;
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            w0[c] = (p[2 * c] & 0xffffu) | (p[2 * c + 1] << 16);
            w1[c] = (p[2 * c] >> 16) | (p[2 * c + 1] & 0xffff0000u);
        }
        ((u32x4 *)S)[f.pd0[i]] = w0;
        ((u32x4 *)S)[f.pd1[i]] = w1;
    }
}
__device__ __forceinline__ void store_a(const ARegs &r, const Fill &f, u16 *S)
{
    u32 *SA = (u32 *)(S + P_STAGE);
#pragma unroll
    for (int i = 0; i < NAT; ++i) {
        if (A_TASKS % NT != 0 && f.ad[i] == ~0u) continue;
#pragma unroll
        for (int t = 0; t < T; ++t) {
            const u32 lo = r.a[i][t / 2], hi = r.a[i][(T + t) / 2];
            const u32 l16 = (t % 2) ? (lo >> 16) : (lo & 0xffffu);
            const u32 h16 = ((T + t) % 2) ? (hi & 0xffff0000u) : (hi << 16);
            SA[f.ad[i] + t * (BM * CS / 2)] = l16 | h16;
        }
    }
}

// One (channel group, tap column) pair: HK x MI kernel fragments stay while the wave's input rows pass by.
struct Place { const u16 *a, *p; };                           // where a pair's fragments begin
__device__ __forceinline__ Place place_of(const u16 *S, int arow, int aperm, int kc, int pix, int u)
{
    const int kk = KKS == 1 ? 0 : u / WK, s = u - kk * WK, c = kk * (KA / 8) + kc, p = pix + s;
    const Place at = {S + P_STAGE + arow + ((c ^ aperm) << 3) + s * (BM * CS), S + p * CS + ((c ^ swz(p)) << 3)};
    return at;
}
constexpr int ROWS = R + HK - 1, AHEAD = 2;
__device__ __forceinline__ frag_t row_frag(const Place &at, int y) { return __builtin_bit_cast(frag_t, *(const u32x4 *)(at.p + y * (PWP * CS))); }
__device__ __forceinline__ void load_frags(frag_t (&af)[HK][MI], frag_t (&bf)[AHEAD + 1], const Place &at)
{
#pragma unroll
    for (int y = 0; y < AHEAD && y < ROWS; ++y) bf[y] = row_frag(at, y);
#pragma unroll
    for (int r = 0; r < HK; ++r)
#pragma unroll
        for (int i = 0; i < MI; ++i) af[r][i] = __builtin_bit_cast(frag_t, *(const u32x4 *)(at.a + (r * WK * BM + i * ATOM) * CS));
}
__device__ __forceinline__ void compute_slab(acc_t (&acc)[MI][R], const u16 *S, int arow, int aperm, int kc, int pix, int wk)
{
    // the next pair's first fragments are read during this pair's last rows (two sets of kernel fragments)
    constexpr int NU = UNITS / KW;
    frag_t af[2][HK][MI], bf[2][AHEAD + 1];
    Place at = place_of(S, arow, aperm, kc, pix, wk);
    load_frags(af[0], bf[0], at);
#pragma unroll
    for (int j = 0; j < NU; ++j) {
        const int h = j & 1;
        const Place next = place_of(S, arow, aperm, kc, pix, wk + (j + 1) * KW);
#pragma unroll
        for (int y = 0; y < ROWS; ++y) {
            if (y + AHEAD < ROWS) bf[h][(y + AHEAD) % (AHEAD + 1)] = row_frag(at, y + AHEAD);
            if (y == (ROWS > 3 ? ROWS - 3 : 0) && j + 1 < NU) load_frags(af[h ^ 1], bf[h ^ 1], next);
#pragma unroll
            for (int r = 0; r < HK; ++r) {
                if (y - r < 0 || y - r >= R) continue;
#pragma unroll
                for (int i = 0; i < MI; ++i) acc[i][y - r] = MFMA(af[h][r][i], bf[h][y % (AHEAD + 1)], acc[i][y - r]);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
        at = next;
    }
}

extern "C" __global__ __launch_bounds__(NT, MINW)
void KERNEL_NAME(const u16 *__restrict__ A, const u16 *__restrict__ B, float *__restrict__ C,
                  unsigned long long *ctl /* unused: members of this template are never folded */)
{
    extern __shared__ __attribute__((aligned(16))) u16 smem[];
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int lrow = lane % ATOM, kc = lane / ATOM;
    const BlockId bid = block_id();
    const ColBlock cb = col_block(bid.n);
    const int wk = __builtin_amdgcn_readfirstlane(wave / (WM * WN));
    const int wmn = wave % (WM * WN), wm = wmn / WN, wn = wmn % WN;
    const int img = wn / (SPR * RG), strip = wn / RG % SPR, rg = wn % RG;
    const int m0 = bid.m * BM;

    Fill fill;
    plan_fill(fill, cb, m0, tid);
    PRegs pr;
    ARegs ar;
    {   // zeros: the fill never writes what lies outside the image
        const u32x4 zero = {0u, 0u, 0u, 0u};
        for (int i = tid; i < P_STAGE / 8; i += NT) ((u32x4 *)smem)[i] = zero;
    }
    const int xl = strip * ATOM + lrow, x = xl < BW ? xl : BW - 1;   // columns past the box read its last pixel and are not stored
    const int pix = (img * PH + rg * R) * PWP + x;
    const int arow = (wm * MI * ATOM + lrow) * CS, aperm = swz(lrow);

    acc_t acc[MI][R];
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < R; ++j)
#pragma unroll
            for (int r = 0; r < NACC; ++r) acc[i][j][r] = 0.f;

#pragma unroll 1
    for (int s = 0; s < KSTEPS; ++s) {
        load_p(pr, fill, B, s);
        if (TOGETHER) load_a(ar, fill, A, s);
        __syncthreads();
        store_p(pr, fill, smem);
        if (!TOGETHER) load_a(ar, fill, A, s);
        store_a(ar, fill, smem);
        __syncthreads();
        compute_slab(acc, smem, arow, aperm, kc, pix, wk);
    }

#if KW == 1
    if (xl < BW) {
        float *c = C + (((long)(cb.nb0 + img) * M + m0 + wm * MI * ATOM) * HOUT + cb.y0 + rg * R) * WOUT + cb.x0 + xl;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int r = 0; r < NACC; ++r) {
                const int row = i * ATOM + (ATOM == 32 ? 8 * (r / 4) + 4 * (lane / 32) + r % 4 : 4 * (lane / 16) + r);
#pragma unroll
                for (int j = 0; j < R; ++j) c[(long)row * (HOUT * WOUT) + j * WOUT] = acc[i][j][r];
            }
    }
#else
    // The KW partial sums, in passes of APP atoms: every wave writes its accumulators to RED[atom][wave][4 registers][lane]; wave k of a tile adds
    // and stores atoms k, k + KW, ... of the pass, always in the order of the waves.
    constexpr int ATOMS = MI * R, Q = NACC / 4;
    constexpr int APP_FIT = LDS_BYTES / (NWAVES * Q * 1024);
    constexpr int APP = APP_FIT < ATOMS ? APP_FIT : ATOMS;
    static_assert(APP >= 1, "the LDS cannot hold one atom of every wave");
    f32x4 *RED = (f32x4 *)smem;
#pragma unroll
    for (int a0 = 0; a0 < ATOMS; a0 += APP) {
        __syncthreads();
#pragma unroll
        for (int a = a0; a < a0 + APP && a < ATOMS; ++a)
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                const acc_t &v = acc[a / R][a % R];
                const f32x4 w = {v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
                RED[(((a - a0) * NWAVES + wave) * Q + q) * 64 + lane] = w;
            }
        __syncthreads();
#pragma unroll 1
        for (int a = a0 + wk; a < a0 + APP && a < ATOMS; a += KW) {
            const int i = a / R, j = a % R;
            float *c = C + (((long)(cb.nb0 + img) * M + m0 + (wm * MI + i) * ATOM) * HOUT + cb.y0 + rg * R + j) * WOUT + cb.x0 + xl;
#pragma unroll
            for (int q = 0; q < Q; ++q) {
                f32x4 sum = RED[(((a - a0) * NWAVES + wmn) * Q + q) * 64 + lane];
#pragma unroll
                for (int k = 1; k < KW; ++k) {
                    const f32x4 v = RED[(((a - a0) * NWAVES + k * (WM * WN) + wmn) * Q + q) * 64 + lane];
                    sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
                }
                if (xl < BW) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) {
                        const int r = 4 * q + e;
                        const int row = ATOM == 32 ? 8 * (r / 4) + 4 * (lane / 32) + r % 4 : 4 * (lane / 16) + r;
                        c[(long)row * (HOUT * WOUT)] = sum[e];
                    }
                }
            }
        }
    }
#endif
}
