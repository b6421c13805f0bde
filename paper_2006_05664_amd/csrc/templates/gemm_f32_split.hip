// fp32 MatMul / BatchMatMul on the bf16 matrix pipes, for long reductions in workgroup tiles of 32 or 64 rows and columns.
//
// Every fp32 value is taken apart into three bf16 values, each the rest rounded to nearest, that add up to it exactly (3 x 8 bits; magnitudes from 2^-100
// on; G. Henry, P. T. P. Tang, A. Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For Higher-Precision Computations", ARITH 2019).
// Of the nine products of two such triples all but the smallest, at most 2^-36 of the whole, are multiplied on 32x32x16 bf16 atoms.  The product of the
// upper parts, exact in fp32, has an accumulator of its own, the seven others (2^-7 of it and less) share one, and the two are added when the waves' sums have met.  A
// bf16 atom whose product is larger than its accumulator cuts the accumulator off at the product's last bit, so that in one
// accumulator a sum of a single product was wrong in the last place in one case of five (norm of the errors 3.4e-8); so it is rounded once,
// as by fp32 arithmetic (normal operands: largest error 5.97e-8, norm 2.54e-8; fp32 atoms 5.95e-8, 2.53e-8), and long sums are rounded once instead of eight
// times for 16 products: against 64 bits, K = 1024 5.7e-7 -> 1.0e-7, 4096 1.1e-6 -> 1.4e-7 (four or eight partial sums; smaller for each of 38 drawn operators).  Sums of 2 - 64
// normal products 0.34 - 0.87 times the fp32 atoms' error; of 2 - 16 products whose magnitudes lie up to 2^48 apart, where that cut falls on the upper parts' sum, 0.4 - 1.2 times.
// Values below 2^-100, sums below 2^-110 (whose smaller parts would be subnormal), infinities, NaN and sums beyond the range take the fp32 atoms (EXACT).
//
// KW waves share a tile: each takes a contiguous part of the reduction with the whole tile as its wave tile, and the sums meet in LDS at the end.  So
// a value is taken apart once per workgroup, no wave waits for another inside the loop, and a workgroup keeps all four SIMDs busy whatever its tile.
//   * B [K][N] (and a first operand stored [K][M]): a lane loads its 8 k rows' values straight into the registers the matrix units take them from, with NI = 2
//     two neighbouring columns at a time (column 2l + j belongs to atom j).
//   * A [M][K]: 16-byte pieces, whole cache lines, loaded straight into a part of the LDS that is the wave's own (two chunks of 32 reduction steps, no
//     barrier), pieces permuted within their row so that the 16 lanes of a turn of a fragment read fall on 16 groups of banks.  Through
//     registers a 64 x 64 tile needs 300 of them: one wave on a SIMD, 512 x 4096 x 1024 44 us; so, and with a fragment read when its turn comes, 251.
//   * While a step's MFMAs run, the next step's values are taken apart between them, and the step after that is on its way.
// What bounds it: instruction issue (15 vector instructions per two values, 7.5 beside every MFMA of a 64 x 64 tile) about as much as the pipes, and on
// the whole chip the pipes' power.  Times on this card, fp32 atoms -> here: 512 x 4096 x 1024 in 64 x 64 tiles 40.1 -> 37.7 us; 2336 x 3200 x 1088
// in 32 x 32 230 -> 178; few workgroups: 64 x 1152 x 4096 (18) 80 -> 48, 672 x 192 x 2560 (126) 53 -> 16.2, 224 x 512 x 896 (56) 20 -> 12.7.
typedef __attribute__((ext_vector_type(8))) __bf16 frag_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef f32x16 acc_t;

constexpr int MI = BM / 32, NI = BN / 32;
constexpr int KC = 32;                              // reduction steps of a chunk: two MFMA steps
constexpr int NCHUNK = K / KC;
static_assert(BM % 32 == 0 && BN % 32 == 0 && K % KC == 0 && MI <= 2 && NI <= 2 && NT == 64 * KW && KW > 1 && KW <= NCHUNK && 8 % KW == 0, "decoder and template disagree");
constexpr int A_WAVE = A_TRANS ? 0 : 2 * BM * KC;   // floats of LDS that are a wave's own
constexpr int RED = KW * BM * BN;                   // floats of the partial sums, in the same place
static_assert(4 * (KW * A_WAVE > RED ? KW * A_WAVE : RED) == LDS_BYTES, "decoder and template disagree");
constexpr u32 SMALL = 2u * (27u << 23) - 1;         // 2^-100 (see magnitude)
constexpr u32 SMALL_SUM = 2u * (17u << 23) - 1;     // 2^-110
constexpr u32 NOT_FINITE = 2u * (255u << 23) - 1;   // infinity

// base (in scalar registers, and left there) + a lane's byte offset
#define GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ T load_at(const float *base, u32 off)
{
    const GLOBAL char *p = (const GLOBAL char *)base;
    asm("" : "+s"(p), "+v"(off));                    // (the offset as well: widened outside the loop, it would be added to the base by a vector instruction each time)
    return *(const GLOBAL T *)(p + off);
}
// a lane's NV neighbouring values of a row
template <int NV> struct Vals { float v[NV]; };
template <int NV>
__device__ __forceinline__ Vals<NV> load_vals(const float *base, u32 off)
{
    Vals<NV> r;
    if constexpr (NV == 2) { const f32x2 t = load_at<f32x2>(base, off); r.v[0] = t.x; r.v[1] = t.y; }
    else r.v[0] = load_at<float>(base, off);
    return r;
}
// operand of k rows: the values of one MFMA step, k = 8 * (lane / 32) + j
template <int NV> struct KRows { Vals<NV> k[8]; };
template <int NV, int LEN>
__device__ __forceinline__ void load_krows(KRows<NV> &r, const float *base, u32 off)
{
#pragma unroll
    for (int j = 0; j < 8; ++j) r.k[j] = load_vals<NV>(base + (long)j * LEN, off);
}

struct Planes { u32x4 h, m, l; };                   // 8 values of a lane: bf16 pairs of their upper, middle and lower parts
__device__ __forceinline__ u32 pack(float a, float b)
{
    const f32x2 v = {a, b};
    return __builtin_bit_cast(u32, __builtin_convertvector(v, bf16x2));
}
__device__ __forceinline__ float lower(u32 v) { return __builtin_bit_cast(float, v << 16); }
__device__ __forceinline__ float upper(u32 v) { return __builtin_bit_cast(float, v & 0xffff0000u); }
// Word i of the planes: values 2i and 2i + 1.  low: the smallest of twice the values' bits - 1, without the sign, where a zero counts as the largest
// (the values' own bits: what is at most 2^-134 has upper parts of zero all the same).
// (The statement that does nothing keeps the values from being taken apart before their turn.)
__device__ __forceinline__ u32 magnitude(float v) { return (__builtin_bit_cast(u32, v) << 1) - 1; }
__device__ __forceinline__ void split(Planes &p, int i, float a, float b, u32 &low)
{
    asm volatile("" : "+v"(a), "+v"(b));
    low = min(min(magnitude(a), magnitude(b)), low);
    const u32 h = pack(a, b);
    a -= lower(h); b -= upper(h);
    const u32 m = pack(a, b);
    a -= lower(m); b -= upper(m);
    p.h[i] = h; p.m[i] = m; p.l[i] = pack(a, b);
}

struct Lane {
    const float *a, *b;                             // the operands' tiles (the same for all lanes), and this lane's byte offset in a chunk
    u32 a_off, b_off;
    const float *lds;                               // (A stored [M][K]) this wave's part of the LDS, and its byte address
    u32 lds_at;
    int lane;
};
#if A_TRANS
struct ARegs { KRows<MI> t[2]; };
__device__ __forceinline__ void load_a(ARegs &r, const Lane &l, int c, int t) { load_krows<MI, M>(r.t[t], l.a + ((long)c * KC + t * 16) * M, l.a_off); }
__device__ __forceinline__ void fetch_a(const ARegs &r, const Lane &, int, int t, int i, float (&x)[8])
{
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = r.t[t].k[j].v[i];
}
#else
// 16-byte pieces, 8 to a row of a chunk, straight into the LDS: lane l's come from row l / 8, l / 8 + 8, ... and go to place l % 8 of it.  Chunk c has half c % 2
// of the wave's part.  The compiler does not see these loads, nor does it wait for them: every wait that they need is a wait_loads.  (M0 needs a
// wait state before the load, and the base a scalar copy, so that it is never read too early after a vector instruction wrote it.)
struct ARegs {};
constexpr int PIECES = BM / 8;                      // loads of a chunk
__device__ __forceinline__ void load_a(const Lane &l, int c, int at)
{
    const float *from = l.a + (long)c * KC;
    const u32 to = l.lds_at + (u32)(at & 1) * (4 * BM * KC);
#pragma unroll
    for (int i = 0; i < PIECES; ++i) {
        const float *copy;
        asm volatile("s_mov_b32 m0, %3\n\ts_mov_b64 %0, %2\n\tglobal_load_lds_dwordx4 %1, %0"
                     : "=&s"(copy) : "v"(i & 1 ? l.a_off ^ 64 : l.a_off), "s"(from + (long)i * 8 * K), "s"(to + i * 1024) : "memory", "m0");
    }
}
template <int LEFT> __device__ __forceinline__ void wait_loads() { asm volatile("s_waitcnt vmcnt(%0)" : : "n"(LEFT) : "memory"); }
__device__ __forceinline__ void fetch_a(const ARegs &, const Lane &l, int c, int t, int i, float (&x)[8])
{
    const f32x4 *const from = (const f32x4 *)(l.lds + (c & 1) * (BM * KC));
    const int row = i * 32 + l.lane % 32, p = 4 * t + 2 * (l.lane / 32), key = row >> 1 & 7;
    const f32x4 u = from[row * 8 + (p ^ key)], v = from[row * 8 + (p + 1 ^ key)];
#pragma unroll
    for (int j = 0; j < 4; ++j) { x[j] = u[j]; x[4 + j] = v[j]; }
}
#endif

__device__ __forceinline__ void clear(acc_t (&acc)[MI][NI])
{
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
}

// A wave's part of the reduction, chunks c0 .. c1 - 1: the sums of the products of upper parts, and of the others.  EXACT: on the fp32 matrix pipes, in acc; with
// only >= 0 that atom of the tile alone, i * NI + j.  Returns what the values' smallest magnitude is judged by.
template <bool EXACT>
__device__ __forceinline__ u32 reduce(acc_t (&hi)[MI][NI], acc_t (&acc)[MI][NI], const Lane &l, int c0, int c1, int only = -1)
{
    clear(acc);
    u32 low = ~0u;
    ARegs a;
    KRows<NI> b[2];
    auto load_b = [&](int c, int t) { load_krows<NI, N>(b[t], l.b + ((long)c * KC + t * 16) * N, l.b_off); };
    auto within = [&](int c) { return c < c1 ? c : c1 - 1; };      // past the last chunk the last one is loaded again
#pragma unroll
    for (int t = 0; t < 2; ++t) {
#if A_TRANS
        load_a(a, l, c0, t);
#else
        load_a(l, within(c0 + t), c0 + t);
#endif
        load_b(c0, t);
    }
#if !A_TRANS
    wait_loads<0>();
#endif
    // (a loop-carried value that is a load on every way in becomes a load at its use: the next chunk would be fetched when it is needed)
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int k = 0; k < 8; ++k) {
#pragma unroll
            for (int j = 0; j < NI; ++j) asm volatile("" : "+v"(b[t].k[k].v[j]));
#if A_TRANS
#pragma unroll
            for (int i = 0; i < MI; ++i) asm volatile("" : "+v"(a.t[t].k[k].v[i]));
#endif
        }
    if constexpr (EXACT) {
#pragma unroll 1
        for (int c = c0; c < c1; ++c) {
            const int cn = within(c + 1);
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                float x[MI][8];
#if !A_TRANS
                if (t == 0) wait_loads<PIECES>();       // all but the chunk after this one, the youngest loads
#endif
#pragma unroll
                for (int i = 0; i < MI; ++i) fetch_a(a, l, c, t, i, x[i]);
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j) {
                        if (only >= 0 && only != i * NI + j) continue;
#pragma unroll
                        for (int k = 0; k < 8; ++k) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i][k], b[t].k[k].v[j], acc[i][j], 0, 0, 0);
                    }
                load_b(cn, t);
#if A_TRANS
                load_a(a, l, cn, t);
#else
                __builtin_amdgcn_sched_barrier(0);      // (chunk c's fragments have been read)
                if (t == 1) load_a(l, within(c + 2), c);
#endif
            }
        }
#if !A_TRANS
        wait_loads<0>();                                // nothing is on its way to the LDS any longer
#endif
        clear(hi);
        return low;
    }
    Planes pa[2][MI], pb[2][NI];
    // words [w0, w1) of the (MI + NI) * 4 of step t, the second operand's first
    auto split_words = [&](int t, int w0, int w1, const float (&x)[MI][8]) {
#pragma unroll
        for (int w = 0; w < 4 * (MI + NI); ++w) {
            if (w < w0 || w >= w1) continue;
            const int at = w / 4, i = w % 4;
            if (at < NI) split(pb[t][at], i, b[t].k[2 * i].v[at], b[t].k[2 * i + 1].v[at], low);
            else split(pa[t][at - NI], i, x[at - NI][2 * i], x[at - NI][2 * i + 1], low);
        }
    };
    // MFMAs of a step; after which of them the second operand's values are no longer waited for, and where the first operand's first fragment is read
    constexpr int WORDS = 4 * (MI + NI), MFMAS = 8 * MI * NI, LOAD_AT = 4 * MFMAS / WORDS, EARLY = 4;
    constexpr auto fetch_at = [](int i) { return MFMAS * (NI + i) / (NI + MI) - EARLY; };
    clear(hi);
    {
        float x[MI][8];
#pragma unroll
        for (int i = 0; i < MI; ++i) fetch_a(a, l, c0, 0, i, x[i]);
        split_words(0, 0, WORDS, x);
        load_b(within(c0 + 1), 0);
#if A_TRANS
        load_a(a, l, within(c0 + 1), 0);
#endif
    }
#pragma unroll 1
    for (int c = c0; c < c1; ++c) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            // multiply step t of chunk c, take the next step's values apart meanwhile
            const int o = t ^ 1, cn = within(c + 1 + t);
            float x[MI][8];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < 8; ++q)
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j) {
                        const u32x4 &u = q == 1 || q == 2 ? pa[t][i].l : q == 0 || q == 4 || q == 5 ? pa[t][i].m : pa[t][i].h;
                        const u32x4 &v = q == 0 || q == 3 ? pb[t][j].l : q == 1 || q == 4 || q == 6 ? pb[t][j].m : pb[t][j].h;
                        acc_t &to = q == 7 ? hi[i][j] : acc[i][j];
                        to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(frag_t, u), __builtin_bit_cast(frag_t, v), to, 0, 0, 0);
                        const int n = (q * MI + i) * NI + j;
#if !A_TRANS
                        // Chunk c was read from for the last time in step 0.  The loads younger than chunk c + 1's, issued in step 1 of chunk c - 1: the second
                        // operand's 8 at the end of that step and 8 at the end of step 0, and those issued here
                        if (t == 1 && n == LOAD_AT) load_a(l, within(c + 2), c);
                        if (t == 1 && n == fetch_at(0)) wait_loads<8 + (fetch_at(0) >= LOAD_AT ? PIECES : 0)>();
#endif
#pragma unroll
                        for (int f = 0; f < MI; ++f)
                            if (n == fetch_at(f)) fetch_a(a, l, c + t, o, f, x[f]);
                        split_words(o, n * WORDS / MFMAS, (n + 1) * WORDS / MFMAS, x);
                        __builtin_amdgcn_sched_barrier(0);
                    }
            load_b(cn, o);
#if A_TRANS
            load_a(a, l, cn, o);
#endif
        }
    }
#if !A_TRANS
    wait_loads<0>();                                    // nothing is on its way to the LDS any longer
#endif
    return low;
}

extern "C" __global__ __launch_bounds__(NT, MINW)
void KERNEL_NAME(const float *__restrict__ A, const float *__restrict__ B, float *__restrict__ C,
                 unsigned long long *ctl /* unused: members of this template are never folded */)
{
    extern __shared__ __attribute__((aligned(16))) float smem_f32[];
    __shared__ int beyond[KW];                      // which waves' sums are not finite
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int l32 = lane & 31, half = lane >> 5;
    const BlockId bid = block_id();
    const int m0 = bid.m * BM, n0 = bid.n * BN;
    const int c0 = NCHUNK * wave / KW, c1 = NCHUNK * (wave + 1) / KW;
    for (int bi = 0; bi < BATCH_INNER; ++bi) {
        const long batch = (long)bid.b * BATCH_INNER + bi;
        const float *Ab = A + batch * M * K, *Bb = B + batch * K * N;
        float *Cb = C + batch * M * N;
        Lane l;
        l.lane = lane;
        l.lds = smem_f32 + wave * A_WAVE;
        l.lds_at = __builtin_amdgcn_readfirstlane((u32)(unsigned long)(__attribute__((address_space(3))) float *)(smem_f32 + wave * A_WAVE));
#if A_TRANS
        l.a = Ab + m0;
        l.a_off = 4u * (u32)(8 * half * M + l32 * MI);
#else
        l.a = Ab + (long)m0 * K;
        l.a_off = 4u * (u32)(lane / 8 * K + (lane % 8 ^ lane >> 4) * 4);      // (rows 8, 24, ... further on: ^ 64)
#endif
        l.b = Bb + n0;
        l.b_off = 4u * (u32)(8 * half * N + l32 * NI);
        if (bi > 0) __syncthreads();
        acc_t hi[MI][NI], acc[MI][NI];
        const u32 low = reduce<false>(hi, acc, l, c0, c1);
        // Sums that are not finite, or too small for their products' parts.  As bits less 2^-110's ordinary ones come first, then what is not finite, zeros, and
        // what is smaller than 2^-110; only if there is any but the first is it told apart.
        auto each = [&](auto f) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j)
#pragma unroll
                    for (int r = 0; r < 16; ++r) f(hi[i][j][r] + acc[i][j][r]);
        };
        u32 last = 0;
        each([&](float v) { last = max(magnitude(v) - SMALL_SUM, last); });
        bool finite = true, small_sum = false;
        if (__any(last >= NOT_FINITE - SMALL_SUM)) {
            // (the sums are added up once more here: kept, they would be 64 registers too many)
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) asm volatile("" : "+v"(hi[i][j]));
            each([&](float v) {
                finite = finite && __builtin_isfinite(v);
                small_sum = small_sum || magnitude(v) < SMALL_SUM;
            });
        }
        // A part with values too small to be taken apart, or sums too small for their products' parts, is added up again on the fp32 atoms.  Where a sum is not
        // finite, the tile's whole reduction is, in one chain for each atom of it, an atom a wave: partial sums of either sign beyond the range would make a NaN of
        // what is infinite in order.  What that costs, 512 x 4096 x 1024 in 64 x 64 tiles / 672 x 192 x 2560 in 32 x 32 (ordinary values 38 / 16 us, also with zeros; on the
        // fp32 atoms alone 39 / 53 whatever the values): one value of 1e-40 50 / 24, one of 1e-32 in every row 67 / 24, every value or sum too small 71 / 29; one
        // infinity or NaN 58 / 79, one in every row 82 / 80 (one wave for the whole tile: 93 - 127 / 71).
        const bool small = __any(low < SMALL || small_sum), mine = __any(!finite);
        if (lane == 0) beyond[wave] = mine;
        __syncthreads();                            // (also: the waves' parts of the LDS have been read)
        bool chain = false;
#pragma unroll
        for (int k = 0; k < KW; ++k) chain |= beyond[k] != 0;
        chain = __builtin_amdgcn_readfirstlane(chain);
        if (chain ? wave < MI * NI : small) reduce<true>(hi, acc, l, chain ? 0 : c0, chain ? NCHUNK : c1, chain ? wave : -1);

        auto row_of = [&](int i, int r) {
            const int row = 8 * (r / 4) + 4 * half + r % 4;
            return A_TRANS ? row * MI + i : i * 32 + row;
        };
        float *const out = Cb + (long)m0 * N + n0 + l32 * NI;
        if (chain) {
#pragma unroll
            for (int i = 0; i < MI; ++i)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    if (wave != i * NI + j) continue;
#pragma unroll
                    for (int r = 0; r < 16; ++r) out[(long)row_of(i, r) * N + j] = acc[i][j][r];
                }
            continue;
        }
        // The waves' sums meet in the LDS, those of the upper parts' products first, then the others.  With the two added up in every wave, which spares 0.3 - 0.9 us, each
        // wave rounded its products before the sum did: sums of two to four normal products had 1.01 - 1.16 times the fp32 atoms' error, now 0.65 - 0.87 times.
        // (A lane's accumulators of consecutive rows go through the LDS together, 16 bytes at a time, so that none is moved to another register first.)
        constexpr int W = MI * 16 / KW < 4 ? 2 : 4, GROUPS = MI * 16 / W, SHARE = GROUPS / KW;      // rows of a group; groups of the tile, and a wave's share
        typedef __attribute__((ext_vector_type(W))) float rows_t;
        rows_t *const red = (rows_t *)smem_f32;
        rows_t sum[SHARE][NI];
        auto meet = [&](const acc_t (&part)[MI][NI], auto f) {
            __syncthreads();                        // nobody reads operands, or the other sums, from the LDS any longer
#pragma unroll
            for (int t = 0; t < GROUPS; ++t)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    rows_t v;
#pragma unroll
                    for (int w = 0; w < W; ++w) v[w] = part[t * W / 16][j][t * W % 16 + w];
                    red[((wave * GROUPS + t) * NI + j) * 64 + lane] = v;
                }
            __syncthreads();
#pragma unroll
            for (int s = 0; s < SHARE; ++s)
#pragma unroll
                for (int j = 0; j < NI; ++j) {
                    const rows_t *const from = red + ((wave + s * KW) * NI + j) * 64 + lane;
                    rows_t all = from[0];
#pragma unroll
                    for (int k = 1; k < KW; ++k) all += from[k * GROUPS * NI * 64];
                    f(sum[s][j], all);
                }
        };
        meet(hi, [](rows_t &to, const rows_t &all) { to = all; });
        meet(acc, [](rows_t &to, const rows_t &all) { to += all; });
#pragma unroll
        for (int s = 0; s < SHARE; ++s)
#pragma unroll
            for (int w = 0; w < W; ++w) {
                const int r = (wave + s * KW) * W + w;
#pragma unroll
                for (int j = 0; j < NI; ++j) out[(long)row_of(r / 16, r % 16) * N + j] = sum[s][j][w];
            }
    }
}
