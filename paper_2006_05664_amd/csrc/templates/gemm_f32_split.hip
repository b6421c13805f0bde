// fp32 MatMul / BatchMatMul on the bf16 matrix pipes, for long reductions in workgroup tiles of 32 or 64 rows and columns.
//
// Every fp32 value is taken apart into three bf16 values, each the rest rounded to nearest, that add up to it exactly (3 x 8 bits; magnitudes from 2^-100 on).
// Of the nine products of two such triples the six above 2^-24 are multiplied on 32x32x16 bf16 atoms and added in fp32, smallest first: what is left out
// is at most 2^-26 of a product, of either sign, and an accumulator is rounded six times for 16 products instead of eight times on 32x32x2 fp32 atoms.
// Against 64 bits, normal operands, the error falls to 0.3 - 0.6 of the fp32 atoms' (K = 1024 5.7e-7 -> 2.4e-7, 4096 1.1e-6 -> 3.5e-7, four or eight partial sums; it
// was smaller for each of 60 drawn operators).  Values below 2^-100, infinities, NaN and sums beyond the range take the fp32 atoms (EXACT).
//
// KW waves share a tile: each takes a contiguous part of the reduction with the whole tile as its wave tile, and the sums meet in LDS at the end.  So
// a value is taken apart once per workgroup, no wave waits for another inside the loop, and a workgroup keeps all four SIMDs busy whatever its tile.
//   * B [K][N] (and a first operand stored [K][M]): a lane loads its 8 k rows' values straight into the registers the matrix units take them from, with NI = 2
//     two neighbouring columns at a time (column 2l + j belongs to atom j).
//   * A [M][K]: 16-byte pieces, whole cache lines, through a part of the LDS that is the wave's own (32 reduction steps, no barrier), pieces
//     permuted within their row so that the 16 lanes of a turn of a fragment read fall on 16 groups of banks.
//   * While a step's MFMAs run, the next step's values are taken apart between them, and the step after that is on its way.
// What bounds it: instruction issue (15 vector instructions per two values; 10 beside every MFMA of a 64 x 64 tile, 95 cycles for what 64 cycles of the
// pipes need) and, on the whole chip, the pipes' power.  Times on this card, fp32 atoms -> here: 512 x 4096 x 1024 in 64 x 64 tiles 46.0 -> 40.6 us; 2336 x 3200 x 1088
// in 32 x 64 240 -> 179; few workgroups: 64 x 1152 x 4096 (18) 80 -> 46, 672 x 192 x 2560 (63) 53 -> 22, 224 x 512 x 896 (56) 20 -> 11.4.
typedef __attribute__((ext_vector_type(8))) __bf16 frag_t;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(2))) float f32x2;
typedef f32x16 acc_t;
#ifndef NT_OUT
#define NT_OUT 0
#endif

constexpr int MI = BM / 32, NI = BN / 32;
constexpr int KC = 32;                              // reduction steps of a chunk: two MFMA steps
constexpr int NCHUNK = K / KC;
static_assert(BM % 32 == 0 && BN % 32 == 0 && K % KC == 0 && MI <= 2 && NI <= 2 && NT == 64 * KW && KW > 1 && KW <= NCHUNK, "decoder and template disagree");
constexpr int A_WAVE = A_TRANS ? 0 : BM * KC;       // floats of LDS that are a wave's own
constexpr int RED = KW * BM * BN;                   // floats of the partial sums, in the same place
static_assert(4 * (KW * A_WAVE > RED ? KW * A_WAVE : RED) == LDS_BYTES, "decoder and template disagree");
constexpr u32 SMALL = 2u * (27u << 23) - 1;         // 2^-100 (see magnitude)

// base (in scalar registers, and left there) + a lane's byte offset
#define GLOBAL __attribute__((address_space(1)))
template <typename T>
__device__ __forceinline__ T load_at(const float *base, u32 off)
{
    const GLOBAL char *p = (const GLOBAL char *)base;
    asm("" : "+s"(p));
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
    float *lds;                                     // (A stored [M][K]) this wave's part of the LDS
    int lane;
};
#if A_TRANS
struct ARegs { KRows<MI> t[2]; };
__device__ __forceinline__ void load_a(ARegs &r, const Lane &l, int c, int t) { load_krows<MI, M>(r.t[t], l.a + ((long)c * KC + t * 16) * M, l.a_off); }
__device__ __forceinline__ void fetch_a(const ARegs &r, const Lane &, int t, int i, float (&x)[8])
{
#pragma unroll
    for (int j = 0; j < 8; ++j) x[j] = r.t[t].k[j].v[i];
}
#else
// 16-byte pieces, 8 to a row of a chunk: lane l has piece l % 8 of rows l / 8, l / 8 + 8, ...
struct ARegs { f32x4 v[BM / 8]; };
__device__ __forceinline__ void load_a(ARegs &r, const Lane &l, int c)
{
#pragma unroll
    for (int i = 0; i < BM / 8; ++i) r.v[i] = load_at<f32x4>(l.a + (long)c * KC + (long)i * 8 * K, l.a_off);
}
__device__ __forceinline__ void store_a(const ARegs &r, const Lane &l)
{
#pragma unroll
    for (int i = 0; i < BM / 8; ++i) {
        const int row = l.lane / 8 + i * 8;
        ((f32x4 *)l.lds)[row * 8 + (l.lane % 8 ^ (row >> 1 & 7))] = r.v[i];
    }
}
__device__ __forceinline__ void fetch_a(const ARegs &, const Lane &l, int t, int i, float (&x)[8])
{
    const int row = i * 32 + l.lane % 32, p = 4 * t + 2 * (l.lane / 32), key = row >> 1 & 7;
    const f32x4 u = ((const f32x4 *)l.lds)[row * 8 + (p ^ key)], v = ((const f32x4 *)l.lds)[row * 8 + (p + 1 ^ key)];
#pragma unroll
    for (int j = 0; j < 4; ++j) { x[j] = u[j]; x[4 + j] = v[j]; }
}
#endif

// A wave's part of the reduction, chunks c0 .. c1 - 1.  EXACT: on the fp32 matrix pipes.  Returns what the values' smallest magnitude is judged by.
template <bool EXACT>
__device__ __forceinline__ u32 reduce(acc_t (&acc)[MI][NI], const Lane &l, int c0, int c1)
{
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < NI; ++j)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[i][j][r] = 0.f;
    u32 low = ~0u;
    ARegs a;
    KRows<NI> b[2];
    auto load_b = [&](int c, int t) { load_krows<NI, N>(b[t], l.b + ((long)c * KC + t * 16) * N, l.b_off); };
#if A_TRANS
    auto load_a_at = [&](int c, int t) { load_a(a, l, c, t); };
#else
    auto load_a_at = [&](int c, int t) { if (t == 0) load_a(a, l, c); };
#endif
#pragma unroll
    for (int t = 0; t < 2; ++t) { load_a_at(c0, t); load_b(c0, t); }
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
#if !A_TRANS
#pragma unroll
    for (int i = 0; i < BM / 8; ++i) asm volatile("" : "+v"(a.v[i]));
#endif
    if constexpr (EXACT) {
#pragma unroll 1
        for (int c = c0; c < c1; ++c) {
            const int cn = c + 1 < c1 ? c + 1 : c;
#if !A_TRANS
            store_a(a, l);
            load_a_at(cn, 0);
#endif
#pragma unroll
            for (int t = 0; t < 2; ++t) {
                float x[MI][8];
#pragma unroll
                for (int i = 0; i < MI; ++i) fetch_a(a, l, t, i, x[i]);
#pragma unroll
                for (int k = 0; k < 8; ++k)
#pragma unroll
                    for (int i = 0; i < MI; ++i)
#pragma unroll
                        for (int j = 0; j < NI; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(x[i][k], b[t].k[k].v[j], acc[i][j], 0, 0, 0);
                load_b(cn, t);
#if A_TRANS
                load_a_at(cn, t);
#endif
            }
        }
        return low;
    }
    Planes pa[2][MI], pb[2][NI];
    // words [w0, w1) of the (MI + NI) * 4 of step t
    auto split_words = [&](int t, int w0, int w1, const float (&x)[MI][8]) {
#pragma unroll
        for (int w = 0; w < 4 * (MI + NI); ++w) {
            if (w < w0 || w >= w1) continue;
            const int at = w / 4, i = w % 4;
            if (at < NI) split(pb[t][at], i, b[t].k[2 * i].v[at], b[t].k[2 * i + 1].v[at], low);
            else split(pa[t][at - NI], i, x[at - NI][2 * i], x[at - NI][2 * i + 1], low);
        }
    };
    constexpr int WORDS = 4 * (MI + NI), MFMAS = 6 * MI * NI;
    {
        float x[MI][8];
#if !A_TRANS
        store_a(a, l);
        load_a_at(c0 + 1 < c1 ? c0 + 1 : c0, 0);
#endif
#pragma unroll
        for (int i = 0; i < MI; ++i) fetch_a(a, l, 0, i, x[i]);
        split_words(0, 0, WORDS, x);
        load_b(c0 + 1 < c1 ? c0 + 1 : c0, 0);
#if A_TRANS
        load_a_at(c0 + 1 < c1 ? c0 + 1 : c0, 0);
#endif
    }
#pragma unroll 1
    for (int c = c0; c < c1; ++c) {
#pragma unroll
        for (int t = 0; t < 2; ++t) {
            // multiply step t of chunk c, take the next step's values apart meanwhile
            const int o = t ^ 1, cn = c + 1 + t < c1 ? c + 1 + t : c1 - 1;
            float x[MI][8];
#if !A_TRANS
            if (t == 1) { store_a(a, l); load_a_at(cn, 0); }
#endif
#pragma unroll
            for (int i = 0; i < MI; ++i) fetch_a(a, l, o, i, x[i]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int j = 0; j < NI; ++j) {
                        const u32x4 &u = q == 0 ? pa[t][i].l : q == 2 || q == 3 ? pa[t][i].m : pa[t][i].h;
                        const u32x4 &v = q == 1 ? pb[t][j].l : q == 2 || q == 4 ? pb[t][j].m : pb[t][j].h;
                        acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(frag_t, u), __builtin_bit_cast(frag_t, v), acc[i][j], 0, 0, 0);
                        const int n = (q * MI + i) * NI + j;
                        split_words(o, n * WORDS / MFMAS, (n + 1) * WORDS / MFMAS, x);
                        __builtin_amdgcn_sched_barrier(0);
                    }
            load_b(cn, o);
#if A_TRANS
            load_a_at(cn, o);
#endif
        }
    }
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
#if A_TRANS
        l.a = Ab + m0;
        l.a_off = 4u * (u32)(8 * half * M + l32 * MI);
#else
        l.a = Ab + (long)m0 * K;
        l.a_off = 4u * (u32)(lane / 8 * K + lane % 8 * 4);
#endif
        l.b = Bb + n0;
        l.b_off = 4u * (u32)(8 * half * N + l32 * NI);
        if (bi > 0) __syncthreads();
        acc_t acc[MI][NI];
        const u32 low = reduce<false>(acc, l, c0, c1);
        float nan = 0.f;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < NI; ++j)
#pragma unroll
                for (int r = 0; r < 16; ++r) nan = __builtin_fmaf(acc[i][j][r], 0.f, nan);
        // A part with values too small to be taken apart is added up again on the fp32 atoms.  Where a sum is not finite, the first wave adds up the
        // whole reduction there, in one chain: partial sums of either sign beyond the range would make a NaN of what is infinite in order.
        const bool small = __any(low < SMALL), mine = __any(nan != 0.f);
        if (lane == 0) beyond[wave] = mine;
        __syncthreads();                            // (also: the waves' parts of the LDS have been read)
        bool chain = false;
#pragma unroll
        for (int k = 0; k < KW; ++k) chain |= beyond[k] != 0;
        chain = __builtin_amdgcn_readfirstlane(chain);
        if (chain ? wave == 0 : small) reduce<true>(acc, l, chain ? 0 : c0, chain ? NCHUNK : c1);

        auto row_of = [&](int i, int r) {
            const int row = 8 * (r / 4) + 4 * half + r % 4;
            return A_TRANS ? row * MI + i : i * 32 + row;
        };
        float *const out = Cb + (long)m0 * N + n0 + l32 * NI;
        if (chain) {
            if (wave == 0) {
#pragma unroll
                for (int i = 0; i < MI; ++i)
#pragma unroll
                    for (int r = 0; r < 16; ++r)
#pragma unroll
                        for (int j = 0; j < NI; ++j) out[(long)row_of(i, r) * N + j] = acc[i][j][r];
            }
            continue;
        }
        __syncthreads();                            // nobody reads operands from the LDS any longer
        Vals<NI> *const red = (Vals<NI> *)smem_f32;
#pragma unroll
        for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                Vals<NI> v;
#pragma unroll
                for (int j = 0; j < NI; ++j) v.v[j] = acc[i][j][r];
                red[((wave * MI + i) * 16 + r) * 64 + lane] = v;
            }
        __syncthreads();
#pragma unroll 2
        for (int t = wave; t < MI * 16; t += KW) {
            Vals<NI> sum = red[t * 64 + lane];
#pragma unroll
            for (int k = 1; k < KW; ++k) {
                const Vals<NI> v = red[(k * MI * 16 + t) * 64 + lane];
#pragma unroll
                for (int j = 0; j < NI; ++j) sum.v[j] += v.v[j];
            }
#pragma unroll
            for (int j = 0; j < NI; ++j) out[(long)row_of(t / 16, t % 16) * N + j] = sum.v[j];
        }
    }
}
