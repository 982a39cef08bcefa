// fp32 GEMM C[M][N] = A[M][K] B[K][N] on gfx950 with v_mfma_f32_16x16x4_f32
// (the fp32 contraction of the paper's App. A example module).
//
// Compile-time schedule (defined by the generated prologue):
//   TM TN TK     workgroup tile (TileSize)
//   WM WN        waves per workgroup along M and N (Parallel)
//   VEC          fp32 elements per global load (Vectorize)
//   STAGES       1: load-store-compute; 2: the next K tiles on their way while
//                one is computed (ComputeLocation): a ring of LDS buffers
//                filled by direct-to-LDS loads where the tile allows it
//                (RING below), else an LDS double buffer with register
//                prefetch of the next K tile; 3: streaming
//                for decode-shaped operators (M <= 16 rows, one MFMA row
//                block): no LDS staging, each wave streams its own slice of
//                the K range straight from memory into MFMA operands with
//                the loads of the next 2 x UNROLL - 1 batches of TK rows in
//                flight (Unroll sets the prefetch depth), the waves' partial sums
//                are added in LDS, and with SPLITS > 1 the workgroups of one
//                column tile split K further and rc_gemm_f32_splitk_reduce
//                adds their partials (in a fixed order)
//   SPLITS       K splits across workgroups (Parallel; STAGES 3 only)
//   UNROLL       unroll factor of the K-tile loop (Unroll)
//   LAYOUT       0: B stored [K][N]; 1: B stored [N][K] (Layout)
//   GM GN GK     problem size.  Stages 1 and 2 take any size: tiles that
//                cross the edge of M, N or K load zeros there and store only
//                inside C (VEC divides the row lengths, so a vector is wholly
//                inside or outside); a problem that every tile divides
//                compiles without the guards.  Stage 3 needs whole tiles.
//
// MFMA lane layout (16x16x4, one block): lane l supplies A[l % 16][l / 16]
// and B[l / 16][l % 16]; accumulator element r of lane l is
// C[4 * (l / 16) + r][l % 16].

#define NT (64 * WM * WN)
#define WTM (TM / WM)
#define WTN (TN / WN)
#define FM (WTM / 16)
#define FN (WTN / 16)
#define KTILES ((GK + TK - 1) / TK)
#define RAGGED ((GM % TM) != 0 || (GN % TN) != 0 || (GK % TK) != 0)
// Stages 2 runs as a ring of NST LDS buffers when the loads are 16-byte
// vectors, a K tile is whole 16-row MFMA blocks, its 1 KiB wave-loads split
// evenly over the waves and 32-bit buffer offsets reach both operands, K
// rounded up to whole tiles (offsets past the end of K are formed too, and
// their top bit marks them).
#define WLOADS ((TM * TK + TN * TK) / 256)
#define KUP (1ull * KTILES * TK)
#define RING (STAGES == 2 && VEC == 4 && TK >= 16 && WLOADS % (WM * WN) == 0 &&                       \
              4ull * GM * KUP < 0x80000000ull && 4ull * KUP * GN < 0x80000000ull)
#define A_LOADS ((TM * TK) / (VEC * NT))
#define B_LOADS ((TK * TN) / (VEC * NT))

typedef float f32x4 __attribute__((ext_vector_type(4)));

template <int V> struct FVec;
template <> struct FVec<1> { typedef float T; };
template <> struct FVec<2> { typedef float __attribute__((ext_vector_type(2))) T; };
template <> struct FVec<4> { typedef float __attribute__((ext_vector_type(4))) T; };
typedef typename FVec<VEC>::T vecT;

struct GemmF32Args {
    const float *A;
    const float *B;
    float *C;
    float *P;          // per-split partial sums [SPLITS][GM][GN] (STAGES 3, SPLITS > 1)
};

__device__ __forceinline__ float vget(const vecT &v, int j) {
#if VEC == 1
    (void)j;
    return v;
#else
    return v[j];
#endif
}

#if STAGES == 3
// Streaming variant.  Workgroup (nt, s) owns columns nt * 64 .. + 63 and the
// s-th of SPLITS equal K ranges; wave w of its NT / 64 waves takes the w-th
// slice of that range, KW rows, in batches of TK rows.
//
// Lane layout of one 16-row block kb .. kb + 15 (k-step e = 0..3 contracts
// the rows kb + 4 q + e, q = lane / 16 being the MFMA's k slot, so that A
// and B agree on which row each slot holds):
//   A: one 16-byte load per lane, A[lane % 16][kb + 4 q .. + 3]; element e
//      is the lane's A operand of k-step e (rows >= GM read as zero)
//   B: for each e one 16-byte load per lane, B[kb + 4 q + e][n0 + 4 c .. + 3]
//      with c = lane % 16; element j is the lane's B operand of the MFMA for
//      column group j (output columns n0 + 4 c + j)
// Accumulator j, element r of lane l is C[4 (l / 16) + r][n0 + 4 (l % 16) + j]:
// for each r a lane owns four consecutive columns.
#define SWAVES (WM * WN)
#define KSPLIT (GK / SPLITS)
#define KW (KSPLIT / SWAVES)
#define NBATCH (KW / TK)
#define BLK (TK / 16)

extern "C" __global__ __launch_bounds__(NT) void rc_gemm_f32(GemmF32Args args) {
    __shared__ f32x4 red[SWAVES][4][64];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int ntn = GN / 64;
    const int nt = blockIdx.x % ntn, sp = blockIdx.x / ntn;
    const int n0 = nt * 64;
    const int k_first = sp * KSPLIT + wave * KW;
    const int q = lane >> 4, c = lane & 15;
    const bool arow = c < GM;
    const float *Arow = args.A + (size_t)(arow ? c : 0) * GK + 4 * q;
    const float *Bcol = args.B + (size_t)(4 * q) * GN + n0 + 4 * c;

    f32x4 acc[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // Ring of PF register sets: the loads of the next PF - 1 batches are in
    // flight while a batch is multiplied (PF = 2 x UNROLL, at most NBATCH).
    constexpr int PF = (2 * UNROLL < NBATCH) ? 2 * UNROLL : NBATCH;
    f32x4 ra[PF][BLK], rb[PF][BLK][4];
    auto load = [&](int k0, int set) {
#pragma unroll
        for (int b = 0; b < BLK; ++b) {
            const int kb = k0 + 16 * b;
            ra[set][b] = arow ? *(const f32x4 *)(Arow + kb) : f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int e = 0; e < 4; ++e) rb[set][b][e] = *(const f32x4 *)(Bcol + (size_t)(kb + e) * GN);
        }
    };
    auto compute = [&](int set) {
#pragma unroll
        for (int b = 0; b < BLK; ++b)
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int j = 0; j < 4; ++j)
                    acc[j] = __builtin_amdgcn_mfma_f32_16x16x4f32(ra[set][b][e], rb[set][b][e][j], acc[j], 0, 0, 0);
    };
#pragma unroll
    for (int p = 0; p < PF; ++p) load(k_first + p * TK, p);
    for (int i = 0; i < NBATCH; i += PF) {
#pragma unroll
        for (int p = 0; p < PF; ++p) {
            if (i + p < NBATCH) {
                compute(p);
                if (i + p + PF < NBATCH) load(k_first + (i + p + PF) * TK, p);
            }
        }
    }

    // add the waves' partial sums in wave order
    if (SWAVES > 1) {
#pragma unroll
        for (int r = 0; r < 4; ++r) red[wave][r][lane] = f32x4{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
        __syncthreads();
        if (wave != 0) return;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            f32x4 v = red[0][r][lane];
#pragma unroll
            for (int w = 1; w < SWAVES; ++w) v += red[w][r][lane];
#pragma unroll
            for (int j = 0; j < 4; ++j) acc[j][r] = v[j];
        }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const int m = 4 * q + r;
        if (m >= GM) continue;
        const f32x4 v = f32x4{acc[0][r], acc[1][r], acc[2][r], acc[3][r]};
#if SPLITS == 1
        *(f32x4 *)(args.C + (size_t)m * GN + n0 + 4 * c) = v;
#else
        *(f32x4 *)(args.P + ((size_t)sp * GM + m) * GN + n0 + 4 * c) = v;
#endif
    }
}

#if SPLITS > 1
// C = sum over splits of the partials in a fixed association: each of four
// threads per 4-column group sums the splits g, g + 4, g + 8, ... in order
// and the four group sums are added in group order through LDS.  A
// workgroup covers 64 four-column groups.
extern "C" __global__ __launch_bounds__(256) void rc_gemm_f32_splitk_reduce(GemmF32Args args) {
    __shared__ f32x4 part[4][64];
    const int t = threadIdx.x, g = t >> 6;
    const size_t i = (size_t)blockIdx.x * 64 + (t & 63);
    const bool ok = i < (size_t)GM * GN / 4;
    f32x4 v = f32x4{0.f, 0.f, 0.f, 0.f};
    if (ok) {
#pragma unroll
        for (int s = g; s < SPLITS; s += 4) v += *(const f32x4 *)(args.P + (size_t)s * GM * GN + 4 * i);
    }
    part[g][t & 63] = v;
    __syncthreads();
    if (g == 0 && ok) *(f32x4 *)(args.C + 4 * i) = ((part[0][t] + part[1][t]) + part[2][t]) + part[3][t];
}
#endif

#elif RING
// Ring variant.  What bounds the double-buffered loop at ordinary sizes is
// the memory latency: a K tile of a 64 x 32 tile is 512 matrix cycles a
// wave, and one tile ahead the next one's loads had about three waves' worth
// of that to arrive in.  Here three tiles are on their way (NST - 1), without
// registers: the loads go straight to LDS, 64 lanes x 16 bytes to 1 KiB.
//
// The loads go through buffer resources whose range check returns zeros:
// vectors past M, N or K get offset OOB (VEC divides the row lengths, so a
// vector is wholly inside or outside).  LDS holds A as rows of TK floats and
// B as rows of TN (LAYOUT 0) or, like A, of TK floats (LAYOUT 1).  A lane
// feeds four k-steps from one 16-byte read of A: k-step e of the 16-row
// block kb contracts rows kb + 4 q + e (q = lane / 16, the MFMA's k slot).
// The 16-byte chunks of a row are XOR-swizzled (by the choice of the global
// chunk a lane loads) so that the lanes of one LDS access hit distinct banks:
//   rows of TK floats: a ds_read_b128 is served 16 lanes at a time, lanes
//     0-3, 12-15, 20-23 and 24-27 together, so a group mixes rows 0-3 and
//     12-15 of one chunk with rows 4-11 of the next; XOR by row / 2 for 8
//     chunks a row, by 0, 2, 3, 1 for the row blocks of 4 with 4 chunks
//   rows of TN floats: the four rows 4 q + e that a ds_read_b32 reads 16
//     columns of sit next to each other (row k of a 16-row block at position
//     4 (k % 4) + k / 4) and take the four 64-byte spans of the banks in turn
// A tile's loads, the next block's fragment reads and the MFMAs are spread
// among each other in a pinned order (UNROLL has no effect here: the loop is
// always unrolled by two tiles).  1000 x 1364 x 900 in 64 x 32 x 32 tiles:
// 34.9 us double-buffered, 29.7 us with the ring and each tile's loads, reads
// and MFMAs in turn, 27.6 us interleaved, 27.0 us (91 TFLOP/s) with the
// XCDs' ranges along the rows; the 688 tiles are 2.7 a CU, and the three of the
// fuller ones take 18.6 us of matrix time.
//
// NST, the depth, is 4, and 3 where that lets the whole grid be resident and
// 4 does not (2048 x 1024 x 128 in 64 x 32 x 32 tiles, 4 workgroups a CU: 8.1
// us double-buffered, 8.3 with 48 KiB, 7.1 with 36), and there are never more
// buffers than K tiles (1600 x 1760 x 64 in 16 x 32 x 32 tiles, us: 7.5
// double-buffered, 8.0 with four buffers, 7.1 with two).
// The last tiles are unrolled, so that their waits and buffers are constants
// (2048 x 1024 x 96 in 64 x 32 x 32 tiles: 6.7 -> 6.2 us).
#define STAGE_BYTES (4 * (TM + TN) * TK)
#define N_TILES (1ull * ((GM + TM - 1) / TM) * ((GN + TN - 1) / TN))
#define RESIDENT(bytes) (N_TILES <= 256 * (163840 / (bytes)))
#define BUFS(n) ((n) < KTILES ? (n) : KTILES)
#define NST (!RESIDENT(BUFS(4) * STAGE_BYTES) && RESIDENT(BUFS(3) * STAGE_BYTES) ? 3 : 4)
#define NBUF BUFS(NST)
#define NW (WM * WN)
#define LPW (WLOADS / NW)                        // wave-loads per wave and K tile
#define A_WL (TM * TK / 256)                     // wave-loads of the A tile (the rest are B's)
#define STAGE_FLOATS ((TM + TN) * TK)

typedef int i32x4 __attribute__((ext_vector_type(4)));
template <int V> struct IntC { static constexpr int value = V; };
// seq<A, B>(f): f(IntC<A>), ... f(IntC<B - 1>), every index a constant
template <class T, T... I> struct ISeq {};
template <int A, class F, int... I> __device__ __forceinline__ void seq_calls(F &f, ISeq<int, I...>) {
    (f(IntC<A + I>{}), ...);
}
template <int A, int B, class F> __device__ __forceinline__ void seq(F &&f) {
    if constexpr (B > A) seq_calls<A>(f, __make_integer_seq<ISeq, int, B - A>{});
}

__device__ __forceinline__ int kswz(int row) {   // XOR of a TK-float row's chunk indices
    return TK == 32 ? (row / 2) % 8 : (0x78 >> (row / 2 % 8 & 6)) & 3;
}
// position of row k of the B tile (LAYOUT 0) in LDS, and back
__device__ __forceinline__ int brow(int k) { return (k & ~15) + 4 * (k & 3) + ((k >> 2) & 3); }
// XOR of the chunk indices of the TN-float row at position p
__device__ __forceinline__ int nswz(int p) { return TN == 64 ? 4 * (p & 3) : TN == 32 ? 4 * ((p >> 1) & 1) : 0; }

extern "C" __global__ __launch_bounds__(NT) void rc_gemm_f32(GemmF32Args args) {
    __shared__ __attribute__((aligned(16))) float ring[NBUF * STAGE_FLOATS];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    __builtin_assume(wave >= 0 && wave < NW);
    const int wm = wave / WN, wn = wave % WN;
    const int q = lane >> 4, c = lane & 15;
    // Workgroups reach the 8 XCDs round-robin: each XCD takes a contiguous
    // range of the tiles, whose operands its L2 then shares.  It reads an
    // eighth of the operand along the slow dimension and all of the other,
    // so the shorter dimension is the fast one; n where they are about equal
    // (128 x 2048 x 1024 in 16 x 16 x 32 tiles, us: 12.6 with the tiles dealt
    // round-robin, 14.2 with n fast, 9.5 with m fast; 2048 x 128 x 1024: 15.6
    // and, n fast, 9.4; 1600 x 1760 x 512, 16 x 16 x 16: 52.2, n fast 41.9,
    // m fast 44.7; 1000 x 1364 x 900, 16 x 32 x 32: 39.7, 36.6 and 33.8).
    constexpr int NTN = (GN + TN - 1) / TN, NTM = (GM + TM - 1) / TM, NTILES = NTN * NTM;
    const int bid = blockIdx.y * NTN + blockIdx.x, xcd = bid & 7;
    const int item = xcd * (NTILES / 8) + min(xcd, NTILES % 8) + (bid >> 3);
    constexpr bool N_FAST = 4ll * GN <= 5ll * GM;
    const int m0 = (N_FAST ? item / NTN : item % NTM) * TM, n0 = (N_FAST ? item % NTN : item / NTM) * TN;

    constexpr unsigned OOB = 0x80000000u;        // past both operands: loads zeros
    auto rsrc = [](const void *base, unsigned bytes) {
        const unsigned long long a = (unsigned long long)base;
        i32x4 r;
        r[0] = __builtin_amdgcn_readfirstlane((int)(unsigned)a);
        r[1] = __builtin_amdgcn_readfirstlane((int)((unsigned)(a >> 32) & 0xFFFFu));   // stride 0
        r[2] = __builtin_amdgcn_readfirstlane((int)bytes);
        r[3] = 0x00020000;                                                             // raw dword access
        return r;
    };
    const i32x4 rsA = rsrc(args.A, 4u * GM * GK), rsB = rsrc(args.B, 4u * GK * GN);
    // this wave's loads: wave-load i * NW + wave of the tile (A's, then B's);
    // the lane's byte offset at K tile 0 and its row of K within the tile
    unsigned off[LPW];
    int krow[LPW];
#pragma unroll
    for (int i = 0; i < LPW; ++i) {
        const int w = i * NW + wave;
        if (w < A_WL) {
            const int ch = w * 64 + lane, row = ch / (TK / 4), col = 4 * ((ch % (TK / 4)) ^ kswz(row));
            krow[i] = col;
            off[i] = m0 + row < GM ? 4u * ((unsigned)(m0 + row) * GK + col) : OOB;
        } else {
            const int ch = (w - A_WL) * 64 + lane;
#if LAYOUT == 0
            const int p = ch / (TN / 4), col = 4 * ((ch % (TN / 4)) ^ nswz(p)), k = brow(p);
            krow[i] = k;
            off[i] = n0 + col < GN ? 4u * ((unsigned)k * GN + n0 + col) : OOB;
#else
            const int row = ch / (TK / 4), col = 4 * ((ch % (TK / 4)) ^ kswz(row));
            krow[i] = col;
            off[i] = n0 + row < GN ? 4u * ((unsigned)(n0 + row) * GK + col) : OOB;
#endif
        }
    }
    typedef __attribute__((address_space(3))) float *lds_p;
    const unsigned ring0 = (unsigned)(size_t)(lds_p)ring;
    auto issue_one = [&](auto ic, int t, int st) __attribute__((always_inline)) {
        constexpr int i = decltype(ic)::value;
        const int w = i * NW + wave;
        const bool is_a = w < A_WL;
        i32x4 rs;
#pragma unroll
        for (int r = 0; r < 4; ++r) rs[r] = is_a ? rsA[r] : rsB[r];
        const unsigned step = is_a || LAYOUT == 1 ? 4u * TK : 4u * TK * GN;
        // past the end of K: offset with its top bit set, out of range
        const unsigned o = off[i] | (GK % TK != 0 ? (unsigned)(GK - t * TK - 1 - krow[i]) & OOB : 0u);
        const unsigned koff = t * step, lds = ring0 + 4u * (st * STAGE_FLOATS) + w * 1024u;
        // inline assembly: invisible to the compiler's wait-count
        // bookkeeping, ordered by the waits below
        asm volatile("s_mov_b32 m0, %3\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %1, %2 offen lds"
                     :: "v"(o), "s"(rs), "s"(koff), "s"(lds) : "memory", "m0");
    };
    auto issue = [&](int t, int st) __attribute__((always_inline)) {
        seq<0, LPW>([&](auto i) __attribute__((always_inline)) { issue_one(i, t, st); });
    };
#define WAIT_VM(n) __builtin_amdgcn_s_waitcnt(((n) & 15) | ((((n) >> 4) & 3) << 14) | (7 << 4) | (15 << 8))

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // fragments of one 16-row block of K: element e feeds k-step e
    struct Frags {
        f32x4 a[FM], b[FN];
    };
    constexpr int NKB = TK / 16, NMF = 4 * FM * FN, NBR = LAYOUT == 0 ? 4 * FN : FN, NRD = FM + NBR;
    auto read_one = [&](auto rc, const float *As, int kb, Frags &f) __attribute__((always_inline)) {
        constexpr int r = decltype(rc)::value;
        if constexpr (r < FM) {
            f.a[r] = *(const f32x4 *)(As + (wm * WTM + r * 16 + c) * TK + 4 * ((kb / 4 + q) ^ kswz(c)));
        } else {
            const float *Bs = As + TM * TK;
#if LAYOUT == 0
            constexpr int e = (r - FM) / FN, j = (r - FM) % FN, p = 4 * e;     // position of row kb + 4 q + e: kb + p + q
            f.b[j][e] = Bs[(kb + p + q) * TN + ((wn * WTN + j * 16 + c) ^ (4 * nswz(p + q)))];
#else
            constexpr int j = r - FM;
            f.b[j] = *(const f32x4 *)(Bs + (wn * WTN + j * 16 + c) * TK + 4 * ((kb / 4 + q) ^ kswz(c)));
#endif
        }
    };
    // One block: its MFMAs, with the next block's fragment reads and, in the
    // steady part, a share of tile t + NST - 1's loads spread between them
    // (the order is pinned: the pipes run side by side).
    auto block = [&](const Frags &f, auto kbc, const float *An, int kbn, Frags &nxt, auto steady, int t, int st)
                     __attribute__((always_inline)) {
        seq<0, NMF>([&](auto mc) __attribute__((always_inline)) {
            constexpr int m = decltype(mc)::value, e = m / (FM * FN), i = m / FN % FM, j = m % FN;
            seq<m * NRD / NMF, (m + 1) * NRD / NMF>([&](auto r) __attribute__((always_inline)) { read_one(r, An, kbn, nxt); });
            if constexpr (decltype(steady)::value) {
                constexpr int s = decltype(kbc)::value * NMF + m;
                seq<s * LPW / (NKB * NMF), (s + 1) * LPW / (NKB * NMF)>(
                    [&](auto d) __attribute__((always_inline)) { issue_one(d, t + NST - 1, st); });
            }
            acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(f.a[i][e], f.b[j][e], acc[i][j], 0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
        });
    };

#pragma unroll
    for (int u = 0; u < NST - 1; ++u)
        if (u < KTILES) issue(u, u);
    if (KTILES > 2 && NST > 3) {
        WAIT_VM(2 * LPW);
    } else if (KTILES > 1) {
        WAIT_VM(LPW);
    } else {
        WAIT_VM(0);
    }
    asm volatile("s_barrier" ::: "memory");
    Frags f[2];
    seq<0, NRD>([&](auto r) __attribute__((always_inline)) { read_one(r, ring, 0, f[0]); });
    int cur = 0;
    auto tile = [&](int t, auto par, auto steady) __attribute__((always_inline)) {
        constexpr int P = decltype(par)::value;
        const int nx = (cur + 1) % NBUF, st = (cur + NST - 1) % NBUF;
        // Tile t + 1 has landed (of the steady part's tiles t + 2 is in
        // flight in a ring of four), and every wave is done with tile t - 1, whose buffer tile
        // t + NST - 1 takes: its reads were consumed by MFMAs issued before.
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (decltype(steady)::value) {
            WAIT_VM((NST - 3) * LPW);
            asm volatile("s_barrier" ::: "memory");
        } else if (t + 1 < KTILES) {
            if (NST > 3 && t + 2 < KTILES) {
                WAIT_VM(LPW);
            } else {
                WAIT_VM(0);
            }
            asm volatile("s_barrier" ::: "memory");
            if (t + NST - 1 < KTILES) issue(t + NST - 1, st);
        }
        const float *As = ring + cur * STAGE_FLOATS, *An = ring + nx * STAGE_FLOATS;  // the last tile reads a stale stage; unused
        seq<0, NKB>([&](auto kbc) __attribute__((always_inline)) {
            constexpr int kb = decltype(kbc)::value, ci = (P * NKB + kb) & 1;
            block(f[ci], kbc, kb + 1 < NKB ? As : An, kb + 1 < NKB ? 16 * (kb + 1) : 0, f[1 - ci], steady, t, st);
        });
        cur = nx;
    };
    constexpr int STEADY_TILES = KTILES >= NST ? ((KTILES - (NST - 1)) & ~1) : 0;
    int t = 0;
#pragma nounroll
    for (; t < STEADY_TILES; t += 2) {
        tile(t, IntC<0>{}, IntC<1>{});
        tile(t + 1, IntC<1>{}, IntC<1>{});
    }
    cur = STEADY_TILES % NBUF;
    seq<STEADY_TILES, KTILES>([&](auto u) __attribute__((always_inline)) {
        tile(decltype(u)::value, IntC<decltype(u)::value & 1>{}, IntC<0>{});
    });
#undef WAIT_VM

#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const int m = m0 + wm * WTM + i * 16 + 4 * q + r, n = n0 + wn * WTN + j * 16 + c;
                if (!RAGGED || (m < GM && n < GN)) args.C[(size_t)m * GN + n] = acc[i][j][r];
            }
}

#else
extern "C" __global__ __launch_bounds__(NT) void rc_gemm_f32(GemmF32Args args) {
    __shared__ float As[STAGES][TM][TK + 1];
    __shared__ float Bs[STAGES][TK][TN + 1];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = tid >> 6;
    const int wm = wave / WN, wn = wave % WN;
    const int m0 = blockIdx.y * TM, n0 = blockIdx.x * TN;

    f32x4 acc[FM][FN];
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j) acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    vecT ra[A_LOADS], rb[B_LOADS];

    // a vector load of row `row`, columns col .. col + VEC - 1 of a
    // rows x cols matrix; zeros outside it (tiles crossing an edge)
    auto ld = [&](const float *base, int row, int col, int rows, int cols) -> vecT {
        if (RAGGED && (row >= rows || col >= cols)) return vecT{};
        return *(const vecT *)(base + (size_t)row * cols + col);
    };
    auto gload = [&](int k0) {
#pragma unroll
        for (int i = 0; i < A_LOADS; ++i) {
            int v = tid + i * NT;
            int r = v / (TK / VEC), c = (v % (TK / VEC)) * VEC;
            ra[i] = ld(args.A, m0 + r, k0 + c, GM, GK);
        }
#pragma unroll
        for (int i = 0; i < B_LOADS; ++i) {
            int v = tid + i * NT;
#if LAYOUT == 0
            int r = v / (TN / VEC), c = (v % (TN / VEC)) * VEC;
            rb[i] = ld(args.B, k0 + r, n0 + c, GK, GN);
#else
            int r = v / (TK / VEC), c = (v % (TK / VEC)) * VEC;
            rb[i] = ld(args.B, n0 + r, k0 + c, GN, GK);
#endif
        }
    };

    auto swrite = [&](int s) {
#pragma unroll
        for (int i = 0; i < A_LOADS; ++i) {
            int v = tid + i * NT;
            int r = v / (TK / VEC), c = (v % (TK / VEC)) * VEC;
#pragma unroll
            for (int j = 0; j < VEC; ++j) As[s][r][c + j] = vget(ra[i], j);
        }
#pragma unroll
        for (int i = 0; i < B_LOADS; ++i) {
            int v = tid + i * NT;
#if LAYOUT == 0
            int r = v / (TN / VEC), c = (v % (TN / VEC)) * VEC;
#pragma unroll
            for (int j = 0; j < VEC; ++j) Bs[s][r][c + j] = vget(rb[i], j);
#else
            int r = v / (TK / VEC), c = (v % (TK / VEC)) * VEC;
#pragma unroll
            for (int j = 0; j < VEC; ++j) Bs[s][c + j][r] = vget(rb[i], j);
#endif
        }
    };

    auto compute = [&](int s) {
#pragma unroll
        for (int kk = 0; kk < TK; kk += 4) {
            float a[FM], b[FN];
#pragma unroll
            for (int i = 0; i < FM; ++i) a[i] = As[s][wm * WTM + i * 16 + (lane & 15)][kk + (lane >> 4)];
#pragma unroll
            for (int j = 0; j < FN; ++j) b[j] = Bs[s][kk + (lane >> 4)][wn * WTN + j * 16 + (lane & 15)];
#pragma unroll
            for (int i = 0; i < FM; ++i)
#pragma unroll
                for (int j = 0; j < FN; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
    };

#if STAGES == 1
#pragma unroll UNROLL
    for (int kt = 0; kt < KTILES; ++kt) {
        gload(kt * TK);
        swrite(0);
        __syncthreads();
        compute(0);
        __syncthreads();
    }
#else
    gload(0);
    swrite(0);
    __syncthreads();
#pragma unroll UNROLL
    for (int kt = 0; kt < KTILES; ++kt) {
        if (kt + 1 < KTILES) gload((kt + 1) * TK);
        compute(kt & 1);
        if (kt + 1 < KTILES) swrite((kt + 1) & 1);
        __syncthreads();
    }
#endif

#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
        for (int j = 0; j < FN; ++j)
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                int m = m0 + wm * WTM + i * 16 + 4 * (lane >> 4) + r;
                int n = n0 + wn * WTN + j * 16 + (lane & 15);
                if (!RAGGED || (m < GM && n < GN)) args.C[(size_t)m * GN + n] = acc[i][j][r];
            }
}
#endif
