// Householder reduction to tridiagonal form with the trailing matrix held in the registers of the whole chip (part of eig_direct.hip:
// included there, in its namespace, after DirMat).
//
// A column of the reduction needs the product of the whole trailing matrix with one vector, and the next column needs that product.
// Read from memory the matrix costs 4 n^2 / 2 bytes a column (8 us of a 4609-wide factor at 5 TB/s) and a launch or two on top.  The 256
// compute units' registers hold 128 MB, a 4609-wide factor is 85: so each workgroup keeps a few rows of it for good, and what is left
// per column is one all-gather of the products between the workgroups of a factor.
//
//  - Workgroup p has rows [p R, p R + R) of the trailing matrix, thread i of it columns i, i + 512, .. of all R rows (S <= 9 column
//    slots; R S <= 192 registers of a thread's 256).  The column x that is being reduced lies in registers the same way, in every
//    workgroup of the factor alike, so norms and inner products are formed by each for itself, in the same order.
//  - Per column: products of the own rows with x (summed over the waves through LDS), published with the own rows' elements of the next
//    column as one 8-byte word per row; then the words of all rows are gathered.  The word itself says whether it is there: the
//    slots hold EMPTY before.  Everything after that is local: reflector, w, the next column, and ONE pass over the registers that
//    applies the rank-2 update (on the matrix cores, as outer products: a third of the pass is left to the vector units) and forms the
//    next products.
//  - The words go through a ring of four columns (eig_chip_ring.h: who publishes, waits and empties when, and why no word is emptied
//    that somebody still looks for).  The s_waitcnt before a publication orders it after what its wave has emptied.  Loads and stores
//    are relaxed agent-scope atomics of 8 bytes.
//  - Polling too early costs more than it gains (the line is fetched empty, and the writer has to take it away again): measured between
//    256 workgroups, 4608 words: 3.0 us a column polling at once, 2.3 after a pause of 1024 cycles; 64 workgroups: 2.3 and 1.5.  In the
//    reduction the workgroups have something to do meanwhile; pauses of 0, 2, 6, 12 and 16 times 64 cycles, whole decompositions in ms: one factor
//    of 577 2.72, 2.68, 2.65, 2.71, 2.77, of 2305 12.4, 12.2, 11.6, 11.9, 12.1, three of 4609 72.7, 72.1, 70.0, 69.5, 70.3.
//
// Measured (whole decompositions, ms, the chain of launches and this): one factor 577 wide 5.2 and 2.5, 2049 19.3 and 10.1, 4609 57.6 and 31.1;
// three of 4609 62.5, twenty of 577 3.5.  A column of a 4609-wide factor takes 4.3 us after a quarter of them (1.4 of it the exchange) and 2.2 at its end, where the chain of
// launches took 13 and 7.  Also measured, and worse: shares of x^T A x among the words, so that nobody has to sum over its waves (a barrier less,
// but every wave looks at up to 262 words more: 577 2.6 -> 3.0 ms, 4609 32.9 -> 37.0); tags beside the values in place of EMPTY (twice the words);
// a flag per workgroup and plain loads after it.
//
// A launch takes every factor some columns further (ChipJob), then the trailing matrices go back to memory and are dealt out anew:
// a matrix that has shrunk needs fewer workgroups, and others take their place.  All workgroups of a launch must be resident at once
// (cooperative launch, one per compute unit that the stream may use).  Another kernel may hold compute units for long all the same (a
// collective that waits for its peer, another process), so every wait is bounded, by KFAC_CHIP_POLLS: 0.1 to 0.3 s.  A workgroup that gives
// up says so (chip_flags); the others of the call and the launches after it look at that and leave.  Factors whose reduction was
// given up are decomposed again with the chain of launches, which needs no two workgroups at once.

constexpr int CHIP_SLOTS = 9;
constexpr int CHIP_WIDE = 512, CHIP_NARROW = 256;         // threads of a workgroup
constexpr int CHIP_NARROW_SLOTS = 8;                      // nine would not leave the registers for anything else
// Columns of a factor that count as one workgroup of a crowd: where the factors of a call are one (more of them than compute units), narrow
// workgroups, two to a compute unit, hide each other's exchange.  ms with 4, 16, 32, and without any narrow ones: thirty factors of 1100 14.0, 14.0, 14.0,
// 16.0, twenty of 577 3.54, 3.53, 3.52, 3.66, nine 3.01, 3.01, 3.08, 3.10, sixty of ResNet-32's widths 3.73, 3.73, 3.91, 3.82; the price is fifty of 300, 2.44, 2.42, 2.39, 2.16.
constexpr int CHIP_CROWD = 16;
constexpr int CHIP_MAX_N = CHIP_WIDE * CHIP_SLOTS + 1;    // the widest factor: its first column is never part of the trailing matrix
constexpr int CHIP_ROWS = 64;                             // rows of a workgroup, at most: the lanes of the wave that publishes
// A workgroup with fewer rows saves less than one more in the exchange costs.  ms with at least 4, 8, 12, 24 rows: one factor of 577 2.66, 2.65, 2.67, 2.84,
// of 2305 11.6, 11.6, 12.2, 12.9, fifty of 300 2.52, 2.42, 2.55, 2.53.
constexpr int CHIP_ROWS_MIN = 8;
constexpr int CHIP_WGS = 256;                             // workgroups of a factor, at most
constexpr int CHIP_JOBS = 64;                             // factors of a launch, at most: a workgroup finds its own by one ballot
constexpr int CHIP_PAUSE = 6;                             // of 64 cycles, before the first look at the others' words
// Up to CHIP_WHOLE columns a factor goes in one launch; the fewest columns of a launch otherwise.  ms up to 256, 400, 640, 900, 1300: one factor of 577 2.88, 2.71,
// 2.65, 2.65, 2.65, of 1153 5.78, 5.58, 5.54, 5.32, 5.06, sixty of ResNet-32's widths 4.24, 4.04, 3.73, 3.72, 3.72, thirty of 1100 14.9, 14.7, 14.0, 13.9, 18.9.
constexpr int CHIP_WHOLE = 640, CHIP_STEPS_MIN = 96;
constexpr int CHIP_LOOK = 256;                            // polls between two looks at whether the call has been given up

// Rows that a workgroup of S column slots can hold, in groups of four (the rows of a matrix instruction; two rows of the nine-slot kind
// are left to ordinary ones), and the rows whose sums are in registers together.
constexpr int chip_rows(int S) { return S == 9 ? 18 : S == 8 ? 20 : S == 7 ? 24 : S == 6 ? 28 : S == 5 ? 32 : S == 4 ? 40 : S == 3 ? 48 : 64; }
constexpr int chip_piece(int S) { return S >= 3 ? 8 : 16; }

struct ChipJob {
    int m;               // factor
    int k0, steps;       // columns k0 .. k0 + steps - 1
    int rows, wgs, base; // rows per workgroup, workgroups, the first of them
    int slots;           // column slots
    int turn;            // launches of this factor before this one; its parity says which half of the ring buffer (the other is emptied for the next)
};

template <int NT> struct ChipSmem {
    static constexpr int WAVES = NT / 64;
    float xs[NT * CHIP_SLOTS + CHIP_ROWS], ys[NT * CHIP_SLOTS + CHIP_ROWS];     // x and y by row, for those that need single elements
    float col[CHIP_ROWS], part[WAVES][CHIP_ROWS], nrm[WAVES];
    double dot[WAVES];
    int failed;
};

// Sums over the wave of N values at once: every step folds two registers into one, the upper half of the lanes taking over the second.
// Lane l ends up with the sum of value chip_fold_index<N>(l).
template <int N> __device__ inline int chip_fold_index(int lane) {      // N or more: this lane holds a copy
    constexpr int n1 = (N + 1) / 2, n2 = (n1 + 1) / 2, n3 = (n2 + 1) / 2, n4 = (n3 + 1) / 2, n5 = (n4 + 1) / 2, n6 = (n5 + 1) / 2;
    static_assert(n6 == 1, "at most 64 values");
    constexpr int n[7] = {N, n1, n2, n3, n4, n5, n6};
    int i = 0;
    bool own = true;
#pragma unroll
    for (int s = 5; s >= 0; --s) {       // step s folded n[s] registers into n[s + 1] by bit 5 - s of the lane
        i += (lane >> (5 - s)) & 1 ? n[s + 1] : 0;
        own = own && i < n[s];
    }
    return own ? i : N;
}
template <int CTRL> __device__ inline float dpp_move(float v) { return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true)); }
template <int H, int N, int CTRL> __device__ inline void chip_fold_dpp(float (&v)[N], int n, bool up) {   // n values, H = ceil(n / 2)
#pragma unroll
    for (int i = 0; i < H; ++i) {
        if (i + H < n) {
            const float keep = up ? v[i + H] : v[i], give = up ? v[i] : v[i + H];
            v[i] = keep + dpp_move<CTRL>(give);
        } else
            v[i] += dpp_move<CTRL>(v[i]);
    }
}
template <int N> __device__ inline float chip_fold(float (&v)[N], int lane) {
    constexpr int h0 = (N + 1) / 2, h1 = (h0 + 1) / 2, h2 = (h1 + 1) / 2, h3 = (h2 + 1) / 2, h4 = (h3 + 1) / 2, h5 = (h4 + 1) / 2;
#pragma unroll
    for (int i = 0; i < h0; ++i) {      // lanes l and l ^ 32
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v[i]), __float_as_uint(v[i + h0 < N ? i + h0 : i]), false, false);
        v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
#pragma unroll
    for (int i = 0; i < h1; ++i) {      // lanes l and l ^ 16
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v[i]), __float_as_uint(v[i + h1 < h0 ? i + h1 : i]), false, false);
        v[i] = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    chip_fold_dpp<h2, N, 0x128>(v, h1, (lane & 8) != 0);     // row_ror:8
    chip_fold_dpp<h3, N, 0x141>(v, h2, (lane & 4) != 0);     // row_half_mirror
    chip_fold_dpp<h4, N, 0x4E>(v, h3, (lane & 2) != 0);      // quad_perm 2,3,0,1
    chip_fold_dpp<h5, N, 0xB1>(v, h4, (lane & 1) != 0);      // quad_perm 1,0,3,2
    return v[0];
}

// C + (rows' factors) (column's factor)^T for four rows, group g of the lanes that hold the rows' factors
__device__ inline floatx4 chip_outer(float rows, float column, floatx4 c, int g) {
    switch (g) {
#define KFAC_CHIP_OUTER(G) case G: return __builtin_amdgcn_mfma_f32_4x4x1f32(rows, column, c, 4, G, 0);
        KFAC_CHIP_OUTER(0) KFAC_CHIP_OUTER(1) KFAC_CHIP_OUTER(2) KFAC_CHIP_OUTER(3) KFAC_CHIP_OUTER(4) KFAC_CHIP_OUTER(5) KFAC_CHIP_OUTER(6) KFAC_CHIP_OUTER(7)
        KFAC_CHIP_OUTER(8) KFAC_CHIP_OUTER(9) KFAC_CHIP_OUTER(10) KFAC_CHIP_OUTER(11) KFAC_CHIP_OUTER(12) KFAC_CHIP_OUTER(13) KFAC_CHIP_OUTER(14)
#undef KFAC_CHIP_OUTER
        default: return __builtin_amdgcn_mfma_f32_4x4x1f32(rows, column, c, 4, 15, 0);
    }
}

// (all of it through global pointers: a flat access also counts on the LDS counter, and every wait for LDS behind it takes a trip to memory)
typedef global_ptr<unsigned long long> ChipWords;
// word i of those at `base`: a scalar base and 32 bits of offset, so that no lane keeps 64-bit addresses
__device__ inline unsigned long long chip_load(ChipWords base, unsigned i) { return __hip_atomic_load(base + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
// of a factor: [0] its reduction was given up (of the one that the launches of a call have in common also [1]: some reduction of the call was)
__device__ inline ChipWords chip_flags(const DirMat &M) { return as_global((unsigned long long *)M.apan) + (size_t)2 * CHIP_RING * M.np; }
__device__ inline void chip_store(ChipWords p, unsigned long long v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

template <int CHIP_NT, int S>
__device__ inline void chip_reduce(const DirMat &M, const ChipJob &J, int p, ChipWords call, int polls, ChipSmem<CHIP_NT> &sm) {
    constexpr int CHIP_WAVES = CHIP_NT / 64, R = chip_rows(S), G = R / 4, X = R % 4, PIECE = chip_piece(S), PIECES = (4 * G + PIECE - 1) / PIECE;
    static_assert((X == 0 || 4 * G % PIECE == 0) && R <= CHIP_ROWS, "extra rows follow whole pieces");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = M.n - 1 - J.k0, r0 = p * J.rows, nr = min(J.rows, m - r0);     // nr >= 1: the last workgroup has row m - 1
    const bool last = p == J.wgs - 1, tail = tid + CHIP_NT * (S - 1) < m;        // only the last column slot reaches past the matrix
    const int j1 = m > 64 * wave ? (m - 1 - 64 * wave) / CHIP_NT : -1;           // the last slot in which this wave has columns
    const int64_t ld = M.ld;
    const global_ptr<float> A0 = as_global(M.A) + (int64_t)J.k0 * ld + J.k0 + 1;      // row k0, from the element beside the diagonal on
    const ChipWords ring = as_global((unsigned long long *)M.apan) + (size_t)(J.turn & 1) * CHIP_RING * M.np;
    const global_ptr<double> Md = as_global(M.d), Me = as_global(M.e);
    const global_ptr<float> Mtau = as_global(M.tau);
    floatx4 a[G][S];
    float ax[X ? X : 1][S];          // the rows past the groups
    float x[S], v[S], w[S], s2 = 0.f;
#pragma unroll
    for (int j = 0; j < S; ++j) {
        const int c = tid + CHIP_NT * j;
        x[j] = (j < S - 1 || tail) ? A0[c] : 0.f;
        v[j] = w[j] = 0.f;
        sm.xs[c] = x[j];
        s2 = fmaf(x[j], c == 0 ? 0.f : x[j], s2);
    }
#pragma unroll
    for (int i = 0; i < R; ++i) {
        const global_ptr<const float> row = A0 + (int64_t)(1 + r0 + min(i, nr - 1)) * ld + tid;
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const float e = (j < S - 1 || tail) ? row[CHIP_NT * j] : 0.f;
            if (i < 4 * G) a[i >> 2][j][i & 3] = e;
            else ax[X ? i - 4 * G : 0][j] = e;
        }
    }
    if (J.turn == 0 && last && tid == 0) Md[J.k0] = (double)A0[-1];
    if (tid < nr) {
        const ChipWords other = as_global((unsigned long long *)M.apan) + (size_t)(~J.turn & 1) * CHIP_RING * M.np + r0 + tid;
#pragma unroll
        for (int q = 0; q < CHIP_RING; ++q) other[(size_t)q * M.np] = CHIP_EMPTY;
    }
    float nv = 0.f, nw = 0.f;       // lane i: -v and -w of row r0 + i
    for (int t = 0;; ++t) {
        // x: column k0 + t, rows t .. m - 1 of the trailing matrix (zero before).  v, w: the reflector before it, not yet applied.
        // s2: this thread's share of the squared norm below the column's first element.
        s2 = wave_sum_all(s2);
        if (lane == 0) sm.nrm[wave] = s2;
        // A <- A - v w^T - w v^T and A x in one pass; rows and columns before t are finished.  The update goes to the matrix cores: 4 x 4 x 1
        // outer products have the lane's own column and four rows in each lane, the rows' factors broadcast from the lanes that have them.
        const int j0 = max(0, (t - 64 * wave - 63 + CHIP_NT - 1) / CHIP_NT);
#pragma unroll
        for (int q = 0; q < PIECES; ++q)
            if (q * PIECE < nr && r0 + q * PIECE + PIECE > t) {
                float acc[PIECE];
#pragma unroll
                for (int i = 0; i < PIECE; ++i) acc[i] = 0.f;
#pragma unroll
                for (int h = 0; h < PIECE; h += 8)
                    if (q * PIECE + h < nr)
#pragma unroll
                        for (int j = 0; j < S; ++j)
                            if (j >= j0 && j <= j1)
#pragma unroll
                                for (int g = (q * PIECE + h) / 4; g < (q * PIECE + h) / 4 + 2 && g < G; ++g) {
                                    floatx4 e = chip_outer(nw, v[j], a[g][j], g);
                                    e = chip_outer(nv, w[j], e, g);
                                    a[g][j] = e;
#pragma unroll
                                    for (int i = 0; i < 4; ++i) acc[4 * g - q * PIECE + i] = fmaf(e[i], x[j], acc[4 * g - q * PIECE + i]);
                                }
                const float sum = chip_fold<PIECE>(acc, lane);
                const int at = chip_fold_index<PIECE>(lane);
                if (at < PIECE) sm.part[wave][q * PIECE + at] = sum;
            }
        if (X > 0 && 4 * G < nr && r0 + R > t)
#pragma unroll
            for (int i = 0; i < X; ++i) {
                const float rv = lane_value(nv, 4 * G + i), rw = lane_value(nw, 4 * G + i);
                float acc = 0.f;
#pragma unroll
                for (int j = 0; j < S; ++j)
                    if (j >= j0 && j <= j1) {
                        ax[i][j] = fmaf(rv, w[j], fmaf(rw, v[j], ax[i][j]));
                        acc = fmaf(ax[i][j], x[j], acc);
                    }
                acc = wave_sum_all(acc);
                if (lane == 0) sm.part[wave][4 * G + i] = acc;
            }
        if (t == J.steps) break;
        const ChipWords slot = ring + (size_t)ChipRing::slot(t) * M.np;
        if (ChipRing::leaves(r0, nr, t)) {         // all rows of this workgroup are finished, and all its waves have gathered column t - 1
            if (tid == 0 && ChipRing::receipt(r0, nr, t) >= 0) chip_store(slot + ChipRing::receipt(r0, nr, t), 0);
            return;
        }
        if (wave == ((t >> 6) & (CHIP_WAVES - 1))) {      // the own rows' elements of column t, by the lane that has it
#pragma unroll
            for (int j = 0; j < S; ++j)
                if (j == t / CHIP_NT && lane == (t & 63))
#pragma unroll
                    for (int g = 0; g < G; ++g)
                        if (g * 4 < nr) *(floatx4 *)(sm.col + 4 * g) = a[g][j];
            if (X > 0)
#pragma unroll
                for (int j = 0; j < S; ++j)
                    if (j == t / CHIP_NT && lane == (t & 63))
#pragma unroll
                        for (int i = 0; i < X; ++i) sm.col[4 * G + i] = ax[i][j];
        }
        __syncthreads();
        const int r = r0 + lane, k = J.k0 + t;
        float art = 0.f;
        if (tid < nr) {
            float y = 0.f;
            art = sm.col[tid];
#pragma unroll
            for (int g = 0; g < CHIP_WAVES; ++g) y += sm.part[g][tid];
            unsigned long long word = (unsigned long long)__float_as_uint(y) | (unsigned long long)__float_as_uint(art) << 32;
            if (word == CHIP_EMPTY) word = 0x7fc000007fc00000ull;      // two NaNs that look like an empty slot
            if (r < t) word = 0;                                       // a finished row's word is only waited for
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // what was emptied after column t - 1 is empty
            chip_store(slot + r0 + tid, word);
        }
        const float alpha = sm.xs[t], xr = sm.xs[r];
        s2 = 0.f;
#pragma unroll
        for (int g = 0; g < CHIP_WAVES; ++g) s2 += sm.nrm[g];
        float beta = alpha, tau = 0.f, scale = 0.f;
        if (s2 > 0.f) {
            beta = -copysignf(sqrtf(fmaf(alpha, alpha, s2)), alpha);
            tau = (beta - alpha) / beta;
            scale = 1.f / (alpha - beta);
        }
        __builtin_amdgcn_s_sleep(CHIP_PAUSE);
        unsigned long long u[S];
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const int c = tid + CHIP_NT * j;
            u[j] = 0;
            if (c >= ChipRing::first(t) && (j < S - 1 || tail)) u[j] = chip_load(slot + CHIP_NT * j, tid);
        }
        for (int spin = 0;; ++spin) {
            bool there = true;
#pragma unroll
            for (int j = 0; j < S; ++j)
                if (u[j] == CHIP_EMPTY) {
                    there = false;
                    u[j] = chip_load(slot + CHIP_NT * j, tid);
                }
            if (__all(there)) break;
            if (spin >= polls || (spin % CHIP_LOOK == CHIP_LOOK - 1 && chip_load(call, 0) != 0)) { sm.failed = 1; break; }
        }
        double dot = 0.0;
#pragma unroll
        for (int j = 0; j < S; ++j) {
            if (j < j0 || j > j1) continue;
            const int c = tid + CHIP_NT * j;
            const float ac = __uint_as_float((unsigned)(u[j] >> 32));
            w[j] = scale * fmaf(-beta, ac, __uint_as_float((unsigned)u[j]));      // y; w = tau y + cw v follows once the inner product is known
            v[j] = c == t ? 1.f : x[j] * scale;
            x[j] = ac;
            sm.ys[c] = w[j];
            dot = fma((double)v[j], (double)w[j], dot);
        }
        dot = wave_sum_f64(dot);
        if (lane == 0) sm.dot[wave] = dot;
        __syncthreads();
        const float yt = sm.ys[t], yr = sm.ys[r];
        const int failed = sm.failed;
        dot = 0.0;
#pragma unroll
        for (int g = 0; g < CHIP_WAVES; ++g) dot += sm.dot[g];
        if (failed) {
            if (tid == 0) {
                chip_store(chip_flags(M), 1);
                chip_store(call, 1);
            }
            return;
        }
        const float cw = (float)(-0.5 * tau * tau * dot), wt = fmaf(tau, yt, cw);
        const float vr = lane < nr && r >= t ? (r == t ? 1.f : xr * scale) : 0.f;
        nv = -vr;
        nw = lane < nr && r >= t ? -fmaf(tau, yr, cw * vr) : 0.f;
        s2 = 0.f;
#pragma unroll
        for (int j = 0; j < S; ++j) {
            if (j < j0 || j > j1) continue;
            const int c = tid + CHIP_NT * j;
            w[j] = fmaf(tau, w[j], cw * v[j]);
            x[j] = c > t ? x[j] - fmaf(v[j], wt, w[j]) : 0.f;
            sm.xs[c] = x[j];
            s2 = fmaf(x[j], c == t + 1 ? 0.f : x[j], s2);
        }
        if (wave == CHIP_WAVES - 1 && lane < nr) A0[(int64_t)t * ld + r] = vr;     // row k: everybody has published, so has read it
        if (tid < nr && r == t) Md[k + 1] = (double)(art - 2.f * wt);
        const int done = ChipRing::emptied(t);      // nobody looks for its words any more
        if (done >= 0 && tid < nr) chip_store(ring + (size_t)ChipRing::slot(done) * M.np + r0 + tid, CHIP_EMPTY);
        if (last && tid == 64) {
            Mtau[k] = tau;
            Me[k] = (double)beta;
        }
    }
    // the trailing matrix and its first column, for the factor's next launch
    const int T = J.steps;
    if (T == m) return;
#pragma unroll
    for (int i = 0; i < R; ++i) {
        if (i >= nr || r0 + i < T) continue;
        const global_ptr<float> row = A0 + (int64_t)(1 + r0 + i) * ld + tid;
#pragma unroll
        for (int j = 0; j < S; ++j)
            if (tid + CHIP_NT * j >= T && (j < S - 1 || tail)) row[CHIP_NT * j] = i < 4 * G ? a[i < 4 * G ? i >> 2 : 0][j][i & 3] : ax[X && i >= 4 * G ? i - 4 * G : 0][j];
    }
    if (last)
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const int c = tid + CHIP_NT * j;
            if (c >= T && (j < S - 1 || tail)) A0[(int64_t)T * ld + c] = x[j];
        }
}

template <int NT> __global__ __launch_bounds__(NT, 2) void dir_chip_kernel(const DirMat *mats, const ChipJob *jobs, int count, int lead, int polls) {
    __shared__ __attribute__((aligned(16))) ChipSmem<NT> sm;
    const int lane = threadIdx.x & 63;
    const int base = lane < count ? jobs[lane].base : INT_MAX;      // ascending
    const ChipJob J = jobs[__popcll(__ballot(base <= (int)blockIdx.x)) - 1];
    const DirMat M = mats[J.m];
    const int p = (int)blockIdx.x - J.base;
    const ChipWords call = as_global((unsigned long long *)mats[lead].apan) + (size_t)2 * CHIP_RING * mats[lead].np + 1;
    if (threadIdx.x == 0) sm.failed = chip_load(call, 0) != 0;
    __syncthreads();
    if (sm.failed) {       // given up, by an earlier launch or in this one
        if (threadIdx.x == 0) chip_store(chip_flags(M), 1);
        return;
    }
    switch (J.slots) {
        case 1: chip_reduce<NT, 1>(M, J, p, call, polls, sm); break;
        case 2: chip_reduce<NT, 2>(M, J, p, call, polls, sm); break;
        case 3: chip_reduce<NT, 3>(M, J, p, call, polls, sm); break;
        case 4: chip_reduce<NT, 4>(M, J, p, call, polls, sm); break;
        case 5: chip_reduce<NT, 5>(M, J, p, call, polls, sm); break;
        case 6: chip_reduce<NT, 6>(M, J, p, call, polls, sm); break;
        case 7: chip_reduce<NT, 7>(M, J, p, call, polls, sm); break;
        case 8: chip_reduce<NT, 8>(M, J, p, call, polls, sm); break;
        default:
            if constexpr (NT == CHIP_WIDE) chip_reduce<NT, 9>(M, J, p, call, polls, sm);
    }
}

// ---- which factor takes how many columns further in which launch ----
struct ChipLaunch { unsigned at; int jobs, wgs, threads; double flops, bytes; };     // at: index of its first job
struct ChipFactor { int m, n, k, turn; };                                           // width n, k columns reduced

inline int chip_slots(int size, int threads) { return (size + threads - 1) / threads; }
inline int chip_need(int size, int threads) {      // workgroups that hold a trailing matrix of this size
    const int rows = chip_rows(chip_slots(size, threads));
    return (size + rows - 1) / rows;
}
inline int chip_widest(int cus) {      // widest factor that fits (0: none does)
    int n = CHIP_MAX_N;
    while (n > 1 && chip_need(n - 1, CHIP_WIDE) > std::min(cus, CHIP_WGS)) --n;
    return n > 1 ? n : 0;
}

// The widest factors that are left come first; narrower ones fill what they leave free.
inline void chip_plan(std::vector<ChipFactor> left, int cus, std::vector<ChipJob> &jobs, std::vector<ChipLaunch> &launches) {
    auto size = [](const ChipFactor &f) { return f.n - 1 - f.k; };
    while (!left.empty()) {
        std::stable_sort(left.begin(), left.end(), [&](const ChipFactor &a, const ChipFactor &b) { return size(a) > size(b); });
        const int widest = size(left[0]);
        // Two narrow workgroups of a compute unit hide each other's exchange where the chip is full of factors; one factor alone has fewer
        // column slots, and shorter sections between the exchanges, in wide ones.
        int crowd = 0;
        for (const ChipFactor &f : left) crowd += (size(f) + CHIP_CROWD - 1) / CHIP_CROWD;
        const int threads = crowd > cus && widest <= CHIP_NARROW * CHIP_NARROW_SLOTS ? CHIP_NARROW : CHIP_WIDE;
        // dealing a matrix out anew costs its bytes and a launch, some 50 us for the widest; not doing it, workgroups that have run out of rows
        // and factors that wait for their turn.  ms with a third, a quarter, a sixth, a twelfth of the columns: one factor of 1153 5.18, 5.28, 5.54, 5.73, of 4609 33.3, 33.2, 33.5,
        // 34.4, thirty of 1100 14.9, 14.4, 14.0, 14.0, three of 4609 71.2, 70.8, 70.0, 69.6
        const int steps = widest <= CHIP_WHOLE ? widest : std::max(CHIP_STEPS_MIN, widest / 6);
        ChipLaunch L{(unsigned)jobs.size(), 0, 0, threads, 0.0, 0.0};
        int free = cus * (CHIP_WIDE / threads);
        std::vector<size_t> taken, sizes;
        for (size_t q = 0; q < left.size() && taken.size() < CHIP_JOBS; ++q) {
            const int z = size(left[q]), need = chip_need(z, threads), S = chip_slots(z, threads);
            if (need > free) continue;
            free -= need;
            taken.push_back(q);
            sizes.push_back(z);
            jobs.push_back(ChipJob{left[q].m, left[q].k, std::min(steps, z), chip_rows(S), need, 0, S, left[q].turn});
        }
        // what is free goes to those that do the most per workgroup, a group less each time
        for (;;) {
            int most = -1;
            for (size_t q = 0; q < taken.size(); ++q) {
                const ChipJob &J = jobs[L.at + q];
                if (J.rows - 4 >= CHIP_ROWS_MIN && (most < 0 || J.rows * J.slots > jobs[L.at + most].rows * jobs[L.at + most].slots)) most = (int)q;
            }
            if (most < 0) break;
            ChipJob &J = jobs[L.at + most];
            const int rows = (J.rows - 1) / 4 * 4, want = ((int)sizes[most] + rows - 1) / rows;
            if (want - J.wgs > free || want > CHIP_WGS) break;
            free -= want - J.wgs;
            J.rows = rows;
            J.wgs = want;
        }
        for (size_t q = 0; q < taken.size(); ++q) {
            ChipJob &J = jobs[L.at + q];
            const double z = (double)sizes[q], e = z - J.steps;
            J.base = L.wgs;
            L.wgs += J.wgs;
            ++L.jobs;
            L.flops += 2.0 * (z * z * z - e * e * e);      // three multiplications and additions per element of the trailing matrix and column
            L.bytes += 4.0 * (z * z + e * e);
            left[taken[q]].k += J.steps;
            ++left[taken[q]].turn;
        }
        launches.push_back(L);
        left.erase(std::remove_if(left.begin(), left.end(), [&](const ChipFactor &f) { return size(f) <= 0; }), left.end());
    }
}
