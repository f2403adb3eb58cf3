// Householder reduction to tridiagonal form with the trailing matrix held in the registers of the whole chip (part of eig_direct.hip:
// included there, in its namespace, after DirMat).
//
// A column of the reduction needs the product of the whole trailing matrix with one vector, and the next column needs that product.
// Read from memory the matrix costs 4 n^2 / 2 bytes a column (8 us of a 4609-wide factor at 5 TB/s) and a launch or two on top.  The 256
// compute units' registers hold 128 MB, a 4609-wide factor is 85: so each workgroup keeps a few rows of it for good, and what is left
// per column is one all-gather of the products between the workgroups of a factor.
//
//  - Workgroup p has rows [p R, p R + R) of the trailing matrix, thread i of it columns i, i + 512, .. of all R rows (S <= 9 column
//    slots; R S <= 162 registers of a thread's 256).  The column x that is being reduced lies in registers the same way, in every
//    workgroup of the factor alike, so norms and inner products are formed by each for itself, in the same order.
//  - Per column: products of the own rows with x (summed over the waves through LDS), published with the own rows' elements of the next
//    column as one 8-byte word per row; then the words of all rows are gathered.  The word itself says whether it is there: the
//    slots hold EMPTY before.  Everything after that is local: reflector, w, the next column, and ONE pass over the registers that
//    applies the rank-2 update and forms the next products.
//  - The words go through a ring of four columns.  A workgroup that has gathered column t knows that all have gathered t - 1, so it
//    empties its own words of t - 1 then; the s_waitcnt before its next publication orders the two, and the words are looked at again
//    only by who has seen that publication.  Loads and stores are relaxed agent-scope atomics of 8 bytes.
//  - Polling too early costs more than it gains (the line is fetched empty, and the writer has to take it away again): measured between
//    256 workgroups, 4608 words: 3.0 us a column polling at once, 2.3 after a pause of 1024 cycles; 64 workgroups: 2.3 and 1.5.
//
// Measured (one factor, whole decomposition): 577 wide 5.2 -> 2.6 ms, 2049 19.3 -> 10.2, 4609 57.6 -> 32.9; a column of a 4609-wide factor takes
// 5.0 us at its beginning (2.6 of them arithmetic) and 2.6 at its end, where the chain of launches took 13 and 7.
//
// A launch takes every factor some columns further (ChipJob), then the trailing matrices go back to memory and are dealt out anew:
// a matrix that has shrunk needs fewer workgroups, and others take their place.  All workgroups of a launch must be resident at once
// (cooperative launch, one per compute unit).  Every wait is bounded; a reduction that gave up leaves a matrix
// T that is not the factor's, which the measured residual shows, and the factor is decomposed by Jacobi iteration like any unsound one.

constexpr int CHIP_NT = 512, CHIP_WAVES = CHIP_NT / 64;
constexpr int CHIP_SLOTS = 9;
constexpr int CHIP_MAX_N = CHIP_NT * CHIP_SLOTS + 1;      // the widest factor: its first column is never part of the trailing matrix
constexpr int CHIP_ROWS = 64;                             // rows of a workgroup, at most: the lanes of the wave that publishes
constexpr int CHIP_JOBS = 64;                             // factors of a launch, at most: a workgroup finds its own by one ballot
constexpr int CHIP_PAUSE_MANY = 12, CHIP_PAUSE_FEW = 6;  // of 64 cycles, before the first look at the others' words (more than 96 workgroups, or fewer)
constexpr int CHIP_WHOLE = 640, CHIP_STEPS_MIN = 96;      // up to here a factor goes in one launch; the fewest columns of a launch otherwise
constexpr int CHIP_SPIN = 1 << 21;                        // polls (0.5 to 1 us each) before a wait is given up

// Rows that a workgroup of S column slots can hold, and rows per piece of its pass: the sums of a piece are in registers together, and
// a workgroup has whole pieces.
constexpr int chip_piece(int S) { return S == 9 ? 9 : 8; }
constexpr int chip_rows(int S) { return S == 9 ? 18 : S >= 7 ? 16 : S == 6 ? 24 : S == 5 ? 32 : S == 4 ? 40 : S == 3 ? 48 : 64; }

struct ChipJob {
    int m;               // factor
    int k0, steps;       // columns k0 .. k0 + steps - 1
    int rows, wgs, base; // rows per workgroup, workgroups, the first of them
    int slots;           // column slots
    int turn;            // launches of this factor before this one; its parity says which half of the ring buffer (the other is emptied for the next)
};

struct ChipSmem {
    float xs[CHIP_NT * CHIP_SLOTS + CHIP_ROWS], ys[CHIP_NT * CHIP_SLOTS + CHIP_ROWS];     // x and y by row, for those that need single elements
    float col[CHIP_ROWS], part[CHIP_WAVES][CHIP_ROWS], nrm[CHIP_WAVES], dot[CHIP_WAVES];
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

// (all of it through global pointers: a flat access also counts on the LDS counter, and every wait for LDS behind it takes a trip to memory)
typedef global_ptr<unsigned long long> ChipRing;
__device__ inline unsigned long long chip_load(ChipRing p) { return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }
__device__ inline void chip_store(ChipRing p, unsigned long long v) { __hip_atomic_store(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT); }

template <int S>
__device__ inline void chip_reduce(const DirMat &M, const ChipJob &J, int p, ChipSmem &sm) {
    constexpr int R = chip_rows(S), CH = chip_piece(S), PIECES = R / CH;
    static_assert(R % CH == 0 && R <= CHIP_ROWS, "whole pieces");
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int m = M.n - 1 - J.k0, r0 = p * J.rows, nr = min(J.rows, m - r0);     // nr >= 1: the last workgroup has row m - 1
    const bool last = p == J.wgs - 1, tail = tid + CHIP_NT * (S - 1) < m;        // only the last column slot reaches past the matrix
    const int64_t ld = M.ld;
    const global_ptr<float> A0 = as_global(M.A) + (int64_t)J.k0 * ld + J.k0 + 1;      // row k0, from the element beside the diagonal on
    const ChipRing ring = as_global((unsigned long long *)M.apan) + (size_t)(J.turn & 1) * CHIP_RING * M.np;
    const global_ptr<double> Md = as_global(M.d), Me = as_global(M.e);
    const global_ptr<float> Mtau = as_global(M.tau);
    float a[R][S], x[S], v[S], w[S], s2 = 0.f;
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
        for (int j = 0; j < S - 1; ++j) a[i][j] = row[CHIP_NT * j];
        a[i][S - 1] = 0.f;
    }
    if (tail)
#pragma unroll
        for (int i = 0; i < R; ++i) a[i][S - 1] = A0[(int64_t)(1 + r0 + min(i, nr - 1)) * ld + tid + CHIP_NT * (S - 1)];
    if (J.turn == 0 && last && tid == 0) Md[J.k0] = (double)A0[-1];
    if (tid < nr) {
        const ChipRing other = as_global((unsigned long long *)M.apan) + (size_t)(~J.turn & 1) * CHIP_RING * M.np + r0 + tid;
#pragma unroll
        for (int q = 0; q < CHIP_RING; ++q) other[(size_t)q * M.np] = CHIP_EMPTY;
    }
    if (tid == 0) sm.failed = 0;
    float nv = 0.f, nw = 0.f;       // lane i: -v and -w of row r0 + i
    for (int t = 0;; ++t) {
        // x: column k0 + t, rows t .. m - 1 of the trailing matrix (zero before).  v, w: the reflector before it, not yet applied.
        // s2: this thread's share of the squared norm below the column's first element.
        s2 = wave_sum_all(s2);
        if (lane == 0) sm.nrm[wave] = s2;
        // A <- A - v w^T - w v^T and A x in one pass; rows and columns before t are finished
        const int j0 = max(0, (t - 64 * wave - 63 + CHIP_NT - 1) / CHIP_NT);
#pragma unroll
        for (int q = 0; q < PIECES; ++q) {
            if (q * CH >= nr || r0 + q * CH + CH <= t) continue;
            float acc[CH], rv[CH], rw[CH];
#pragma unroll
            for (int i = 0; i < CH; ++i) {
                acc[i] = 0.f;
                rv[i] = lane_value(nv, q * CH + i);
                rw[i] = lane_value(nw, q * CH + i);
            }
#pragma unroll
            for (int j = 0; j < S; ++j) {
                if (j < j0) continue;
#pragma unroll
                for (int i = 0; i < CH; ++i) {
                    float &e = a[q * CH + i][j];
                    e = fmaf(rv[i], w[j], fmaf(rw[i], v[j], e));
                    acc[i] = fmaf(e, x[j], acc[i]);
                }
            }
            const float sum = chip_fold<CH>(acc, lane);
            const int at = chip_fold_index<CH>(lane);
            if (at < CH) sm.part[wave][q * CH + at] = sum;
        }
        if (t == J.steps) break;
        if (r0 + nr <= t) return;          // all rows of this workgroup are finished
        if (wave == ((t >> 6) & (CHIP_WAVES - 1))) {      // the own rows' elements of column t, by the lane that has it
#pragma unroll
            for (int j = 0; j < S; ++j)
                if (j == t / CHIP_NT)
#pragma unroll
                    for (int q = 0; q < PIECES; ++q)
                        if (q * CH < nr && lane == (t & 63))
#pragma unroll
                            for (int i = q * CH; i < q * CH + CH; ++i) sm.col[i] = a[i][j];
        }
        __syncthreads();
        const ChipRing slot = ring + (size_t)(t & (CHIP_RING - 1)) * M.np;
        const int r = r0 + lane, k = J.k0 + t;
        float art = 0.f;
        if (tid < nr) {
            float y = 0.f;
            art = sm.col[tid];
#pragma unroll
            for (int g = 0; g < CHIP_WAVES; ++g) y += sm.part[g][tid];
            unsigned long long word = (unsigned long long)__float_as_uint(y) | (unsigned long long)__float_as_uint(art) << 32;
            if (word == CHIP_EMPTY) word = 0x7fc000007fc00000ull;      // two NaNs that look like an empty slot
            asm volatile("s_waitcnt vmcnt(0)" ::: "memory");           // what was emptied for column t - 1 is empty
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
        if (J.wgs > 96) __builtin_amdgcn_s_sleep(CHIP_PAUSE_MANY);
        else __builtin_amdgcn_s_sleep(CHIP_PAUSE_FEW);
        unsigned long long u[S];
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const int c = tid + CHIP_NT * j;
            u[j] = 0;
            if (c >= t && (j < S - 1 || tail)) u[j] = chip_load(slot + c);
        }
        for (int spin = 0;; ++spin) {
            bool there = true;
#pragma unroll
            for (int j = 0; j < S; ++j)
                if (u[j] == CHIP_EMPTY) {
                    there = false;
                    u[j] = chip_load(slot + tid + CHIP_NT * j);
                }
            if (__all(there)) break;
            if (spin > CHIP_SPIN) { sm.failed = 1; break; }
        }
        float dot = 0.f;
#pragma unroll
        for (int j = 0; j < S; ++j) {
            if (j < j0) continue;
            const int c = tid + CHIP_NT * j;
            const float ac = __uint_as_float((unsigned)(u[j] >> 32));
            w[j] = scale * fmaf(-beta, ac, __uint_as_float((unsigned)u[j]));      // y; w = tau y + cw v follows once the inner product is known
            v[j] = c == t ? 1.f : x[j] * scale;
            x[j] = ac;
            sm.ys[c] = w[j];
            dot = fmaf(v[j], w[j], dot);
        }
        dot = wave_sum_all(dot);
        if (lane == 0) sm.dot[wave] = dot;
        __syncthreads();
        const float yt = sm.ys[t], yr = sm.ys[r];
        const int failed = sm.failed;
        dot = 0.f;
#pragma unroll
        for (int g = 0; g < CHIP_WAVES; ++g) dot += sm.dot[g];
        if (failed) return;                // the result is not sound, and is found not to be
        const float cw = -0.5f * tau * tau * dot, wt = fmaf(tau, yt, cw);
        const float vr = lane < nr && r >= t ? (r == t ? 1.f : xr * scale) : 0.f;
        nv = -vr;
        nw = lane < nr && r >= t ? -fmaf(tau, yr, cw * vr) : 0.f;
        s2 = 0.f;
#pragma unroll
        for (int j = 0; j < S; ++j) {
            if (j < j0) continue;
            const int c = tid + CHIP_NT * j;
            w[j] = fmaf(tau, w[j], cw * v[j]);
            x[j] = c > t ? x[j] - fmaf(v[j], wt, w[j]) : 0.f;
            sm.xs[c] = x[j];
            s2 = fmaf(x[j], c == t + 1 ? 0.f : x[j], s2);
        }
        if (wave == CHIP_WAVES - 1 && lane < nr) A0[(int64_t)t * ld + r] = vr;     // row k: everybody has published, so has read it
        if (tid < nr && r == t) Md[k + 1] = (double)(art - 2.f * wt);
        // all have published t, so all have gathered t - 1
        if (t >= 1 && tid < nr) chip_store(ring + (size_t)((t - 1) & (CHIP_RING - 1)) * M.np + r0 + tid, CHIP_EMPTY);
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
            if (tid + CHIP_NT * j >= T && (j < S - 1 || tail)) row[CHIP_NT * j] = a[i][j];
    }
    if (last)
#pragma unroll
        for (int j = 0; j < S; ++j) {
            const int c = tid + CHIP_NT * j;
            if (c >= T && (j < S - 1 || tail)) A0[(int64_t)T * ld + c] = x[j];
        }
}

__global__ __launch_bounds__(CHIP_NT, 2) void dir_chip_kernel(const DirMat *mats, const ChipJob *jobs, int count) {
    __shared__ ChipSmem sm;
    const int lane = threadIdx.x & 63;
    const int base = lane < count ? jobs[lane].base : INT_MAX;      // ascending
    const ChipJob J = jobs[__popcll(__ballot(base <= (int)blockIdx.x)) - 1];
    const DirMat M = mats[J.m];
    const int p = (int)blockIdx.x - J.base;
    switch (J.slots) {
        case 1: chip_reduce<1>(M, J, p, sm); break;
        case 2: chip_reduce<2>(M, J, p, sm); break;
        case 3: chip_reduce<3>(M, J, p, sm); break;
        case 4: chip_reduce<4>(M, J, p, sm); break;
        case 5: chip_reduce<5>(M, J, p, sm); break;
        case 6: chip_reduce<6>(M, J, p, sm); break;
        case 7: chip_reduce<7>(M, J, p, sm); break;
        case 8: chip_reduce<8>(M, J, p, sm); break;
        default: chip_reduce<9>(M, J, p, sm); break;
    }
}

// ---- which factor takes how many columns further in which launch ----
struct ChipLaunch { unsigned at; int jobs, wgs; double flops, bytes; };     // at: index of its first job
struct ChipFactor { int m, n, k, turn; };                                  // width n, k columns reduced

inline int chip_slots(int size) { return (size + CHIP_NT - 1) / CHIP_NT; }
inline int chip_need(int size) {      // workgroups that hold a trailing matrix of this size
    const int rows = chip_rows(chip_slots(size));
    return (size + rows - 1) / rows;
}
inline int chip_widest(int capacity) {      // widest factor that fits (0: none does)
    int n = CHIP_MAX_N;
    while (n > 1 && chip_need(n - 1) > capacity) --n;
    return n > 1 ? n : 0;
}

// The widest factors that are left come first; narrower ones fill what they leave free.
inline void chip_plan(std::vector<ChipFactor> left, int capacity, std::vector<ChipJob> &jobs, std::vector<ChipLaunch> &launches) {
    auto size = [](const ChipFactor &f) { return f.n - 1 - f.k; };
    while (!left.empty()) {
        std::stable_sort(left.begin(), left.end(), [&](const ChipFactor &a, const ChipFactor &b) { return size(a) > size(b); });
        const int widest = size(left[0]);
        // dealing a matrix out anew costs its bytes and a launch, some 50 us for the widest: a sixth of its columns take 40 times that
        const int steps = widest <= CHIP_WHOLE ? widest : std::max(CHIP_STEPS_MIN, widest / 6);
        ChipLaunch L{(unsigned)jobs.size(), 0, 0, 0.0, 0.0};
        int free = capacity;
        std::vector<size_t> taken, sizes;
        for (size_t q = 0; q < left.size() && taken.size() < CHIP_JOBS; ++q) {
            const int z = size(left[q]), need = chip_need(z);
            if (need > free) continue;
            free -= need;
            taken.push_back(q);
            sizes.push_back(z);
            jobs.push_back(ChipJob{left[q].m, left[q].k, std::min(steps, z), chip_rows(chip_slots(z)), need, 0, chip_slots(z), left[q].turn});
        }
        // what is free goes to those that do the most per workgroup, a piece less each time
        for (;;) {
            int most = -1;
            for (size_t q = 0; q < taken.size(); ++q) {
                const ChipJob &J = jobs[L.at + q];
                if (J.rows > chip_piece(J.slots) && (most < 0 || J.rows * J.slots > jobs[L.at + most].rows * jobs[L.at + most].slots)) most = (int)q;
            }
            if (most < 0) break;
            ChipJob &J = jobs[L.at + most];
            const int rows = J.rows - chip_piece(J.slots), want = ((int)sizes[most] + rows - 1) / rows;
            if (want - J.wgs > free) break;
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
