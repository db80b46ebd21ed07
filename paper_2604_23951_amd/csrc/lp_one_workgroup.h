// One-workgroup solver: the whole restarted PDHG loop of an LP in one workgroup. Included by
// lp_kernels.hip (inside its namespace) after the epilogues and the evaluation.
//
// What bounds it: these LPs move little data, so an iteration is two dependent chains
// (gather, row sum, update) with a barrier after each, and the time is the latency of the
// accesses on those chains. So a row is summed by one thread, straight from the gathered
// values (no products staged in LDS, one barrier per half-iteration instead of two), the two
// vectors that are gathered live in LDS, and each thread keeps the operands of the rows and
// columns it owns in registers for a whole evaluation period. The matrices are stored as
// slices of 64 rows, two consecutive entries of a row per slot (Sell): a wave reads one slot
// of its 64 rows with consecutive addresses, 4 bytes of columns and 16 (FP32: 8) of values
// per lane. With 256 and 512 threads the first kSoloRegSlots slots of a thread's row and
// column stay in registers; other slots come from LDS, for the slices that fit, or the L2. Rows
// are dealt to slices longest first, so that a slice pads little and the longest chains are
// the ones in LDS. Padding is zero entries whose column is a zero slot behind the gathered
// vector, so the loop has no lane predicates; a row sum is the products added in CSR order,
// and adding +0 or -0 to a sum that starts at +0 changes nothing: bit-identical to the
// row-tile kernels.
//
// Measured (us per iteration, evaluations every 64 iterations included, FP64 Halpern form),
// row tiles staged in LDS or, above the budget, from global memory / this solver: 50 x 100
// 4.5 / 0.84, 200 x 400 5.5 / 1.2, 601 x 1202 transportation (kernel per phase 11.7) / 1.75,
// 330 x 660 with 11,047 entries 23 / 3.6; 64 LPs of 50 to 900 rows in FP32 77 / 16 (the slowest).
//
// The evaluation runs on the arrays in global memory with the same terms, split over the
// 256-thread groups of the workgroup by quantity; every sum keeps the order of the
// 256-thread kernels (nblk virtual blocks of them).

constexpr int kSoloEvalBlocks = 16;  // virtual reduction blocks at most
static_assert(kSoloMaxDim <= kSoloEvalBlocks * 1024, "every admitted LP's reduction grid fits");
constexpr int kSoloWeights = 64;  // iteration weights computed together, one per thread
constexpr int kSoloRegSlots = 8;

struct SoloShared {
    Scalars sc;
    double red[(kBlock / 64) * kNT];
    double part[kSoloEvalBlocks * kNT];
    double tot[kNT];
    double weight[kSoloWeights];
    int job;
};

// The one instance of it, known to be LDS wherever it is used.
__device__ __forceinline__ SoloShared& solo_shared() {
    __shared__ SoloShared S;
    return S;
}

// LDS offsets of one LP: the gathered vectors (y, then the primal point; together also the
// FP64 vector of an evaluation product), then the staged slots of A and of A^T.
struct SoloLds {
    int xs, a_col, a_val, at_col, at_val, end;
};

__host__ __device__ inline SoloLds solo_lds_layout(int m, int n, int fp32, int a_slots, int at_slots) {
    const int sv = fp32 ? 4 : 8;
    auto up = [](int b) { return (b + 15) & ~15; };
    SoloLds L;
    L.xs = up(sv * (m + 1));
    int off = L.xs + up(sv * (n + 1));
    const int eval = up(8 * ((m > n ? m : n) + 1));
    if (off < eval) off = eval;
    L.a_col = off;
    L.a_val = L.a_col + 4 * a_slots;
    L.at_col = L.a_val + 2 * sv * a_slots;
    L.at_val = L.at_col + 4 * at_slots;
    L.end = L.at_val + 2 * sv * at_slots;
    return L;
}

template <class T>
struct Pair;
template <>
struct Pair<double> { using type = double2; };
template <>
struct Pair<float> { using type = float2; };

template <class T>
__device__ inline const T* sell_vals(const Sell& S);
template <>
__device__ inline const double* sell_vals<double>(const Sell& S) { return S.v; }
template <>
__device__ inline const float* sell_vals<float>(const Sell& S) { return S.v32; }

// Where a Sell matrix is read from: its slices below `staged` from LDS (byte offsets of the
// columns and values), the others from global memory.
struct SellAt {
    const unsigned* col;
    const void* val;
    int col_off, val_off;
    int staged;
    int limit;  // columns + 1 (the zero slot): the checked build's bound
    int staged_slots, slots;  // bounds of a slot number in LDS and in global memory (checked build)
};

template <class T, int C>
struct SellChunk {
    using V = typename Pair<T>::type;
    unsigned c[C];
    V v[C];
};

// LC: the columns are staged, LV: the values are.
template <class T, int C, bool LC, bool LV>
__device__ __forceinline__ SellChunk<T, C> sell_load(int slot, const SellAt& M, const char* lds) {
    using V = typename Pair<T>::type;
    SellChunk<T, C> K;
#pragma unroll
    for (int k = 0; k < C; ++k) {
        const int at = checked_index(slot + 64 * k, LC ? M.staged_slots : M.slots, 16u);
        if constexpr (LC) K.c[k] = *reinterpret_cast<const unsigned*>(lds + M.col_off + 4 * at);
        else K.c[k] = M.col[at];
        if constexpr (LV) K.v[k] = *reinterpret_cast<const V*>(lds + M.val_off + static_cast<int>(sizeof(V)) * at);
        else K.v[k] = static_cast<const V*>(M.val)[at];
    }
    return K;
}

// The first D of a chunk's C slots (2 D entries of one row) added to s in order; `gat` is the
// LDS vector gathered from.
template <class T, int D, int C>
__device__ __forceinline__ T sell_add(T s, const SellChunk<T, C>& K, int limit, const T* gat) {
    T g0[D], g1[D];
#pragma unroll
    for (int k = 0; k < D; ++k) {
        g0[k] = gat[checked_index(K.c[k] & 0xffffu, limit, 4u)];
        g1[k] = gat[checked_index(K.c[k] >> 16, limit, 4u)];
    }
#pragma unroll
    for (int k = 0; k < D; ++k) {
        s += K.v[k].x * g0[k];
        s += K.v[k].y * g1[k];
    }
    return s;
}

// Slots slot, slot + 64, ... (width of them) of one row added to s; the next four are loaded
// while the current four are gathered and added.
template <class T, bool LC, bool LV>
__device__ __forceinline__ T sell_slots(T s, int slot, int width, const SellAt& M, const char* lds, const T* gat) {
    if (width >= 4) {
        SellChunk<T, 4> K = sell_load<T, 4, LC, LV>(slot, M, lds);
        for (; width >= 8; width -= 4) {
            slot += 256;
            const SellChunk<T, 4> N = sell_load<T, 4, LC, LV>(slot, M, lds);
            s = sell_add<T, 4>(s, K, M.limit, gat);
            K = N;
        }
        s = sell_add<T, 4>(s, K, M.limit, gat);
        slot += 256;
        width -= 4;
    }
    if (width & 2) {
        s = sell_add<T, 2>(s, sell_load<T, 2, LC, LV>(slot, M, lds), M.limit, gat);
        slot += 128;
    }
    if (width & 1) s = sell_add<T, 1>(s, sell_load<T, 1, LC, LV>(slot, M, lds), M.limit, gat);
    return s;
}

// One row sum of slice sl (base: the lane's first slot).
template <class T>
__device__ __forceinline__ T sell_row(T s, int sl, int slot, int width, const SellAt& M, const char* lds, const T* gat) {
    if (sl < M.staged) return sell_slots<T, true, true>(s, slot, width, M, lds, gat);
    return sell_slots<T, false, false>(s, slot, width, M, lds, gat);
}

// out = M xin in FP64 (the products of an evaluation); LV: the staged values are FP64 ones.
// Ends with a barrier.
template <int NT, bool LV>
__device__ __forceinline__ void solo_product(const Sell& S, const SellAt& M, int rows, int cols, const double* xin, double* out) {
    extern __shared__ __align__(16) char solo_lds[];
    double* gat = reinterpret_cast<double*>(solo_lds);
    const int tid = threadIdx.x, lane = tid & 63;
    for (int i = tid; i < cols; i += NT) gat[i] = xin[i];
    if (tid == 0) gat[cols] = 0.0;
    __syncthreads();
    for (int sl = __builtin_amdgcn_readfirstlane(tid >> 6); sl < S.slices; sl += NT / 64) {
        const int base = S.ptr[sl], width = (S.ptr[sl + 1] - base) >> 6;
        const int r = S.row[sl * 64 + lane];
        double s = 0.0;
        if (sl < M.staged) s = sell_slots<double, true, LV>(s, base + lane, width, M, solo_lds, gat);
        else s = sell_slots<double, false, false>(s, base + lane, width, M, solo_lds, gat);
        if (r < rows) out[r] = s;
    }
    __syncthreads();
}

// One quantity set of an evaluation over rows and columns start, start + stride, ... (see
// eval_terms for the candidates): 0 the current point's terms, 1 the average's, 2 and 3 the
// two rays, 4 the residual restarts. Returns the number of quantities and their first slot.
__device__ inline int eval_set(const DevLP& P, int mode, int set, int start, int stride, double* acc, int* first) {
    const bool both = mode == 0 && !P.method;
    const bool cand = (mode == 0 || mode == 2) && P.method;
    const bool rays = mode == 0 && P.xp != nullptr;
    const double* ex = cand ? P.xa : P.x;
    const double* ey = cand ? P.ya : P.y;
    const double* eax = cand ? P.axa : P.ax;
    const double* eaty = cand ? P.atya : P.aty;
    if (set <= 1) {
        *first = set * kNQ;
        if (set == 1 && !both) return kNQ;
        const double *tx = set ? P.xa : ex, *ty = set ? P.ya : ey, *tax = set ? P.axa : eax, *taty = set ? P.atya : eaty;
        for (int i = start; i < P.m; i += stride) row_terms(P, i, tax, ty, acc);
        for (int j = start; j < P.n; j += stride) col_terms(P, j, tx, taty, acc);
        return kNQ;
    }
    if (set <= 3) {
        *first = 2 * kNQ + 4 * (set - 2);
        if (!rays) return 4;
        const bool anch = set == 3;
        const double *ty = anch ? P.ya : ey, *tax = anch ? P.axa : eax, *tx = anch ? P.xa : ex, *taty = anch ? P.atya : eaty;
        const double *by = anch ? P.yan : P.yp, *bax = anch ? P.axan : P.axp, *bx = anch ? P.xan : P.xp, *baty = anch ? P.atyan : P.atyp;
        for (int i = start; i < P.m; i += stride) row_ray_terms(P, i, ty, tax, by, bax, acc);
        for (int j = start; j < P.n; j += stride) col_ray_terms(P, j, tx, taty, bx, baty, acc);
        return 4;
    }
    *first = kNT - kNF;
    if (mode == 0 && residual_restarts(P)) residual_terms(P, start, stride, acc);
    return kNF;
}

// The evaluation's sums into S.tot, in the order of nblk blocks of kBlock threads. One group
// of threads takes every quantity in one pass over the rows and columns (the candidates share
// their loads); several groups share out the quantity sets.
template <int NT>
__device__ __forceinline__ void solo_kkt(const DevLP& P, int mode, int nblk) {
    SoloShared& S = solo_shared();
    constexpr int kGroups = NT / kBlock, kWaves = kBlock / 64, kMain = kNT - kNF;
    const int group = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kBlock);
    const int vt = threadIdx.x % kBlock, lane = vt & 63, w = vt >> 6;
    for (int blk = 0; blk < nblk; ++blk) {
        const int start = blk * kBlock + vt, stride = nblk * kBlock;
        if constexpr (kGroups == 1) {
            double acc[kMain];
#pragma unroll
            for (int q = 0; q < kMain; ++q) acc[q] = 0.0;
            eval_terms(P, mode, start, stride, acc);
#pragma unroll
            for (int q = 0; q < kMain; ++q) {
                const double v = wave_sum(acc[q]);
                if (lane == 0) S.red[w * kNT + q] = v;
            }
        }
        for (int set = kGroups == 1 ? 4 : group; set < 5; set += kGroups) {
            double acc[kNQ] = {0, 0, 0, 0, 0, 0, 0, 0};
            int first = 0;
            const int nq = eval_set(P, mode, set, start, stride, acc, &first);
#pragma unroll
            for (int q = 0; q < kNQ; ++q) {
                const double v = wave_sum(acc[q]);
                if (lane == 0 && q < nq) S.red[w * kNT + first + q] = v;
            }
        }
        __syncthreads();
        if (threadIdx.x < kNT) {
            double t = 0.0;
            for (int k = 0; k < kWaves; ++k) t += S.red[k * kNT + threadIdx.x];
            S.part[blk * kNT + threadIdx.x] = t;
        }
        __syncthreads();
    }
    if (nblk == 1) {
        if (threadIdx.x < kNT) S.tot[threadIdx.x] = S.part[threadIdx.x];
    } else {  // decide_body's sum over the blocks: lane b holds block b's partial
        const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x >> 6));
        for (int q = wave; q < kNT; q += NT / 64) {
            const int b = threadIdx.x & 63;
            const double v = wave_sum(b < nblk ? S.part[b * kNT + q] : 0.0);
            if (b == 0) S.tot[q] = v;
        }
    }
    __syncthreads();
}

template <int FORM>
__device__ inline auto solo_primal(const DevLP& P) {
    if constexpr (FORM == 0) return epi_primal(P, P.sc, 0);
    else if constexpr (FORM == 1) return epi_primal_h(P, P.sc, 0);
    else if constexpr (FORM == 2) return epi_primal32(P, P.sc, 0);
    else return epi_primal32_h(P, P.sc, 0);
}
template <int FORM>
__device__ inline auto solo_dual(const DevLP& P) {
    if constexpr (FORM == 0) return epi_dual(P, P.sc, 0);
    else if constexpr (FORM == 1) return epi_dual_h(P, P.sc, 0);
    else if constexpr (FORM == 2) return epi_dual32(P, P.sc, 0);
    else return epi_dual32_h(P, P.sc, 0);
}

// The slices a thread works on, K of them, NT / 64 apart: first slot and width (uniform over
// the wave; width -1: no such slice) and, for sorted slices, the lane's row.
template <int NT, int K, bool SORTED>
struct SoloSlices {
    int base[K], width[K], row[SORTED ? K : 1];
    __device__ __forceinline__ void load(const Sell& S, int wave, int lane) {
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const int sl = wave + k * (NT / 64);
            const bool any = sl < S.slices;
            base[k] = any ? S.ptr[sl] : 0;
            width[k] = any ? (S.ptr[sl + 1] - base[k]) >> 6 : -1;
            if constexpr (SORTED) row[k] = any ? S.row[sl * 64 + lane] : 0x7fffffff;
        }
    }
    __device__ __forceinline__ int row_of(int k, int wave, int lane) const {
        if constexpr (SORTED) return row[k];
        else return (wave + k * (NT / 64)) * 64 + lane;
    }
};

// A row's first kSoloRegSlots slots in registers and its sum: with few waves per CU nothing
// hides the LDS latency of the columns, so they are not read again at every iteration.
template <class T>
struct SoloRegRow {
    SellChunk<T, kSoloRegSlots> K;
    __device__ __forceinline__ void load(int slot, int width, const SellAt& M, const char* lds) {
#pragma unroll
        for (int k = 0; k < kSoloRegSlots; ++k) {
            const unsigned zero = static_cast<unsigned>(M.limit - 1);
            K.c[k] = zero | (zero << 16);
            K.v[k].x = K.v[k].y = 0;
            if (k < width) {  // (a slice without entries has no slot to read)
                const SellChunk<T, 1> one = sell_load<T, 1, true, true>(slot + 64 * k, M, lds);
                K.c[k] = one.c[0];
                K.v[k] = one.v[0];
            }
        }
    }
    __device__ __forceinline__ T sum(int slot, int width, const SellAt& M, const char* lds, const T* gat) const {
        T s = 0;
        if (width <= 2) return sell_add<T, 2>(s, K, M.limit, gat);
        if (width <= 4) return sell_add<T, 4>(s, K, M.limit, gat);
        if (width <= 6) return sell_add<T, 6>(s, K, M.limit, gat);
        s = sell_add<T, 8>(s, K, M.limit, gat);
        if (width <= kSoloRegSlots) return s;
        return sell_slots<T, true, true>(s, slot + 64 * kSoloRegSlots, width - kSoloRegSlots, M, lds, gat);
    }
};

// `steps` iterations from the state in global memory and back to it. KC columns and KR rows
// per thread are held in registers (KC = 0: every operand is read and written in global
// memory at every iteration). Every thread calls it; ends with a barrier.
template <int FORM, int NT, int KC, int KR>
__device__ __forceinline__ void solo_period(const BatchJob& J, int steps) {
    extern __shared__ __align__(16) char solo_lds[];
    if (steps <= 0) return;
    SoloShared& S = solo_shared();
    const DevLP& P = J.P;
    auto ep = solo_primal<FORM>(P);
    auto ed = solo_dual<FORM>(P);
    using T = typename decltype(ep)::T;
    constexpr bool kHalpern = (FORM & 1) != 0, kRegs = NT < 1024;
    const SoloLds L = solo_lds_layout(P.m, P.n, FORM >= 2, J.a_slots, J.at_slots);
    T* ys = reinterpret_cast<T*>(solo_lds);
    T* xs = reinterpret_cast<T*>(solo_lds + L.xs);
    const int m = P.m, n = P.n;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const SellAt A{P.sA.col, sell_vals<T>(P.sA), L.a_col, L.a_val, J.a_slices, n + 1, J.a_slots, P.sA.slots};
    const SellAt AT{P.sAT.col, sell_vals<T>(P.sAT), L.at_col, L.at_val, J.at_slices, m + 1, J.at_slots, P.sAT.slots};
    const double tau = S.sc.tau, sigma = S.sc.sigma;
    const long long t0 = S.sc.t;
    const bool resid = kHalpern && P.restart_metric == 1;
    auto weights = [&](int it) {  // of iterations it, it + 1, ...: one division per thread
        if (tid < kSoloWeights) S.weight[tid] = decltype(ep)::weight(t0 + it + tid);
    };
    auto scalars = [&](int it) {
        const double w = S.weight[it % kSoloWeights];
        ep.set_weight(tau, w, t0 + it);
        ed.set_weight(sigma, w, t0 + it);
        if constexpr (kHalpern) {
            ep.set_record(it == steps - 1, t0 + it);
            ed.set_record(it == steps - 1, t0 + it);
        }
    };
    weights(0);
    if (tid == 0) {
        ys[m] = 0;
        xs[n] = 0;
    }
    if constexpr (KC > 0) {
        typename decltype(ep)::Pre pc[KC];
        typename decltype(ed)::Pre pr[KR];
        constexpr bool kSorted = KC <= 2;
        SoloSlices<NT, KC, kSorted> C;
        SoloSlices<NT, KR, kSorted> R;
        C.load(P.sAT, wave, lane);
        R.load(P.sA, wave, lane);
        SoloRegRow<T> rc, rr;
        if constexpr (kRegs) {
            static_assert(KC == 1 && KR == 1, "one row and one column per thread");
            rc.load(C.base[0] + lane, C.width[0], AT, solo_lds);
            rr.load(R.base[0] + lane, R.width[0], A, solo_lds);
        }
#pragma unroll
        for (int k = 0; k < KC; ++k) pc[k] = ep.load(min(C.row_of(k, wave, lane), n - 1));
#pragma unroll
        for (int k = 0; k < KR; ++k) {
            const int i = R.row_of(k, wave, lane);
            pr[k] = ed.load(min(i, m - 1));
            if (i < m) ys[i] = pr[k].y;
        }
        __syncthreads();
        for (int it = 0; it < steps; ++it) {
            const bool last = it == steps - 1;
            scalars(it);
            // Addresses are formed again at every iteration: hoisted out of the loop, those of
            // several rows per thread take the registers that the operands need.
            int ln = lane;
            if constexpr (!kRegs) asm volatile("" : "+v"(ln));
#pragma unroll
            for (int k = 0; k < KC; ++k) {
                if (C.width[k] >= 0) {
                    const int j = C.row_of(k, wave, ln);
                    T s;
                    if constexpr (kRegs) s = rc.sum(C.base[k] + ln, C.width[k], AT, solo_lds, ys);
                    else s = sell_row<T>(T(0), wave + k * (NT / 64), C.base[k] + ln, C.width[k], AT, solo_lds, ys);
                    const auto q = pc[k];
                    const T g = ep.step(pc[k], s);
                    if (j < n) {
                        xs[j] = g;
                        if (last) ep.store(j, pc[k]);
                        if constexpr (kHalpern)
                            if (resid) ep.record(j, q, pc[k], s);
                    }
                }
            }
            __syncthreads();
            if constexpr (!kRegs) asm volatile("" : "+v"(ln));
#pragma unroll
            for (int k = 0; k < KR; ++k) {
                if (R.width[k] >= 0) {
                    const int i = R.row_of(k, wave, ln);
                    T s;
                    if constexpr (kRegs) s = rr.sum(R.base[k] + ln, R.width[k], A, solo_lds, xs);
                    else s = sell_row<T>(T(0), wave + k * (NT / 64), R.base[k] + ln, R.width[k], A, solo_lds, xs);
                    const auto q = pr[k];
                    const T g = ed.step(pr[k], s);
                    if (i < m) {
                        ys[i] = g;
                        if (last) ed.store(i, pr[k]);
                        if constexpr (kHalpern)
                            if (resid) ed.record(i, q, pr[k], s);
                    }
                }
            }
            if ((it + 1) % kSoloWeights == 0) weights(it + 1);
            __syncthreads();
        }
    } else {
        for (int i = tid; i < m; i += NT) ys[i] = ed.y[i];
        __syncthreads();
        for (int it = 0; it < steps; ++it) {
            scalars(it);
            for (int sl = wave; sl < P.sAT.slices; sl += NT / 64) {
                const int base = P.sAT.ptr[sl], width = (P.sAT.ptr[sl + 1] - base) >> 6, j = P.sAT.row[sl * 64 + lane];
                auto p = ep.load(min(j, n - 1));
                const T s = sell_row<T>(T(0), sl, base + lane, width, AT, solo_lds, ys);
                if (j < n) {
                    const auto q = p;
                    xs[j] = ep.step(p, s);
                    ep.store(j, p);
                    if constexpr (kHalpern)
                        if (resid) ep.record(j, q, p, s);
                }
            }
            __syncthreads();
            for (int sl = wave; sl < P.sA.slices; sl += NT / 64) {
                const int base = P.sA.ptr[sl], width = (P.sA.ptr[sl + 1] - base) >> 6, i = P.sA.row[sl * 64 + lane];
                auto p = ed.load(min(i, m - 1));
                const T s = sell_row<T>(T(0), sl, base + lane, width, A, solo_lds, xs);
                if (i < m) {
                    const auto q = p;
                    ys[i] = ed.step(p, s);
                    ed.store(i, p);
                    if constexpr (kHalpern)
                        if (resid) ed.record(i, q, p, s);
                }
            }
            if ((it + 1) % kSoloWeights == 0) weights(it + 1);
            __syncthreads();
        }
    }
    __syncthreads();
}

template <int NT, class T>
__device__ inline void solo_stage(char* dst, const T* src, int bytes) {
    const int4* s4 = reinterpret_cast<const int4*>(src);  // slot counts are multiples of 64: whole 16-byte words
    int4* d4 = reinterpret_cast<int4*>(dst);
    for (int i = threadIdx.x; i < bytes / 16; i += NT) d4[i] = s4[i];
}

// The evaluation of the initial point (mode 1) or at a period's end (mode 0) and what follows
// from it: products, sums, decision, the point the next evaluation's rays start from, the
// restart. A call of its own: its registers stay apart from the iterations'.
template <int NT, bool FP32>
__device__ __noinline__ void solo_evaluate(const BatchJob& J, int mode) {
    SoloShared& S = solo_shared();
    const DevLP& P = J.P;
    const SoloLds L = solo_lds_layout(P.m, P.n, FP32, J.a_slots, J.at_slots);
    const int tid = threadIdx.x, m = P.m, n = P.n, mx = m > n ? m : n;
    const SellAt A{P.sA.col, P.sA.v, L.a_col, L.a_val, J.a_slices, n + 1, J.a_slots, P.sA.slots};
    const SellAt AT{P.sAT.col, P.sAT.v, L.at_col, L.at_val, J.at_slices, m + 1, J.at_slots, P.sAT.slots};
    const bool halpern = P.method != 0;
    if (FP32 && mode == 0) {
        for (int g = tid; g < mx; g += NT) materialize_at(P, g);
        __syncthreads();
    }
    // A~ x and A~^T y of the iterate, A~ xa and A~^T ya of the other candidate
    if (mode == 1 || (FP32 && !halpern)) solo_product<NT, !FP32>(P.sA, A, m, n, P.x, P.ax);
    if (mode == 1 || !halpern) solo_product<NT, !FP32>(P.sAT, AT, n, m, P.y, P.aty);
    if (mode == 0 && (!halpern || FP32)) solo_product<NT, !FP32>(P.sA, A, m, n, P.xa, P.axa);
    if (mode == 0) solo_product<NT, !FP32>(P.sAT, AT, n, m, P.ya, P.atya);
    solo_kkt<NT>(P, mode, J.eval_blocks);
    const bool late = mode == 0 && time_limit_passed<NT>(P, J, &S.sc, S.tot, S.red, S.part, kSoloEvalBlocks * kNT);
    if (tid == 0) decide_logic(P, &S.sc, S.tot, mode, late);
    __syncthreads();
    const bool running = S.sc.status == kRunning;
    const int lr = mode == 1 ? 1 : S.sc.last_restart;
    if (running) {
        for (int g = tid; g < mx; g += NT) save_prev_at(P, mode == 1 ? 0 : lr, mode == 1, g);
        __syncthreads();
    }
    if ((mode == 1 && FP32) || (mode == 0 && lr)) {
        for (int g = tid; g < mx; g += NT) {
            if (FP32) rebase_at(P, lr, g);
            else apply_restart_at(P, lr, g);
        }
        __syncthreads();
    }
}

// One LP from start to stop in one workgroup; the phases are those of wg_solve.
template <int FORM, int NT, int KC, int KR>
__device__ __forceinline__ void solo_solve(const BatchJob& J) {
    extern __shared__ __align__(16) char solo_lds[];
    SoloShared& S = solo_shared();
    const DevLP& P = J.P;
    constexpr bool kFp32 = FORM >= 2;
    using T = typename std::conditional<kFp32, float, double>::type;
    const SoloLds L = solo_lds_layout(P.m, P.n, kFp32, J.a_slots, J.at_slots);
    const int tid = threadIdx.x, mx = P.m > P.n ? P.m : P.n;
    if (tid == 0) {
        S.sc = *P.sc;
        reset_scalars(&S.sc, J);
    }
    solo_stage<NT>(solo_lds + L.a_col, P.sA.col, 4 * J.a_slots);
    solo_stage<NT>(solo_lds + L.a_val, sell_vals<T>(P.sA), 2 * static_cast<int>(sizeof(T)) * J.a_slots);
    solo_stage<NT>(solo_lds + L.at_col, P.sAT.col, 4 * J.at_slots);
    solo_stage<NT>(solo_lds + L.at_val, sell_vals<T>(P.sAT), 2 * static_cast<int>(sizeof(T)) * J.at_slots);
    for (int g = tid; g < mx; g += NT) init_state_at(P, g, J.x0, J.y0);
    __syncthreads();
    solo_evaluate<NT, kFp32>(J, 1);
    while (S.sc.status == kRunning) {
        const long long left = S.sc.max_iters - S.sc.k;
        solo_period<FORM, NT, KC, KR>(J, static_cast<int>(left < S.sc.eval_every ? left : S.sc.eval_every));
        solo_evaluate<NT, kFp32>(J, 0);
    }
    for (int g = tid; g < mx; g += NT) {
        extract_at(P, S.sc.out_avg, S.sc.status, S.sc.ray_scale, S.sc.ray_src, g);
        result_to_host(J, &S.sc, g);
    }
    __syncthreads();
    if (tid == 0) *P.sc = S.sc;
}

template <int NT, int KC, int KR>
__device__ __forceinline__ void solo_form(const BatchJob& J) {
    const int form = 2 * J.P.fp32 + (J.P.method ? 1 : 0);
    if (form == 0) solo_solve<0, NT, KC, KR>(J);
    else if (form == 1) solo_solve<1, NT, KC, KR>(J);
    else if (form == 2) solo_solve<2, NT, KC, KR>(J);
    else solo_solve<3, NT, KC, KR>(J);
}

// Persistent launch with NT threads per workgroup: every workgroup takes LPs from the counter
// until it passes `count`; all of its waves return together. Each LP runs the variant that
// its job names (256 and 512 threads have one each).
template <int NT>
__global__ __launch_bounds__(NT, NT == 1024 ? 4 : 2) void solo_kernel(const BatchJob* jobs, const int* order, int count,
                                                                     int* counter) {
    SoloShared& S = solo_shared();
    for (;;) {
        __syncthreads();
        if (threadIdx.x == 0) S.job = atomicAdd(counter, 1);
        __syncthreads();
        const int j = S.job;
        if (j >= count) return;
        const BatchJob& J = jobs[order[j]];
        if constexpr (NT != 1024) {
            solo_form<NT, 1, 1>(J);
        } else {
            if (J.variant == SOLO_1024) solo_form<1024, 2, 1>(J);
            else if (J.variant == SOLO_WIDE) solo_form<1024, 4, 2>(J);
            else if (J.variant == SOLO_WIDE32) {
                if (J.P.method) solo_solve<3, 1024, 10, 5>(J);
                else solo_solve<2, 1024, 10, 5>(J);
            } else solo_form<1024, 0, 0>(J);
        }
    }
}

// ------------------------------------------------------------- norm estimate of a small LP
// The whole power iteration of an LP with Sell matrices in one workgroup: the vectors in LDS,
// the matrices staged there as far as they fit, the products summed as in solo_product, the
// norms in the order of sumsq2_kernel and normalize_kernel (nred blocks of kBlock threads,
// then a wave's halving sum), the chunk test of the set-up on the device: the same estimate
// bit for bit. What bounds it is latency, as above; the kernel-per-phase loop pays four
// launches per step (17 us) and a host round trip per chunk.
struct SoloPowerShared {
    double red[1024 / 64], part[kSoloEvalBlocks], total, sigma, prev;
};

// Sum of squares of a[0, count) in LDS; every thread gets it. Ends with a barrier.
__device__ __forceinline__ double solo_sumsq(const double* a, int count, int nred, SoloPowerShared& S) {
    const int group = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kBlock);
    const int vt = threadIdx.x % kBlock, lane = threadIdx.x & 63;
    constexpr int kGroups = 1024 / kBlock;
    for (int b0 = 0; b0 < nred; b0 += kGroups) {
        double v = 0.0;
        if (b0 + group < nred)
            for (int i = (b0 + group) * kBlock + vt; i < count; i += nred * kBlock) v += a[i] * a[i];
        v = wave_sum(v);
        if (lane == 0) S.red[threadIdx.x >> 6] = v;
        __syncthreads();
        if (vt == 0 && b0 + group < nred) {
            double t = 0.0;
            for (int k = 0; k < kBlock / 64; ++k) t += S.red[group * (kBlock / 64) + k];
            S.part[b0 + group] = t;
        }
        __syncthreads();
    }
    if (threadIdx.x < 64) {
        const double v = wave_sum(lane < nred ? S.part[lane] : 0.0);
        if (lane == 0) S.total = v;
    }
    __syncthreads();
    return S.total;
}

__global__ __launch_bounds__(1024) void solo_power_kernel(DevLP P, SoloStage G, unsigned long long seed, int iters,
                                                          int chunks) {
    extern __shared__ __align__(16) char solo_lds[];
    __shared__ SoloPowerShared S;
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), m = P.m, n = P.n;
    const SoloLds L = solo_lds_layout(m, n, 0, G.a_slots, G.at_slots);
    double* u = reinterpret_cast<double*>(solo_lds);
    double* v = reinterpret_cast<double*>(solo_lds + L.xs);
    const SellAt A{P.sA.col, P.sA.v, L.a_col, L.a_val, G.a_slices, n + 1, G.a_slots, P.sA.slots};
    const SellAt AT{P.sAT.col, P.sAT.v, L.at_col, L.at_val, G.at_slices, m + 1, G.at_slots, P.sAT.slots};
    solo_stage<1024>(solo_lds + L.a_col, P.sA.col, 4 * G.a_slots);
    solo_stage<1024>(solo_lds + L.a_val, P.sA.v, 16 * G.a_slots);
    solo_stage<1024>(solo_lds + L.at_col, P.sAT.col, 4 * G.at_slots);
    solo_stage<1024>(solo_lds + L.at_val, P.sAT.v, 16 * G.at_slots);
    for (int k = tid; k < n; k += 1024) v[k] = splitmix_centered(seed, static_cast<unsigned long long>(k));
    if (tid == 0) {
        u[m] = 0.0;
        v[n] = 0.0;
        S.sigma = S.prev = 0.0;
    }
    __syncthreads();
    const double start = sqrt(solo_sumsq(v, n, P.nred, S));
    if (start > 0.0)
        for (int k = tid; k < n; k += 1024) v[k] = v[k] / start;
    __syncthreads();
    auto product = [&](const Sell& M, const SellAt& at, int rows, const double* gat, double* out) {
        for (int sl = wave; sl < M.slices; sl += 1024 / 64) {
            const int base = M.ptr[sl], width = (M.ptr[sl + 1] - base) >> 6, r = M.row[sl * 64 + lane];
            const double s = sell_row<double>(0.0, sl, base + lane, width, at, solo_lds, gat);
            if (r < rows) out[r] = s;
        }
        __syncthreads();
    };
    // Each step: u = A v, sigma = ||u||, v = A^T u / ||A^T u||. A^T u replaces v as it is formed
    // (v is not read again); when its norm is not positive v would stay and every later step
    // repeat this one, so the iteration ends there.
    bool ended = false;
    for (int c = 0; c < chunks && !ended; ++c) {
        for (int it = 0; it < iters && !ended; ++it) {
            product(P.sA, A, m, v, u);
            const double su = solo_sumsq(u, m, P.nred, S);
            if (tid == 0) {
                S.prev = S.sigma;
                S.sigma = sqrt(su);
            }
            product(P.sAT, AT, n, u, v);
            const double nrm = sqrt(solo_sumsq(v, n, P.nred, S));
            ended = !(nrm > 0.0);
            if (!ended)
                for (int i = tid; i < n; i += 1024) v[i] = v[i] / nrm;
            __syncthreads();
        }
        if (S.sigma - S.prev <= 1e-8 * S.sigma) ended = true;
    }
    if (tid == 0) {
        P.sc->sigma_max = S.sigma;
        P.sc->sigma_prev = S.prev;
    }
}
