// Two-phase sparse products for matrices whose gathered vector exceeds an XCD's L2. Included
// by lp_kernels.hip (inside its namespace) after the tile kernels and the epilogues.
//
// What bounds a one-pass product there: one L2 request per entry for the gathered value, ~80 in
// flight per CU (1.2e7 entries: 72 us at best, 106-125 us with the update), whatever the
// stream needs. So no value is gathered from beyond LDS: phase 1 takes one block of columns per
// workgroup, holds its slice of the vector in LDS, streams the block's entries (value, 16-bit
// column inside the block) and writes the products in the same order; phase 2 takes one tile
// of rows per workgroup, reads its products (for every block one run of consecutive
// products), puts each at its CSR position in LDS and sums and updates its rows as a row tile
// does. The products and the order of the additions are those of the one-pass kernels, bit for
// bit. It moves 30 bytes per entry (FP32: 17) instead of 12 (8) and a 64-byte line per gather,
// in streams and in runs of ~270 bytes, and the products, written and read within ~100 us,
// stay in the 256 MB Infinity Cache. Measured on 1.2e7 entries, FP64 Halpern form: products
// 42-45 us (216 MB, 5 TB/s: the rate of a copy), rows 66 us with the primal and 52 us with the
// dual update (260 / 220 MB, 4.1 TB/s), against 124 and 106 us in one pass.

constexpr int kTpThreads = 512;
constexpr int kTpUnroll = 4;  // vectors of entries a thread of phase 1 has in flight

// Phase 1: workgroup blockIdx.x / kTpSplit works on block blockIdx.x / kTpSplit.
template <class T>
__device__ inline const T* tp_vals(const TwoPhase& M);
template <>
__device__ inline const double* tp_vals<double>(const TwoPhase& M) { return M.v; }
template <>
__device__ inline const float* tp_vals<float>(const TwoPhase& M) { return M.v32; }

template <class T>
struct TpVec;
template <>
struct TpVec<double> { typedef double type __attribute__((ext_vector_type(2))); static constexpr int n = 2; };
template <>
struct TpVec<float> { typedef float type __attribute__((ext_vector_type(4))); static constexpr int n = 4; };

template <class T, class Epi>
__global__ __launch_bounds__(kTpThreads) void tp_products_kernel(TwoPhase M, const T* __restrict__ xin, Epi epi) {
    extern __shared__ __align__(16) unsigned char tp_lds[];
    if (!epi.begin()) return;
    using V = typename TpVec<T>::type;
    constexpr int N = TpVec<T>::n;
    typedef unsigned short Cols __attribute__((ext_vector_type(N)));
    T* g = reinterpret_cast<T*>(tp_lds);
    const int blk = blockIdx.x / kTpSplit, part = blockIdx.x % kTpSplit, tid = threadIdx.x;
    const int c0 = blk << M.width_bits, width = min(1 << M.width_bits, M.cols - c0);
    // whole vectors of N entries; block starts are multiples of 4
    const int first = M.block_start[blk] / N, last = (M.block_start[blk + 1] + N - 1) / N;
    const int share = (last - first + kTpSplit - 1) / kTpSplit;
    const int i0 = first + part * share, i1 = min(last, i0 + share);
    const V* __restrict__ vp = reinterpret_cast<const V*>(tp_vals<T>(M));
    const Cols* __restrict__ cp = reinterpret_cast<const Cols*>(M.lcol);
    V* __restrict__ out = reinterpret_cast<V*>(M.buf);
    for (int j = tid; j < width; j += kTpThreads) g[j] = xin[c0 + j];
    __syncthreads();
    auto stream = [&](auto keep) {
        for (int i = i0 + tid; i < i1; i += kTpThreads * kTpUnroll) {
            V v[kTpUnroll];
            Cols c[kTpUnroll];
#pragma unroll
            for (int k = 0; k < kTpUnroll; ++k) {
                const int q = min(i + k * kTpThreads, i1 - 1);
                v[k] = stream_load<keep.value>(vp + q);
                c[k] = stream_load<keep.value>(cp + q);
            }
#pragma unroll
            for (int k = 0; k < kTpUnroll; ++k) {
                V p;
#pragma unroll
                for (int e = 0; e < N; ++e) p[e] = v[k][e] * g[checked_index(static_cast<int>(c[k][e]), width, 1u)];
                if (i + k * kTpThreads < i1) out[i + k * kTpThreads] = p;
            }
        }
    };
    if (M.keep) stream(std::true_type{});
    else stream(std::false_type{});
}

// Phase 2: one tile of rows per workgroup. The tiles of long rows (the last ones, numbered
// over the list of long rows) come first, then the rows longer than a tile, one workgroup
// each. Consecutive tiles go to one XCD (their runs meet inside cache lines).
//
// A tile is a chain of loads (chunk masks, run deltas, products) and two barriers with two
// tiles on a CU, so the chain is kept short: a wave loads the masks of all its chunks
// at once, one per lane, and the operands of the rows before the products.
template <class T, class Epi>
__global__ __launch_bounds__(kTpThreads, 6) void tp_rows_kernel(TwoPhase M, Csr L, const T* __restrict__ xin, Epi epi) {
    extern __shared__ __align__(16) unsigned char tp_lds[];
    __shared__ double red[kTpThreads / 64];
    if (!epi.begin()) return;
    const int nbig = M.tiles_padded;
    if (static_cast<int>(blockIdx.x) >= nbig) {
        row_tree_body<tile_nnz_of(1), T>(L, L.rowlist[blockIdx.x - nbig], xin, epi, red);
        return;
    }
    const int t = M.tiles - 1 - ((blockIdx.x % kTpXcds) * (M.tiles_padded / kTpXcds) + blockIdx.x / kTpXcds);
    if (t < 0) return;
    T* prod = reinterpret_cast<T*>(tp_lds);
    const T* __restrict__ buf = static_cast<const T*>(M.buf);
    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    constexpr int kWaves = kTpThreads / 64;
    const bool longs = t >= M.tiles_short;
    const int* __restrict__ trp = longs ? M.trp + L.rows + 1 : M.trp;
    const int r0 = M.tile_row[t + (longs ? 1 : 0)], r1 = M.tile_row[t + (longs ? 2 : 1)];
    const int p0 = trp[r0], count = trp[r1] - p0;
    const int q0 = M.tile_chunk[t], chunks = (count + 63) >> 6;
    const int* __restrict__ delta = M.delta + static_cast<long long>(t) * M.blocks;
    const unsigned short* __restrict__ posp = M.pos + static_cast<long long>(q0) * 64;
    const unsigned long long upto = lane == 63 ? ~0ull : (2ull << lane) - 1ull;
    // lane l: mask and first run of the wave's chunk l (a tile has at most 64 of them per wave)
    static_assert(kTpTileLds / 4 / 64 / kWaves <= 64, "one lane per chunk of a wave");
    const int mine = q0 + max(0, min(wave + lane * kWaves, chunks - 1));
    const unsigned long long mask_l = M.mask[mine];
    const int first_l = M.first[mine];
    constexpr int kRows = sizeof(T) == 8 ? 2 : 3;  // rows per thread whose operands are loaded ahead
    typename Epi::Pre pre[kRows];
    int a[kRows], b[kRows];
    if (!longs) {
#pragma unroll
        for (int k = 0; k < kRows; ++k) {
            const int r = min(r0 + tid + k * kTpThreads, r1 - 1);
            pre[k] = epi.load(r);
            a[k] = trp[r] - p0;
            b[k] = trp[r + 1] - p0;
        }
    }
    constexpr int U = 8;
    auto fetch = [&](auto keep) {
        for (int i = 0; wave + i * kWaves < chunks; i += U) {  // the wave's chunks i, i + 1, ...
            int src[U];
            unsigned short pos[U];
            T v[U];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int at = min(i + k, 63);
                const unsigned lo = __builtin_amdgcn_readlane(static_cast<unsigned>(mask_l), at);
                const unsigned hi = __builtin_amdgcn_readlane(static_cast<unsigned>(mask_l >> 32), at);
                const int first = __builtin_amdgcn_readlane(first_l, at);
                const int c = min(wave + (i + k) * kWaves, chunks - 1);
                const int run = first + __popcll(((static_cast<unsigned long long>(hi) << 32) | lo) & upto) - 1;
                const int e = min(c * 64 + lane, count - 1);
                src[k] = e + delta[min(max(run, 0), M.blocks - 1)];
                pos[k] = stream_load<keep.value>(posp + e);
            }
#pragma unroll
            for (int k = 0; k < U; ++k) v[k] = buf[checked_index(max(0, min(src[k], M.slots - 1)), M.slots, 1u)];
#pragma unroll
            for (int k = 0; k < U; ++k) {
                const int c = wave + (i + k) * kWaves;
                if (c < chunks && c * 64 + lane < count) prod[checked_index(static_cast<int>(pos[k]), M.tile_nnz, 2u)] = v[k];
            }
        }
    };
    if (M.keep) fetch(std::true_type{});
    else fetch(std::false_type{});
    __syncthreads();
    if (longs) {
        // as row_tree_body: thread t of kBlock adds the row's products t, t + kBlock, ... in
        // order, then the tree over kBlock threads; two rows at a time
        constexpr int kHalves = kTpThreads / kBlock;
        const int half = tid / kBlock, vt = tid % kBlock;
        for (int i = r0; i < r1; i += kHalves) {
            const int li = min(i + half, r1 - 1);
            T s = 0;
            for (int e = trp[li] - p0 + vt; e < trp[li + 1] - p0; e += kBlock) s += prod[e];
            const double w = wave_sum(static_cast<double>(s));
            if (lane == 0) red[wave] = w;
            __syncthreads();
            if (vt == 0 && i + half < r1) {
                double sum = 0.0;
                for (int k = 0; k < kBlock / 64; ++k) sum += red[half * (kBlock / 64) + k];
                const int r = M.longs[li];
                epi.finish(r, static_cast<T>(sum), epi.load(r));
            }
            __syncthreads();
        }
        return;
    }
#pragma unroll
    for (int k = 0; k < kRows; ++k) {
        const int r = r0 + tid + k * kTpThreads;
        if (r < r1 && !(M.is_long && M.is_long[r])) epi.finish(r, row_sum<true>(prod, a[k], b[k]), pre[k]);
    }
    for (int r = r0 + tid + kRows * kTpThreads; r < r1; r += kTpThreads) {
        if (M.is_long && M.is_long[r]) continue;
        const typename Epi::Pre p = epi.load(r);
        epi.finish(r, row_sum<true>(prod, trp[r] - p0, trp[r + 1] - p0), p);
    }
}

// ------------------------------------------------------------------------- set-up
// Row (in the matrix) of row i of tile t's numbering.
__device__ inline int tp_row(const TwoPhase& M, int t, int i) { return t >= M.tiles_short ? M.longs[i] : i; }

// Entries of every (block, tile) cell: counts[block * tiles + tile].
__global__ __launch_bounds__(kBlock) void tp_count_kernel(TwoPhase M, Csr A, int* counts) {
    __shared__ int hist[kTpMaxBlocks];
    const int t = blockIdx.x;
    for (int b = threadIdx.x; b < M.blocks; b += kBlock) hist[b] = 0;
    __syncthreads();
    const bool longs = t >= M.tiles_short;
    const int r0 = M.tile_row[t + (longs ? 1 : 0)], r1 = M.tile_row[t + (longs ? 2 : 1)];
    for (int i = r0 + static_cast<int>(threadIdx.x); i < r1; i += kBlock) {
        const int r = tp_row(M, t, i);
        if (!longs && M.is_long && M.is_long[r]) continue;
        for (int e = A.rp[r]; e < A.rp[r + 1]; ++e) atomicAdd(&hist[A.ci[e] >> M.width_bits], 1);
    }
    __syncthreads();
    for (int b = threadIdx.x; b < M.blocks; b += kBlock) counts[static_cast<long long>(b) * M.tiles + t] = hist[b];
}

// Places the entries of one tile (one wave, 64 CSR positions at a time, so that the order
// inside every cell is the CSR order): column and value at the cell's place in block order,
// the CSR position at the cell's place in tile order.
__global__ __launch_bounds__(64) void tp_fill_kernel(TwoPhase M, Csr A, const int* cell_base, const int* cell_k,
                                                     unsigned short* lcol, double* v, float* v32, unsigned short* pos) {
    __shared__ int placed[kTpMaxBlocks];
    const int t = blockIdx.x, lane = threadIdx.x;
    for (int b = lane; b < M.blocks; b += 64) placed[b] = 0;
    __syncthreads();
    const bool longs = t >= M.tiles_short;
    const int* trp = longs ? M.trp + A.rows + 1 : M.trp;
    const int r0 = M.tile_row[t + (longs ? 1 : 0)], r1 = M.tile_row[t + (longs ? 2 : 1)], p0 = trp[r0], count = trp[r1] - p0;
    for (int base = 0; base < count; base += 64) {
        const bool valid = base + lane < count;
        const int p = p0 + min(base + lane, count - 1);
        int lo = r0, hi = r1;  // the last row with trp[lo] <= p (empty rows before it hold no entry)
        while (hi - lo > 1) {
            const int mid = (lo + hi) >> 1;
            if (trp[mid] <= p) lo = mid;
            else hi = mid;
        }
        const int e = A.rp[tp_row(M, t, lo)] + (p - trp[lo]);
        const int col = A.ci[e], b = col >> M.width_bits;
        unsigned long long same = __ballot(valid);
        for (int bit = 0; (1 << bit) < M.blocks; ++bit) {
            const unsigned long long s = __ballot((b >> bit) & 1);
            same &= (b >> bit) & 1 ? s : ~s;
        }
        const int before = __popcll(same & ((1ull << lane) - 1ull));
        const int at = placed[b] + before;
        __syncthreads();
        if (valid) {
            if (before == 0) placed[b] += __popcll(same);
            const long long o = cell_base[static_cast<long long>(b) * M.tiles + t] + at;
            lcol[o] = static_cast<unsigned short>(col - (b << M.width_bits));
            if (v32) v32[o] = static_cast<float>(A.v[e]);
            else v[o] = A.v[e];
            pos[static_cast<long long>(M.tile_chunk[t]) * 64 + cell_k[static_cast<long long>(t) * M.blocks + b] + at] =
                static_cast<unsigned short>(p - p0);
        }
        __syncthreads();
    }
}
