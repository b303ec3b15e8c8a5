// Sparse kernels for gfx950: CSR SpMM (value-less, weighted, scaled), the
// element-wise SDDMM instances, the segmented edge softmax, degree counts.
//
// Work decomposition shared by every kernel that reduces over rows: the
// non-zeros are cut into chunks of T entries and one 64-lane wavefront owns
// one chunk (x one feature tile for SpMM).  A row that lies inside a chunk is
// finished by that wavefront.  A row that crosses a chunk boundary is written
// in pieces - the piece in the chunk where the row starts goes to the output
// row unscaled, each later piece goes to a per-chunk carry slot - and a small
// fix-up kernel adds the carry slots to the row in chunk order.  No float
// atomics: the summation order is fixed, results are reproducible, and a hub
// row of a power-law graph is spread over as many wavefronts as it needs.
#include <cfloat>
#include <type_traits>

#include "row_search.h"
#include "sensei_internal.h"

namespace sensei {

namespace {

constexpr int kBlock = kSideThreads;
constexpr int kWavesPerBlock = kBlock / 64;
constexpr int kXcds = 8;               // accelerator dies; workgroups go to them round robin
constexpr int kMaxPanels = SENSEI_MAX_PANELS;
constexpr int kShortRowNnz = 12;  // chunks whose rows average fewer non-zeros than this use one neighbour group per row

// ------------------------------------------------------------------ chunk plan

__global__ __launch_bounds__(kSideThreads) void k_side(SideWork w) { side_block(w, (int)blockIdx.x); }

// ------------------------------------------------------------------------ SpMM

template <int VEC> struct Vec;
template <> struct Vec<1> {
    float v[1];
    __device__ static Vec load(const float *p) { Vec r; r.v[0] = *p; return r; }
    __device__ void store(float *p) const { *p = v[0]; }
};
template <> struct Vec<2> {
    float v[2];
    __device__ static Vec load(const float *p) { float2 t = *reinterpret_cast<const float2 *>(p); Vec r; r.v[0] = t.x; r.v[1] = t.y; return r; }
    __device__ void store(float *p) const { *reinterpret_cast<float2 *>(p) = make_float2(v[0], v[1]); }
};
template <> struct Vec<4> {
    float v[4];
    __device__ static Vec load(const float *p) { float4 t = *reinterpret_cast<const float4 *>(p); Vec r; r.v[0] = t.x; r.v[1] = t.y; r.v[2] = t.z; r.v[3] = t.w; return r; }
    __device__ void store(float *p) const { *reinterpret_cast<float4 *>(p) = make_float4(v[0], v[1], v[2], v[3]); }
};

struct SpmmArgs {
    const int32_t *row_ptr, *col_idx, *chunk_row;
    const float *val, *r, *c, *B;
    const float2 *mz;  // softmax mode: per-row (max logit, sum of exp(logit - max))
    int val_stride;    // floats from the value of one entry to the next (1, or 2 when the values sit in (value, other) pairs)
    long long c_tile;  // floats from feature tile t of C to tile t + 1: VEC*LPG for a row-major C, n_rows * 32 for a slice-major one (ldc = 32)
    int c_tf, c_shift; // columns per feature tile (VEC * LPG, a power of two) and their logarithm
    float *C, *carry;
    long long ldb, ldc;
    long long tile_stride_b;  // bytes from feature tile t of B to tile t + 1: 4*VEC*LPG when rows are contiguous, a whole slice otherwise
    int n_rows, nnz, chunk_nnz, n_chunks;
    int f, f_store, f_carry, n_tiles, act, store_vec_ok;
    int tiles_live, n_groups;  // feature tiles worked on at the same time; chunk groups (blocks per tile)
    int accumulate, finalize;  // column panels: add to what C holds; apply row scale and activation (last panel only)
    int fix_quads;      // k_spmm_fixup: groups of four columns per workgroup
    int32_t *find_rows; // k_spmm_flat: chunk_row is still to be filled in (null: it is there)
    int scale_weights;  // k_spmm_flat: the row factor (or 1 / z) is applied to the weights of the entries, by every panel pass
    // fused attention mode: the two score vectors, the LeakyReLU slope, and where the (max, sum) pairs of row pieces go
    const float *s_l, *s_r;
    float slope;
    long long head_vec, head_mz;  // several heads of one tile each: floats from one head's score vectors to the next, pairs from one head's mz_out to the next (0: one head)
    int head_cols;   // several heads: columns of a head that are stored (c_tile apart)
    float2 *mz_out, *carry_mz;  // per row: pair of a first piece whose row goes on in the next chunk; per chunk: pair of its continued row
};

// value of `x` held by the lane whose number is byte_lane / 4 (all lanes must be active)
__device__ __forceinline__ int lane_read(int byte_lane, int x) { return __builtin_amdgcn_ds_bpermute(byte_lane, x); }
__device__ __forceinline__ float lane_read(int byte_lane, float x) {
    return __int_as_float(__builtin_amdgcn_ds_bpermute(byte_lane, __float_as_int(x)));
}

__device__ __forceinline__ float uni_f(float x) { return __int_as_float(__builtin_amdgcn_readfirstlane(__float_as_int(x))); }
// 1/z of a softmax row; a row without entries (z = 0) gives 0, never inf
__device__ __forceinline__ float inv_z(float z) { return z > 0.f ? 1.f / z : 0.f; }

struct NnzArgs {
    const int32_t *row_ptr, *col_idx, *chunk_row;
    int n_rows, nnz, chunk_nnz, n_chunks;
};

// ---- flat walk: the same chunk ownership, but the lanes walk the entries of the chunk and not its rows
//
// Walking a chunk row by row costs one chain of memory round trips per row: on a pattern with 20 entries per row a chunk of 512 entries
// has 25 rows and more, and the per-entry kernels ran at a tenth of the memory rate (row sum of 2.1 M values: 173 us).  Here a wavefront
// first marks in LDS where the rows of its chunk start (row pointers read 64 at a time) and spreads the marks by a running maximum, which
// gives every entry its row; everything after that is independent of where the rows end.  (PAD: words left free after each of PARTS equal parts
// of the chunk's entries, for a kernel whose lane groups read the same place of their parts at the same time.)  Entries are read in striped order (entry
// 64 u + lane: coalesced); sums over rows are segmented sums in blocked order (a lane owns PER consecutive entries: they are added in the
// lane, one scan over the lanes joins the pieces), the values change order through LDS.  PER = chunk_nnz / 64.
template <int PER, int PAD = 0, int PARTS = 8> __device__ __forceinline__ int flat_at(int p) { return PAD ? p + (p / (64 * PER / PARTS)) * PAD : p; }

template <int PER> struct FlatLds {
    __attribute__((aligned(16))) int row[kWavesPerBlock][64 * PER];     // row of every entry of the wavefront's chunk
    __attribute__((aligned(16))) float val[kWavesPerBlock][64 * PER];   // values on their way from striped to blocked order
};

// LDS written by other lanes of the wavefront is read after this point (the hardware keeps a wavefront's LDS operations in order; the
// compiler has to be told)
__device__ __forceinline__ void lds_exchange() {
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

// value of x in another lane by a data-parallel-primitive move (no LDS traffic), `none` where the move has no source; every lane is active where
// these are used
template <int CTRL> __device__ __forceinline__ int dpp_i32(int x, int none = 0) { return __builtin_amdgcn_update_dpp(none, x, CTRL, 0xF, 0xF, false); }
template <int CTRL> __device__ __forceinline__ float dpp_f32(float x, float none = 0.f) { return __int_as_float(dpp_i32<CTRL>(__float_as_int(x), __float_as_int(none))); }

// One step of a scan over the wavefront's lanes by data-parallel-primitive moves: what the lane gets from the one a step below, `none` where there is
// no such lane.  Steps 0 to 3 reach 1, 2, 4 and 8 lanes down within a row of 16 lanes, step 4 hands the last lane of rows 0 and 2 to all of
// rows 1 and 3, step 5 lane 31 to the upper half: after six steps of v = op(from, v) every lane holds the sum up to itself.  A move by the LDS
// crossbar (__shfl) waits a hundred cycles a step, these a few.  All lanes must be active.
template <int STEP> __device__ __forceinline__ int scan_from(int x, int none) {
    constexpr int kCtrl[6] = {0x111, 0x112, 0x114, 0x118, 0x142, 0x143}, kRows[6] = {0xF, 0xF, 0xF, 0xF, 0xA, 0xC};
    return __builtin_amdgcn_update_dpp(none, x, kCtrl[STEP], kRows[STEP], 0xF, false);
}
template <int STEP> __device__ __forceinline__ float scan_from(float x, float none) {
    return __int_as_float(scan_from<STEP>(__float_as_int(x), __float_as_int(none)));
}
// calls step(std::integral_constant<int, s>) for s = 0 .. 5
template <class Step> __device__ __forceinline__ void scan_steps(Step step) {
    step(std::integral_constant<int, 0>()); step(std::integral_constant<int, 1>()); step(std::integral_constant<int, 2>());
    step(std::integral_constant<int, 3>()); step(std::integral_constant<int, 4>()); step(std::integral_constant<int, 5>());
}
// the value of the lane before / behind, `none` in the first / last lane
__device__ __forceinline__ int lane_before(int x, int none) { return dpp_i32<0x138>(x, none); }
__device__ __forceinline__ float lane_before(float x, float none) { return dpp_f32<0x138>(x, none); }
__device__ __forceinline__ int lane_behind(int x, int none) { return dpp_i32<0x130>(x, none); }
__device__ __forceinline__ float lane_behind(float x, float none) { return dpp_f32<0x130>(x, none); }

template <int PER> struct FlatChunk {
    int lo, hi, i_first, i1;
    bool cont;              // the first row began in an earlier chunk: its sum goes to the chunk's carry slot
    int rid[PER];           // rows of this lane's entries in blocked order
    unsigned starts;        // bit e: blocked entry e of this lane is the first of its row in the chunk
    int prev_row;           // row of the entry before this lane's first one
};

// The entries of a chunk, which depend on its number alone: what a kernel loads per entry is issued before flat_rows, whose row pointers are
// two dependent round trips.
template <int PER> struct ChunkSpan {
    int lo, hi;
    __device__ __forceinline__ ChunkSpan(const NnzArgs &a, int chunk) : lo(chunk * (64 * PER)), hi(a.nnz - lo > 64 * PER ? lo + 64 * PER : a.nnz) {}
    // place of the lane's u-th entry in striped order; past the end of the chunk, its first (last of the pattern if it has none)
    __device__ __forceinline__ int at(int u, int lane) const { const int k = lo + u * 64 + lane; return k < hi ? k : lo < hi ? lo : hi - 1; }
};

// empty(r0, none) is called for every 64 rows of the chunk, by all lanes: `none` says that row r0 + lane is owned and has no entries
template <int PER, int PAD = 0, int PARTS = 8, class Empty>
__device__ __forceinline__ FlatChunk<PER> flat_rows_from(const NnzArgs &a, int chunk, int i0, int i1, int lane, int *rows, Empty empty) {
    FlatChunk<PER> c;
    c.lo = chunk * (64 * PER);
    c.hi = (a.nnz - c.lo > 64 * PER) ? c.lo + 64 * PER : a.nnz;
    c.i1 = i1;
    // rows from i0 - 1 on, the one that may go on from the chunk before: whether it does is in the first lane's own row pointers
    const int r_first = i0 > 0 ? i0 - 1 : 0;
    int s = 0, e = 0;
    if (r_first + lane < c.i1 || lane == 0) {
        const int r = r_first + lane;
        if (r < a.n_rows) { s = a.row_ptr[r]; e = a.row_ptr[r + 1]; }
    }
#pragma unroll
    for (int u = 0; u < PER; ++u) rows[flat_at<PER, PAD, PARTS>(u * 64 + lane)] = -1;
    lds_exchange();
    c.cont = i0 > 0 && __builtin_amdgcn_readfirstlane(e) > c.lo && a.nnz > 0;
    c.i_first = c.cont ? i0 - 1 : i0;
    // the next 64 rows' pointers are under way while these are marked: a chunk of short or empty rows goes round several times (2 M entries on
    // 100,000 rows, half of them empty: row sums 15.2 -> 11.7 us, attention statistics 20.5 -> 17.4)
    for (int r0 = r_first; r0 < c.i1; r0 += 64) {
        const int r = r0 + lane, ahead = r + 64;
        int s_ahead = 0, e_ahead = 0;
        if (ahead < c.i1) { s_ahead = a.row_ptr[ahead]; e_ahead = a.row_ptr[ahead + 1]; }
        bool none = false;
        if (r < c.i1 && r >= c.i_first) {
            none = e <= s;
            if (!none) rows[flat_at<PER, PAD, PARTS>(s > c.lo ? s - c.lo : 0)] = r;   // the rows of a chunk that have entries start at different places
        }
        empty(r0, none);
        s = s_ahead;
        e = e_ahead;
    }
    lds_exchange();
    c.starts = 0u;
    int top = -1;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        const int r = rows[flat_at<PER, PAD, PARTS>(lane * PER + e)];
        c.starts |= (r >= 0 ? 1u : 0u) << e;
        top = r > top ? r : top;
        c.rid[e] = top;
    }
    int run = top;
    scan_steps([&](auto st) {
        const int o = scan_from<decltype(st)::value>(run, -1);
        run = o > run ? o : run;
    });
    c.prev_row = lane_before(run, -1);
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        c.rid[e] = c.rid[e] > c.prev_row ? c.rid[e] : c.prev_row;
        rows[flat_at<PER, PAD, PARTS>(lane * PER + e)] = c.rid[e];
    }
    lds_exchange();
    return c;
}

template <int PER, int PAD = 0, int PARTS = 8, class Empty>
__device__ __forceinline__ FlatChunk<PER> flat_rows(const NnzArgs &a, int chunk, int lane, int *rows, Empty empty) {
    return flat_rows_from<PER, PAD, PARTS>(a, chunk, __builtin_amdgcn_readfirstlane(a.chunk_row[chunk]), __builtin_amdgcn_readfirstlane(a.chunk_row[chunk + 1]), lane,
                                           rows, empty);
}

// The first rows starting at or after the two ends of a chunk, found by the wavefront itself: both row pointers' places narrowed together.
__device__ __forceinline__ int2 find_chunk_rows(const NnzArgs &a, int chunk, int lane) {
    const long long t0 = (long long)chunk * a.chunk_nnz, t1 = t0 + a.chunk_nnz;
    RowSearch first = {0, a.n_rows}, last = first;
    while (first.open() || last.open()) {
        const int p0 = first.place(lane), p1 = last.place(lane);
        const long long v0 = a.row_ptr[p0], v1 = a.row_ptr[p1];   // row_ptr[n_rows] exists: both are read whether they count or not
        first.narrow(__popcll(__ballot(p0 < first.hi && v0 < t0)));
        last.narrow(__popcll(__ballot(p1 < last.hi && v1 < t1)));
    }
    return make_int2(first.lo, chunk + 1 < a.n_chunks ? last.lo : a.n_rows);
}

// Segmented sum of v (blocked order; entries past the end of the chunk hold 0): write(row, sum, end, last) once per
// row piece of the chunk: end is the place of its last entry in the chunk, last that entry's number in this lane (-1: the lane before's last; past the end of the
// chunk entries count as the last piece's).
// A lane's entries fall into a head (up to its first row start), whole rows, and a tail; the heads are completed by the scan.
template <int PER, int N, class Write>
__device__ __forceinline__ void flat_sums(const FlatChunk<PER> &c, int lane, const float (&v)[N][PER], Write write) {
    float head[N], run[N], before[N];
#pragma unroll
    for (int n = 0; n < N; ++n) head[n] = run[n] = 0.f;
    int head_last = 0;
    bool started = false;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
        if ((c.starts >> e) & 1u) {
            if (started) write(c.rid[e > 0 ? e - 1 : 0], run, lane * PER + e - 1, e - 1);
            else head_last = e - 1;
#pragma unroll
            for (int n = 0; n < N; ++n) {
                if (!started) head[n] = run[n];
                run[n] = 0.f;
            }
            started = true;
        }
#pragma unroll
        for (int n = 0; n < N; ++n) run[n] += v[n][e];
    }
    int f = started;   // run: the tail from here on
    scan_steps([&](auto st) {
        const int of = scan_from<decltype(st)::value>(f, 0);
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const float o = scan_from<decltype(st)::value>(run[n], 0.f);
            run[n] += f ? 0.f : o;
        }
        f |= of;
    });
#pragma unroll
    for (int n = 0; n < N; ++n) before[n] = lane_before(run[n], 0.f);   // the open row piece of the lanes before this one
    const int head_row = (c.starts & 1u) ? c.prev_row : c.rid[0];
    if (started && head_row >= 0 && lane > 0) {
#pragma unroll
        for (int n = 0; n < N; ++n) head[n] = before[n] + head[n];
        write(head_row, head, lane * PER + head_last, head_last);
    }
    if (lane == 63) write(c.rid[PER - 1], run, c.hi - c.lo - 1, PER - 1);
}
template <int PER, class Write>
__device__ __forceinline__ void flat_sum(const FlatChunk<PER> &c, int lane, const float (&v)[PER], Write write) {
    float one[1][PER];
#pragma unroll
    for (int e = 0; e < PER; ++e) one[0][e] = v[e];
    flat_sums<PER, 1>(c, lane, one, [&](int row, const float (&sum)[1], int end, int) { write(row, sum[0], end); });
}

// x[last], before for last = -1 (flat_sums' `last`: a constant but for a lane's first piece)
template <int PER>
__device__ __forceinline__ float last_value(const float (&x)[PER], float before, int last) {
    float v = before;
#pragma unroll
    for (int q = 0; q < PER; ++q) v = last >= q ? x[q] : v;
    return v;
}

// The maximum over every row piece, for each of its entries (blocked order; entries past the end of the chunk hold -inf): inside the lane,
// then what lies before the lane (forward scan of the tails) and behind it (backward scan of the heads).
template <int PER>
__device__ __forceinline__ void flat_piece_max(const FlatChunk<PER> &c, int lane, const float (&e)[PER], float (&mx)[PER]) {
#pragma unroll
    for (int q = 0; q < PER; ++q) mx[q] = (q > 0 && !((c.starts >> q) & 1u)) ? fmaxf(mx[q > 0 ? q - 1 : 0], e[q]) : e[q];
#pragma unroll
    for (int q = PER - 2; q >= 0; --q)
        if (!((c.starts >> (q + 1)) & 1u)) mx[q] = mx[q + 1];
    float fwd = mx[PER - 1], bwd = (c.starts & 1u) ? -INFINITY : mx[0];
    int ff = c.starts != 0u, fb = ff;
    scan_steps([&](auto st) {
        const float o = scan_from<decltype(st)::value>(fwd, -INFINITY);
        const int g = scan_from<decltype(st)::value>(ff, 0);
        fwd = ff ? fwd : fmaxf(fwd, o);
        ff |= g;
    });
    // backwards: within the rows of 16 lanes, then what lies behind the row (its first lanes' values, at most three)
    auto back = [&](float o, int g) {
        bwd = fb ? bwd : fmaxf(bwd, o);
        fb |= g;
    };
    back(dpp_f32<0x101>(bwd, -INFINITY), dpp_i32<0x101>(fb, 0));
    back(dpp_f32<0x102>(bwd, -INFINITY), dpp_i32<0x102>(fb, 0));
    back(dpp_f32<0x104>(bwd, -INFINITY), dpp_i32<0x104>(fb, 0));
    back(dpp_f32<0x108>(bwd, -INFINITY), dpp_i32<0x108>(fb, 0));
    auto first_of = [&](int l) { return __int_as_float(__builtin_amdgcn_readlane(__float_as_int(bwd), l)); };
    const float b3 = first_of(48);
    const float b2 = __builtin_amdgcn_readlane(fb, 32) ? first_of(32) : fmaxf(first_of(32), b3);
    const float b1 = __builtin_amdgcn_readlane(fb, 16) ? first_of(16) : fmaxf(first_of(16), b2);
    if (!fb && lane < 48) bwd = fmaxf(bwd, lane < 16 ? b1 : lane < 32 ? b2 : b3);
    const float before = lane_before(fwd, -INFINITY), behind = lane_behind(bwd, -INFINITY);
    bool open = true;   // entries up to the lane's first row start belong to a piece that began before the lane
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if ((c.starts >> q) & 1u) open = false;
        if (open) mx[q] = fmaxf(mx[q], before);
        if ((c.starts >> q) < 2u) mx[q] = fmaxf(mx[q], behind);   // no row starts after entry q: its piece goes on behind the lane
    }
}

// A value per row for entries in striped order.  Chunks of at most 64 rows keep the values of their rows in the lanes' registers and hand
// them out by cross-lane reads; the others gather them (a gather costs the vector cache path what the entry's own gather costs:
// statistics pass on 98,000 rows of 1,021 entries 0.73 ms with it, 0.48 without).
template <int PER>
__device__ __forceinline__ void row_values(const FlatChunk<PER> &c, int lane, const float *__restrict__ src, const int (&row)[PER], float (&x)[PER]) {
    if (c.i1 - c.i_first <= 64) {
        const float mine = c.i_first + lane < c.i1 ? src[c.i_first + lane] : 0.f;
#pragma unroll
        for (int u = 0; u < PER; ++u) x[u] = lane_read((row[u] - c.i_first) * 4, mine);
    } else {
#pragma unroll
        for (int u = 0; u < PER; ++u) x[u] = src[row[u]];
    }
}

// values from striped to blocked order (val[] of the wavefront)
template <int PER>
__device__ __forceinline__ void to_blocked(float *val, int lane, const float (&striped)[PER], float (&blocked)[PER]) {
#pragma unroll
    for (int u = 0; u < PER; ++u) val[u * 64 + lane] = striped[u];
    lds_exchange();
#pragma unroll
    for (int e = 0; e < PER; ++e) blocked[e] = val[lane * PER + e];
}

// SpMM on a row-major operand whose rows allow only 8- or 4-byte loads (odd leading dimension or width), and value-less on patterns of
// very short rows (spmm_by_rows); everything else takes k_spmm_flat below.  One wavefront = one (chunk, feature tile).  The 64 lanes form G = 64/LPG
// neighbour groups of LPG lanes; a group reads VEC*LPG consecutive floats of
// one neighbour row per step, so G
// neighbours are in flight per step and 4 steps are issued back to back.
// Column indices (and weights) are fetched 64 at a time, one per lane, and
// handed to the groups by cross-lane reads.  The inner loop carries no
// predicates: full steps of G neighbours run unmasked, the ragged end of a row
// piece is one masked step, and lanes past the last feature column read
// column 0 and never store.  With OFF32 the gathered matrix is smaller than
// 4 GiB with fewer than 2^24 rows of fewer than 2^24 bytes, and addresses are
// a uniform base plus a 32-bit byte offset formed by one 24-bit multiply-add.
// Consecutive workgroups go to consecutive XCDs and take consecutive tiles of
// the live tile set, so each XCD's L2 keeps seeing the same slice of
// the gathered matrix; the number of live tiles bounds how much of that matrix
// is in use at one time.
// MODE kSpmmSoftmax: `val` holds attention logits; the weight of an entry is exp(logit - m_i) and the row is
// scaled by 1/z_i when it is complete, so the normalised attention weights are never stored (Eq. 6).
// MODE kSpmmAttnFused: score, softmax and weighted sum in one walk (Eq. 5-6 with nothing stored per entry): the logit
// LeakyReLU(s_l[i] + s_r[j]) is formed from the two score vectors as the neighbour is gathered, every lane keeps a running
// maximum m, the sum z of exp(logit - m) and its partial row relative to m, rescaling both when the maximum grows; the
// lanes' (m, z, row) triples are merged when the row (piece) ends.  A piece of a row that spans chunks leaves its pair
// beside its partial row (mz_out / carry_mz) and k_spmm_fixup_attn merges the pieces in chunk order.
template <int VEC, int LPG, int MODE, bool OFF32>
__global__ __launch_bounds__(kBlock) void k_spmm(SpmmArgs a) {
    constexpr int G = 64 / LPG;
    constexpr int TF = VEC * LPG;
    constexpr int U = 4;  // steps issued back to back
    const int lane = threadIdx.x & 63;
    // blocks are ordered: tile set (tiles_live tiles each) major, then chunk group, then tile within the set
    const int per_set = a.n_groups * a.tiles_live;
    const int set = blockIdx.x / per_set, in_set = blockIdx.x % per_set;
    const int tile = set * a.tiles_live + in_set % a.tiles_live;
    if (tile >= a.n_tiles) return;
    // wave-uniform by construction; readfirstlane lets the compiler keep the row walk in scalar registers
    const int chunk = (in_set / a.tiles_live) * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (chunk >= a.n_chunks) return;
    const int g = lane / LPG;
    const int f0 = tile * TF + (lane % LPG) * VEC;
    const bool fok = f0 < a.f;
    const char *Bb = reinterpret_cast<const char *>(a.B) + (long long)tile * a.tile_stride_b;
    const unsigned f0_b = fok ? (unsigned)((lane % LPG) * VEC) * 4u : 0u;
    float *c_tile_base = a.C + (size_t)tile * a.c_tile + (lane % LPG) * VEC;  // this lane's columns of row 0 of C
    const unsigned ldb_b32 = (unsigned)(a.ldb * 4);
    const size_t ldb_b64 = (size_t)a.ldb * 4;

    auto gather = [&](int j) -> Vec<VEC> {
        if (OFF32) return Vec<VEC>::load(reinterpret_cast<const float *>(Bb + (__umul24((unsigned)j, ldb_b32) + f0_b)));
        return Vec<VEC>::load(reinterpret_cast<const float *>(Bb + ((size_t)j * ldb_b64 + f0_b)));
    };

    const long long lo_ll = (long long)chunk * a.chunk_nnz;
    const int lo = (int)lo_ll;
    const int hi = (int)((lo_ll + a.chunk_nnz < (long long)a.nnz) ? lo_ll + a.chunk_nnz : (long long)a.nnz);
    const int i0 = a.chunk_row[chunk];
    const int i1 = a.chunk_row[chunk + 1];

    // first row touched: the one crossing `lo` if there is one, else the first owned row
    // (the row walk is wave-uniform; uni() pins its state to scalar registers)
    auto uni = [](int x) { return __builtin_amdgcn_readfirstlane(x); };
    bool cont = (a.nnz > 0) && (a.row_ptr[i0] > lo);
    int i = uni(cont ? i0 - 1 : i0);
    int re = uni((i < a.n_rows) ? a.row_ptr[i + 1] : 0x7fffffff);
    float m_row = 0.f;  // softmax mode: max logit of row i; fused attention mode: s_l of row i
    if (MODE == kSpmmSoftmax) m_row = uni_f((i < a.n_rows) ? a.mz[i].x : 0.f);
    if (MODE == kSpmmAttnFused) m_row = uni_f((i < a.n_rows) ? a.s_l[i] : 0.f);
    float m_run = -INFINITY, z_run = 0.f;  // fused attention mode: this lane's running maximum and sum of exp(logit - maximum)

    Vec<VEC> acc;
#pragma unroll
    for (int e = 0; e < VEC; ++e) acc.v[e] = 0.f;

    auto accumulate = [&](const Vec<VEC> &b, float ww) {
        if (MODE == kSpmmAttnFused) {  // ww = s_r of the neighbour
            const float t = m_row + ww;
            const float lg = t > 0.f ? t : a.slope * t;
            const float mn = lg > m_run ? lg : m_run;
            const float keep = __expf(m_run - mn);  // 0 on the first neighbour (m_run = -inf), 1 while the maximum stands
            const float p = __expf(lg - mn);
            z_run = fmaf(z_run, keep, p);
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc.v[e] = fmaf(acc.v[e], keep, p * b.v[e]);
            m_run = mn;
            return;
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) {
            if (MODE == SENSEI_SPMM_PATTERN) acc.v[e] += b.v[e];
            else acc.v[e] = fmaf(ww, b.v[e], acc.v[e]);
        }
    };

    auto finish_row = [&](bool complete) {
        float m_all = 0.f;
        if (MODE == kSpmmAttnFused) {  // bring every group's partial row to the common maximum of the row piece
            m_all = m_run;
#pragma unroll
            for (int off = LPG; off < 64; off <<= 1) {
                const float o = __shfl_xor(m_all, off, 64);
                m_all = o > m_all ? o : m_all;
            }
            const float sc = m_run > -INFINITY ? __expf(m_run - m_all) : 0.f;  // a group that saw no neighbour holds zeros
            z_run *= sc;
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc.v[e] *= sc;
#pragma unroll
            for (int off = LPG; off < 64; off <<= 1) z_run += __shfl_xor(z_run, off, 64);
        }
#pragma unroll
        for (int off = LPG; off < 64; off <<= 1) {
#pragma unroll
            for (int e = 0; e < VEC; ++e) acc.v[e] += __shfl_xor(acc.v[e], off, 64);
        }
        if (MODE == kSpmmAttnFused && lane == 0 && tile == 0) {  // every feature tile of the chunk forms the same pair: one writes it
            if (cont) a.carry_mz[chunk] = make_float2(m_all, z_run);
            else if (!complete) a.mz_out[i] = make_float2(m_all, z_run);
        }
        if (g == 0 && fok) {
            if (cont) {
                acc.store(a.carry + (size_t)chunk * a.f_carry + f0);
            } else {
                float *dst = c_tile_base + (size_t)i * a.ldc;
                const bool vec_store = a.store_vec_ok && f0 + VEC <= a.f_store;
                if (a.accumulate) {  // later column panel: add to what the earlier panels left in C
                    if (vec_store) {
                        const Vec<VEC> old = Vec<VEC>::load(dst);
#pragma unroll
                        for (int e = 0; e < VEC; ++e) acc.v[e] += old.v[e];
                    } else {
#pragma unroll
                        for (int e = 0; e < VEC; ++e) if (f0 + e < a.f_store) acc.v[e] += dst[e];
                    }
                }
                if (complete && a.finalize) {
                    const float sc = (MODE == kSpmmAttnFused) ? inv_z(z_run) : (MODE == kSpmmSoftmax) ? inv_z(a.mz[i].y) : (a.r ? a.r[i] : 1.f);
#pragma unroll
                    for (int e = 0; e < VEC; ++e) {
                        float y = acc.v[e] * sc;
                        if (a.act == SENSEI_ACT_RELU) y = y > 0.f ? y : 0.f;
                        acc.v[e] = y;
                    }
                }
                if (vec_store) {
                    acc.store(dst);
                } else {
#pragma unroll
                    for (int e = 0; e < VEC; ++e) if (f0 + e < a.f_store) dst[e] = acc.v[e];
                }
            }
        }
#pragma unroll
        for (int e = 0; e < VEC; ++e) acc.v[e] = 0.f;
        m_run = -INFINITY;
        z_run = 0.f;
    };

    // Many short rows in this chunk: walking them one after another would leave most neighbour groups
    // idle and serialise one memory round trip per row.  Give every group a row of its own instead; a
    // group then holds the whole feature slice of its row and needs no cross-lane reduction.
    const int i_first = cont ? i0 - 1 : i0;
    if ((long long)(i1 - i_first) * kShortRowNnz > (long long)(hi - lo)) {
        for (int ib = i_first; ib < i1; ib += G) {
            const int row = ib + g;
            const bool rok = row < i1;
            int rs = 0, rend = 0, row_end = 0;
            float2 mz_g = make_float2(0.f, 0.f);
            if (rok) {
                if (MODE == kSpmmSoftmax) mz_g = a.mz[row];
                rs = a.row_ptr[row];
                row_end = a.row_ptr[row + 1];
                rs = rs > lo ? rs : lo;
                rend = row_end < hi ? row_end : hi;
            }
            Vec<VEC> racc;
#pragma unroll
            for (int e = 0; e < VEC; ++e) racc.v[e] = 0.f;
            float rm = -INFINITY, rz = 0.f;  // fused attention mode: running maximum and sum of the group's row
            const float sl_g = (MODE == kSpmmAttnFused && rok) ? a.s_l[row] : 0.f;
            for (int k = rs; k < rend; k += U) {
                Vec<VEC> b[U];
                float ww[U];
                unsigned live[U];   // a weight of 0 alone would make NaN of an infinity (masks, not branches around the gathers)
#pragma unroll
                for (int q = 0; q < U; ++q) {
                    const bool valid = k + q < rend;
                    const int kq = valid ? k + q : k;
                    const int j = a.col_idx[kq];
                    float wq = 1.f;
                    if (MODE == SENSEI_SPMM_WEIGHTED) wq = a.val[(size_t)kq * a.val_stride];
                    if (MODE == SENSEI_SPMM_SCALED) wq = a.c[j];
                    if (MODE == kSpmmSoftmax) wq = __expf(a.val[(size_t)kq * a.val_stride] - mz_g.x);
                    if (MODE == kSpmmAttnFused) {
                        const float t = sl_g + a.s_r[j];
                        wq = valid ? (t > 0.f ? t : a.slope * t) : -INFINITY;  // the logit; an entry past the end weighs exp(-inf) = 0
                        ww[q] = wq;
                    } else {
                        ww[q] = valid ? wq : 0.f;
                    }
                    b[q] = gather(j);
                    live[q] = valid ? ~0u : 0u;
                }
                if (MODE == kSpmmAttnFused) {  // one rescale for the four neighbours of the step
                    float mn = rm;
#pragma unroll
                    for (int q = 0; q < U; ++q) mn = ww[q] > mn ? ww[q] : mn;
                    const float keep = __expf(rm - mn);
                    rz *= keep;
#pragma unroll
                    for (int e = 0; e < VEC; ++e) racc.v[e] *= keep;
#pragma unroll
                    for (int q = 0; q < U; ++q) {
                        ww[q] = __expf(ww[q] - mn);
                        rz += ww[q];
                    }
                    rm = mn;
                }
#pragma unroll
                for (int q = 0; q < U; ++q) {
#pragma unroll
                    for (int e = 0; e < VEC; ++e) racc.v[e] = fmaf(ww[q], __uint_as_float(__float_as_uint(b[q].v[e]) & live[q]), racc.v[e]);
                }
            }
            if (MODE == kSpmmAttnFused && rok && tile == 0 && (lane % LPG) == 0) {
                if (cont && row == i_first) a.carry_mz[chunk] = make_float2(rm, rz);
                else if (row_end > hi) a.mz_out[row] = make_float2(rm, rz);
            }
            if (rok && fok) {
                if (cont && row == i_first) {
                    racc.store(a.carry + (size_t)chunk * a.f_carry + f0);
                } else {
                    float *dst = c_tile_base + (size_t)row * a.ldc;
                    const bool vec_store = a.store_vec_ok && f0 + VEC <= a.f_store;
                    if (a.accumulate) {
                        if (vec_store) {
                            const Vec<VEC> old = Vec<VEC>::load(dst);
#pragma unroll
                            for (int e = 0; e < VEC; ++e) racc.v[e] += old.v[e];
                        } else {
#pragma unroll
                            for (int e = 0; e < VEC; ++e) if (f0 + e < a.f_store) racc.v[e] += dst[e];
                        }
                    }
                    if (row_end <= hi && a.finalize) {
                        const float sc = (MODE == kSpmmAttnFused) ? inv_z(rz) : (MODE == kSpmmSoftmax) ? inv_z(mz_g.y) : (a.r ? a.r[row] : 1.f);
#pragma unroll
                        for (int e = 0; e < VEC; ++e) {
                            float y = racc.v[e] * sc;
                            if (a.act == SENSEI_ACT_RELU) y = y > 0.f ? y : 0.f;
                            racc.v[e] = y;
                        }
                    }
                    if (vec_store) {
                        racc.store(dst);
                    } else {
#pragma unroll
                        for (int e = 0; e < VEC; ++e) if (f0 + e < a.f_store) dst[e] = racc.v[e];
                    }
                }
            }
        }
        return;
    }

    int pos = lo;
    for (int base = lo; base < hi; base += 64) {
        const int k = base + lane;
        int col = 0;
        float w = 0.f;
        if (k < hi) {
            col = a.col_idx[k];
            if (MODE == SENSEI_SPMM_WEIGHTED || MODE == kSpmmSoftmax) w = a.val[(size_t)k * a.val_stride];
            if (MODE == SENSEI_SPMM_SCALED) w = a.c[col];
            if (MODE == kSpmmAttnFused) w = a.s_r[col];
        }
        const int bhi = (base + 64 < hi) ? base + 64 : hi;
        while (pos < bhi) {
            while (re <= pos) {  // rows ending here (or empty): close them and move on
                finish_row(true);
                cont = false;
                i = uni(i + 1);
                re = uni(a.row_ptr[i + 1]);
                if (MODE == kSpmmSoftmax) m_row = uni_f(a.mz[i].x);
                if (MODE == kSpmmAttnFused) m_row = uni_f(a.s_l[i]);
            }
            const int seg_hi = uni(re < bhi ? re : bhi);
            const int u0 = uni(pos - base), n = uni(seg_hi - pos);
            const int full = n / G;
            int src4 = (u0 + g) * 4;  // byte-lane address of this group's next neighbour
            int it = 0;
            for (; it + U <= full; it += U) {
                Vec<VEC> b[U];
                float ww[U];
#pragma unroll
                for (int q = 0; q < U; ++q) {
                    const int j = lane_read(src4 + q * G * 4, col);
                    ww[q] = (MODE == SENSEI_SPMM_PATTERN) ? 1.f : lane_read(src4 + q * G * 4, w);
                    if (MODE == kSpmmSoftmax) ww[q] = __expf(ww[q] - m_row);
                    b[q] = gather(j);
                }
#pragma unroll
                for (int q = 0; q < U; ++q) accumulate(b[q], ww[q]);
                src4 += U * G * 4;
            }
            for (; it < full; ++it) {
                const int j = lane_read(src4, col);
                float ww = (MODE == SENSEI_SPMM_PATTERN) ? 1.f : lane_read(src4, w);
                if (MODE == kSpmmSoftmax) ww = __expf(ww - m_row);
                accumulate(gather(j), ww);
                src4 += G * 4;
            }
            const int rem = n - full * G;
            if (rem > 0) {  // ragged end of the piece: groups g < rem take one more neighbour
                const bool ok = g < rem;
                const int s4 = ok ? src4 : u0 * 4;
                const int j = lane_read(s4, col);
                float ww = (MODE == SENSEI_SPMM_PATTERN) ? 1.f : lane_read(s4, w);
                if (MODE == kSpmmSoftmax) ww = __expf(ww - m_row);
                if (ok) accumulate(gather(j), ww);
            }
            pos = seg_hi;
        }
    }
    // close what is left: the current row if it ends in this chunk, then owned empty rows
    while (i < i1) {
        if (re <= hi) {
            finish_row(true);
            cont = false;
            i = uni(i + 1);
            re = uni((i < a.n_rows) ? a.row_ptr[i + 1] : 0x7fffffff);
        } else {
            finish_row(false);
            break;
        }
    }
}

// SpMM as a flat walk.  k_spmm walks the rows of its chunk one after the other, two or three dependent memory round trips each: with 20
// entries per row a chunk of 512 entries is a chain of 75 round trips (2.1 M entries x 32 columns: 67 us).  Here the chunk's entries are cut
// into eight equal parts, one per group of eight lanes, whatever rows they belong to; a group gathers its entries in order, eight in
// flight, and closes a row where the entry holds one in LDS (the row's last entry in the chunk; -1 elsewhere).
// The first row a group closes and what it has left at the end are joined over the groups by a scan; rows in between are written
// directly.  The row that goes on in the next chunk is closed nowhere: it is what the last group is left with.  Columns, weights and row factors are in LDS
// before the loop, and what an iteration needs of them and of the rows' ends is read ahead of it, so that a close waits for nothing.  Tiles, chunk ownership, carry slots and fix-up are those of k_spmm.
// Where no entry needs its row (no weights, or weights without a row factor) the lane that holds a row's pointers marks its end, and the first eight gathers
// leave as soon as the columns are there, before the row pointers are; elsewhere the rows are spread over the entries by flat_rows first.
// PLAIN: rows are written in whole 16-byte pieces and not added to; the code for the rest, unrolled into every close, costs 1 to 3 %.
// Bound by the gathers: of lines, 4 ps each from the L2s and up to 18 from far, whatever part of a line a row fills.  With the ends as flags and the rows
// looked up at a close (which the chunks of the shortest rows, the slowest, did for every entry) and the gathers behind the row pointers, before / now:
// 2.1 M entries on 100,000 rows x 64 columns 56 / 39 us (gathers alone 30), 105,000 entries x 100 columns 16.1 / 13.1 us, 42 M entries of a panel-major
// remainder x 256 columns 2.10 / 2.03 ms, 127 M entries on 2.45 M rows x 512 columns 24.7 / 23.7 ms.
// kSpmmAttnFused: the logits of the chunk are formed before the loop, and with them the maximum and the sum of every row piece
// (segmented scans), so that the loop is a plain weighted sum.
// B is row-major (a row holds all its 32-column tiles) or slice-major (all rows of tile 0, then all rows of tile 1, ...: what an XCD
// gathers from is then one contiguous range, which spreads evenly over the memory channels whatever the row pitch).
template <int MODE, int PER, int LPG, bool OFF32, bool PLAIN>
__global__ __launch_bounds__(kBlock) void k_spmm_flat(SpmmArgs a) {
    constexpr int G = 64 / LPG, T = 64 * PER, PART = T / G, PAD = 4, U = 8, WORDS = T + G * PAD;
    constexpr bool kWeights = MODE != SENSEI_SPMM_PATTERN;
    // where entries have weights the row factor goes into them (launch_spmm tells the fix-up so); a third array in LDS would cost a
    // third of the wavefronts
    constexpr bool kScaleRows = MODE == SENSEI_SPMM_PATTERN || MODE == kSpmmAttnFused;
    __shared__ __attribute__((aligned(16))) int s_col[kWavesPerBlock][WORDS];
    __shared__ __attribute__((aligned(16))) int s_row[kWavesPerBlock][WORDS];
    __shared__ __attribute__((aligned(16))) float s_scale[kScaleRows ? kWavesPerBlock : 1][kScaleRows ? WORDS : 4];
    __shared__ __attribute__((aligned(16))) float s_w[kWeights ? kWavesPerBlock : 1][kWeights ? WORDS : 4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane / LPG, li = lane % LPG;
    const int per_set = a.n_groups * a.tiles_live;
    const int set = blockIdx.x / per_set, in_set = blockIdx.x % per_set;
    const int tile = set * a.tiles_live + in_set % a.tiles_live;
    if (tile >= a.n_tiles) return;
    const int chunk = (in_set / a.tiles_live) * kWavesPerBlock + __builtin_amdgcn_readfirstlane(wave);
    if (chunk >= a.n_chunks) return;
    const int f0 = tile * (4 * LPG) + li * 4;
    const bool fok = f0 < a.f;
    const int f_end = MODE == kSpmmAttnFused && a.head_vec ? tile * 32 + a.head_cols : a.f_store;   // columns from here on are not stored
    const char *Bb = reinterpret_cast<const char *>(a.B) + (long long)tile * a.tile_stride_b;
    const unsigned f0_b = fok ? (unsigned)li * 16u : 0u;
    float *c_lane = a.C + (size_t)tile * a.c_tile + li * 4;   // this lane's columns of row 0 of C
    const unsigned ldb_b32 = (unsigned)(a.ldb * 4);
    const size_t ldb_b64 = (size_t)a.ldb * 4;
    auto gather = [&](int j) -> float4 {
        if (OFF32) return *reinterpret_cast<const float4 *>(Bb + (__umul24((unsigned)j, ldb_b32) + f0_b));
        return *reinterpret_cast<const float4 *>(Bb + ((size_t)j * ldb_b64 + f0_b));
    };
    int *rows = s_row[wave], *cols = s_col[wave];
    float *scale = s_scale[kScaleRows ? wave : 0], *wgt = s_w[kWeights ? wave : 0];
    const bool vec = PLAIN ? f0 < f_end : a.store_vec_ok && f0 + 4 <= f_end;
    auto old_row = [&](int row) {   // later column panel: what the earlier panels left in C
        float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
        const float *src = c_lane + (size_t)row * a.ldc;
        if (vec) {
            o = *reinterpret_cast<const float4 *>(src);
        } else {
            if (f0 < f_end) o.x = src[0];
            if (f0 + 1 < f_end) o.y = src[1];
            if (f0 + 2 < f_end) o.z = src[2];
            if (f0 + 3 < f_end) o.w = src[3];
        }
        return o;
    };
    auto plus = [](float4 v, const float4 &o) { v.x += o.x; v.y += o.y; v.z += o.z; v.w += o.w; return v; };
    // a finished row, or (finish = false) a piece of one that goes on in the next chunk
    auto store_row = [&](int row, float sc, float4 v, bool finish) {
        float *dst = c_lane + (size_t)row * a.ldc;
        if (a.finalize && finish) {
            v.x *= sc; v.y *= sc; v.z *= sc; v.w *= sc;
            if (a.act == SENSEI_ACT_RELU) {
                v.x = v.x > 0.f ? v.x : 0.f; v.y = v.y > 0.f ? v.y : 0.f; v.z = v.z > 0.f ? v.z : 0.f; v.w = v.w > 0.f ? v.w : 0.f;
            }
        }
        if (vec) {
            *reinterpret_cast<float4 *>(dst) = v;
        } else if (!PLAIN) {
            if (f0 < f_end) dst[0] = v.x;
            if (f0 + 1 < f_end) dst[1] = v.y;
            if (f0 + 2 < f_end) dst[2] = v.z;
            if (f0 + 3 < f_end) dst[3] = v.w;
        }
    };
    auto write_row = [&](int row, float sc, float4 v) {
        if (!PLAIN && a.accumulate) v = plus(v, old_row(row));
        store_row(row, sc, v, true);
    };
    const NnzArgs nz = {a.row_ptr, a.col_idx, a.chunk_row, a.n_rows, a.nnz, a.chunk_nnz, a.n_chunks};
    const int lo = chunk * T, hi = a.nnz - lo > T ? lo + T : a.nnz, n = hi - lo;
    float es[PER];
    int col[PER];
    if (a.nnz > 0) {
        const ChunkSpan<PER> span(nz, chunk);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const size_t k = span.at(u, lane);
            col[u] = a.col_idx[k];
            if (MODE == SENSEI_SPMM_WEIGHTED || MODE == kSpmmSoftmax) es[u] = a.val[k * a.val_stride];
        }
    }
    int i0, i1;
    if (a.find_rows) {   // nobody has: for the fix-up to read, too
        const int2 ends = find_chunk_rows(nz, chunk, lane);
        i0 = ends.x;
        i1 = ends.y;
        if (tile == 0 && lane == 0) {
            a.find_rows[chunk] = i0;
            if (chunk + 1 == a.n_chunks) a.find_rows[chunk + 1] = i1;
        }
    } else {
        i0 = __builtin_amdgcn_readfirstlane(a.chunk_row[chunk]);
        i1 = __builtin_amdgcn_readfirstlane(a.chunk_row[chunk + 1]);
    }
    auto empty_rows = [&](int r0, bool none) {   // rows without entries: one per group at a time
        unsigned long long m = __ballot(none);
        for (int b = 0; m; ++b, m >>= G) {
            if (!((m >> g) & 1ull)) continue;
            const int row = r0 + b * G + g;
            write_row(row, MODE == SENSEI_SPMM_PATTERN && a.r ? a.r[row] : 1.f, make_float4(0.f, 0.f, 0.f, 0.f));
        }
    };
    const bool use_scale = MODE == kSpmmSoftmax ? a.scale_weights != 0 : MODE != kSpmmAttnFused && a.r && (kWeights ? a.scale_weights != 0 : a.finalize != 0);
    int cont_row = -1, open_row = -1;   // the row continued from the chunk before; the row that goes on in the next chunk
    const int part0 = g * (PART + PAD);
    float4 b[U];
    auto fetch = [&](int s) {   // the gathers of a group's entries s .. s + U - 1
#pragma unroll
        for (int q = 0; q < U; q += 4) {
            const int4 t = *reinterpret_cast<const int4 *>(&cols[part0 + s + q]);
            b[q] = gather(t.x); b[q + 1] = gather(t.y); b[q + 2] = gather(t.z); b[q + 3] = gather(t.w);
        }
    };
    if (MODE == SENSEI_SPMM_PATTERN || ((MODE == SENSEI_SPMM_WEIGHTED || MODE == SENSEI_SPMM_SCALED) && !use_scale)) {
        // No entry needs to know its row: the last entry of every row is marked with it (and its factor) by the lane that has its pointers, and
        // the first gathers are under way before those arrive.
        const int r_first = i0 > 0 ? i0 - 1 : 0;
        int rs = 0, re = 0;
        float sc = 1.f;
        auto pointers = [&](int r, int &s, int &e, float &x) {
            if (r < a.n_rows) {
                s = a.row_ptr[r];
                e = a.row_ptr[r + 1];
                if (kScaleRows && use_scale) x = a.r[r];
            }
        };
        if (r_first + lane < i1 || lane == 0) pointers(r_first + lane, rs, re, sc);
        for (int i = lane; i < WORDS / 4; i += 64) reinterpret_cast<int4 *>(rows)[i] = make_int4(-1, -1, -1, -1);
        if (n > 0) {
#pragma unroll
            for (int u = 0; u < PER; ++u) cols[flat_at<PER, PAD, G>(u * 64 + lane)] = col[u];
            if (MODE == SENSEI_SPMM_SCALED) {
#pragma unroll
                for (int u = 0; u < PER; ++u) es[u] = a.c[col[u]];
            }
        }
        lds_exchange();
        if (n > 0) fetch(0);
        const bool cont = i0 > 0 && __builtin_amdgcn_readfirstlane(re) > lo && a.nnz > 0;
        const int i_first = cont ? i0 - 1 : i0;
        if (cont) cont_row = i_first;
        for (int r0 = r_first; r0 < i1; r0 += 64) {
            const int r = r0 + lane, ahead = r + 64;
            int s_ahead = 0, e_ahead = 0;
            float sc_ahead = 1.f;
            if (ahead < i1) pointers(ahead, s_ahead, e_ahead, sc_ahead);
            const bool mine = r < i1 && r >= i_first, none = mine && re <= rs;
            if (mine && !none && re <= hi) {
                const int at = flat_at<PER, PAD, G>(re - 1 - lo);
                rows[at] = r;
                if (kScaleRows) scale[at] = sc;
            }
            const unsigned long long open = __ballot(mine && !none && re > hi);
            if (open) open_row = r0 + __ffsll((long long)open) - 1;
            empty_rows(r0, none);
            rs = s_ahead;
            re = e_ahead;
            sc = sc_ahead;
        }
        if (n <= 0) return;
        if (kWeights) {
#pragma unroll
            for (int u = 0; u < PER; ++u) wgt[flat_at<PER, PAD, G>(u * 64 + lane)] = es[u];
        }
        lds_exchange();
    } else {
        const FlatChunk<PER> c = flat_rows_from<PER, PAD, G>(nz, chunk, i0, i1, lane, rows, empty_rows);
        if (n <= 0) return;
        if (c.cont) cont_row = c.i_first;
        const int last_row = __builtin_amdgcn_readfirstlane(__shfl(c.rid[PER - 1], 63, 64));
        if (__builtin_amdgcn_readfirstlane(a.row_ptr[last_row + 1]) > hi) open_row = last_row;
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            cols[flat_at<PER, PAD, G>(u * 64 + lane)] = col[u];
            if (MODE == SENSEI_SPMM_SCALED) es[u] = a.c[col[u]];
            if (MODE == kSpmmAttnFused) es[u] = a.s_r[tile * a.head_vec + col[u]];
        }
        int rw[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) rw[u] = rows[flat_at<PER, PAD, G>(u * 64 + lane)];
        if (MODE == kSpmmSoftmax) {
            // (max, sum) pairs of the rows; gathered per entry where the chunk has more rows than lanes
            const bool in_lanes = c.i1 - c.i_first <= 64;
            float2 st = make_float2(0.f, 0.f);
            if (in_lanes && c.i_first + lane < c.i1) st = a.mz[c.i_first + lane];
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                float2 p;
                if (in_lanes) p = make_float2(lane_read((rw[u] - c.i_first) * 4, st.x), lane_read((rw[u] - c.i_first) * 4, st.y));
                else p = a.mz[rw[u]];
                es[u] = __expf(es[u] - p.x);
                if (use_scale) es[u] *= inv_z(p.y);
            }
        } else if (MODE != kSpmmAttnFused) {
            float x[PER];
            row_values<PER>(c, lane, a.r, rw, x);
#pragma unroll
            for (int u = 0; u < PER; ++u) es[u] *= x[u];
        } else {
            float x[PER];
            row_values<PER>(c, lane, a.s_l + tile * a.head_vec, rw, x);
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const float t = x[u] + es[u];
                es[u] = t > 0.f ? t : a.slope * t;
            }
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) wgt[flat_at<PER, PAD, G>(u * 64 + lane)] = es[u];
        lds_exchange();
        fetch(0);
        {   // the last entry of a row in the chunk keeps its row, the others and the row that goes on are no place to close one
            unsigned ends = (c.starts >> 1) | ((unsigned)lane_behind((int)(c.starts & 1u), 0) << (PER - 1));
            const int e_last = n - 1 - lane * PER;
            if (e_last >= 0 && e_last < PER && open_row < 0) ends |= 1u << e_last;
#pragma unroll
            for (int e = 0; e < PER; ++e) rows[flat_at<PER, PAD, G>(lane * PER + e)] = (ends >> e) & 1u ? c.rid[e] : -1;
        }
        if (MODE == kSpmmAttnFused) {
            float e[PER], mx[PER], p[PER];
            const int n_mine = n - lane * PER;
#pragma unroll
            for (int q = 0; q < PER; ++q) e[q] = q < n_mine ? wgt[flat_at<PER, PAD, G>(lane * PER + q)] : -INFINITY;
            flat_piece_max<PER>(c, lane, e, mx);
#pragma unroll
            for (int q = 0; q < PER; ++q) {
                p[q] = q < n_mine ? __expf(e[q] - mx[q]) : 0.f;
                wgt[flat_at<PER, PAD, G>(lane * PER + q)] = p[q];
                scale[flat_at<PER, PAD, G>(lane * PER + q)] = mx[q];
            }
            lds_exchange();
            flat_sum<PER>(c, lane, p, [&](int i, float z, int end) {
                const int at = flat_at<PER, PAD, G>(end);
                if (tile == 0 || a.head_vec) {   // every feature tile of the chunk forms the same pairs: one writes them (a tile is a head: each its own)
                    if (i == cont_row) a.carry_mz[(a.head_vec ? (size_t)tile * a.n_chunks : 0) + chunk] = make_float2(scale[at], z);
                    else if (i == open_row) a.mz_out[tile * a.head_mz + i] = make_float2(scale[at], z);
                }
                scale[at] = inv_z(z);
            });
        }
        lds_exchange();
    }

    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f), head = acc;
    int head_row = -1;
    float head_sc = 1.f;
    const bool scaled = MODE == kSpmmAttnFused || (MODE == SENSEI_SPMM_PATTERN && use_scale);
    for (int s = 0; s < PART && s < n; s += U) {
        int end[U];
        float w[U], sc[U];
#pragma unroll
        for (int q = 0; q < U; q += 4) {
            const int4 r4 = *reinterpret_cast<const int4 *>(&rows[part0 + s + q]);
            float4 w4 = make_float4(1.f, 1.f, 1.f, 1.f), s4 = w4;
            if (kWeights) w4 = *reinterpret_cast<const float4 *>(&wgt[part0 + s + q]);
            if (kScaleRows && scaled) s4 = *reinterpret_cast<const float4 *>(&scale[part0 + s + q]);
            end[q] = r4.x; end[q + 1] = r4.y; end[q + 2] = r4.z; end[q + 3] = r4.w;
            w[q] = w4.x; w[q + 1] = w4.y; w[q + 2] = w4.z; w[q + 3] = w4.w;
            sc[q] = s4.x; sc[q + 1] = s4.y; sc[q + 2] = s4.z; sc[q + 3] = s4.w;
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (kWeights) {
                acc.x = fmaf(w[q], b[q].x, acc.x); acc.y = fmaf(w[q], b[q].y, acc.y); acc.z = fmaf(w[q], b[q].z, acc.z); acc.w = fmaf(w[q], b[q].w, acc.w);
            } else {
                acc.x += b[q].x; acc.y += b[q].y; acc.z += b[q].z; acc.w += b[q].w;
            }
            if (end[q] >= 0) {
                if (head_row < 0) {
                    head = acc;
                    head_row = end[q];
                    head_sc = sc[q];
                } else {
                    write_row(end[q], sc[q], acc);
                }
                acc = make_float4(0.f, 0.f, 0.f, 0.f);
            }
        }
        if (s + U < PART) fetch(s + U);
    }
    // a group's first row joins what the groups before it have left; the row that goes on in the next chunk is what the last group is left with
    const bool writes_head = head_row >= 0 && head_row != cont_row, writes_open = open_row >= 0 && open_row != cont_row && g == G - 1;
    float4 old_head = make_float4(0.f, 0.f, 0.f, 0.f), old_open = old_head;   // under way while the groups join
    if (!PLAIN && a.accumulate) {
        if (writes_head) old_head = old_row(head_row);
        if (writes_open) old_open = old_row(open_row);
    }
    int f = head_row >= 0;
#pragma unroll
    for (int off = LPG; off < 64; off <<= 1) {
        const float x = __shfl_up(acc.x, off, 64), y = __shfl_up(acc.y, off, 64), z = __shfl_up(acc.z, off, 64), w = __shfl_up(acc.w, off, 64);
        const int of = __shfl_up(f, off, 64);
        if (lane >= off) {
            if (!f) { acc.x += x; acc.y += y; acc.z += z; acc.w += w; }
            f |= of;
        }
    }
    auto write_carry = [&](const float4 &v) {
        if (fok) *reinterpret_cast<float4 *>(a.carry + (size_t)chunk * a.f_carry + f0) = v;
    };
    if (writes_open) store_row(open_row, 1.f, plus(acc, old_open), false);
    else if (open_row >= 0 && g == G - 1) write_carry(acc);
    const float4 in = make_float4(__shfl_up(acc.x, LPG, 64), __shfl_up(acc.y, LPG, 64), __shfl_up(acc.z, LPG, 64), __shfl_up(acc.w, LPG, 64));
    if (head_row >= 0) {
        if (g > 0) { head.x += in.x; head.y += in.y; head.z += in.z; head.w += in.w; }
        if (writes_head) store_row(head_row, head_sc, plus(head, old_head), true);
        else write_carry(head);
    }
}

// First chunk of a row that spans several chunks, seen from the chunk c that holds its first continuation: returns the row, or -1 where
// chunk c starts with a row of its own or continues a row that an earlier chunk already continued; c_last: last chunk of the row.
__device__ __forceinline__ int continued_row(const NnzArgs &a, int c, int &c_last) {
    const long long lo = (long long)c * a.chunk_nnz;
    const int i0 = a.chunk_row[c];
    if ((long long)a.row_ptr[i0] <= lo) return -1;
    const int i = i0 - 1;
    if ((long long)a.row_ptr[i] < lo - a.chunk_nnz) return -1;
    c_last = (a.row_ptr[i + 1] - 1) / a.chunk_nnz;
    return i;
}

// Rows that span several chunks, one lane per chunk: a row of up to kFixupSerial pieces is finished by the lane of its first continuation
// (serial(i, c, c_last)), a longer one by the whole wavefront (wide(i, c, c_last), uniform arguments; a hub row of 109,000 entries has 213
// pieces).  One wavefront per chunk instead costs three dependent loads per wavefront: 58 us against 12 on 195,000 chunks.
constexpr int kFixupSerial = 8;
template <class Serial, class Wide>
__device__ __forceinline__ void fixup_rows(const NnzArgs &a, Serial serial, Wide wide) {
    const int c = 1 + blockIdx.x * blockDim.x + threadIdx.x;
    int c_last = 0, i = -1;
    if (c < a.n_chunks) i = continued_row(a, c, c_last);
    const bool is_long = i >= 0 && c_last - c >= kFixupSerial;
    if (i >= 0 && !is_long) serial(i, c, c_last);
    unsigned long long todo = __ballot(is_long);
    while (todo) {
        const int l = __ffsll((long long)todo) - 1;
        todo &= todo - 1;
        wide(__builtin_amdgcn_readlane(i, l), __builtin_amdgcn_readlane(c, l), __builtin_amdgcn_readlane(c_last, l));
    }
}

// Adds the carry slots of the rows that span several chunks to their output rows, then applies the row scale and the activation.  A
// wavefront looks for such rows in kFixupChunks chunks (one per lane) and then spreads (row, four columns) pairs over its lanes; rows of
// more than kFixupSerial pieces are summed by eight groups of lanes that take the pieces in turn and are added in group order.
// blockIdx.y: the columns are dealt out 128 at a time, 32 where there are few chunks.  Bound by the traffic of the rows and slots: with one wavefront per chunk, each
// waiting for four dependent loads, 248,000 chunks x 512 columns took 0.85 ms, now 0.2 ms; with 64 chunks a wavefront a graph of 4,100
// chunks keeps too few wavefronts busy (20 us instead of 7).
constexpr int kFixupChunks = 8;
struct FixupRows {
    int i, c, c_last;            // this lane's chunk: the row it continues first (-1: none) and that row's last chunk
    unsigned long long serial, wide;
    int n_serial;
};
struct FixupLds { int row[kWavesPerBlock][kFixupChunks], first[kWavesPerBlock][kFixupChunks], last[kWavesPerBlock][kFixupChunks]; };
__device__ __forceinline__ FixupRows fixup_find(const SpmmArgs &a, FixupLds &lds, int wave, int lane) {
    const NnzArgs nz = {a.row_ptr, a.col_idx, a.chunk_row, a.n_rows, a.nnz, a.chunk_nnz, a.n_chunks};
    FixupRows r;
    r.c = 1 + (blockIdx.x * kWavesPerBlock + wave) * kFixupChunks + lane;
    r.c_last = 0;
    r.i = -1;
    if (lane < kFixupChunks && r.c < a.n_chunks) r.i = continued_row(nz, r.c, r.c_last);
    const bool is_long = r.i >= 0 && r.c_last - r.c >= kFixupSerial;
    r.serial = __ballot(r.i >= 0 && !is_long);
    r.wide = __ballot(is_long);
    r.n_serial = __popcll(r.serial);
    if (r.i >= 0 && !is_long) {
        const int at = __popcll(r.serial & ((1ull << lane) - 1));
        lds.row[wave][at] = r.i;
        lds.first[wave][at] = r.c;
        lds.last[wave][at] = r.c_last;
    }
    lds_exchange();
    return r;
}

__global__ __launch_bounds__(kBlock) void k_spmm_fixup(SpmmArgs a) {
    __shared__ FixupLds lds;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    const FixupRows fr = fixup_find(a, lds, wave, lane);
    unsigned long long wide = fr.wide;
    const int q0 = blockIdx.y * a.fix_quads, n_q = min((a.f_store + 3) / 4 - q0, a.fix_quads);   // quads of columns of this workgroup
    auto add4 = [](float4 &x, const float4 &y) { x.x += y.x; x.y += y.y; x.z += y.z; x.w += y.w; };
    const bool vec_ok = a.store_vec_ok && a.ldc % 4 == 0 && (reinterpret_cast<uintptr_t>(a.C) & 15) == 0;
    // a quad of columns never straddles feature tiles (c_tf is a power of two, 8 or more)
    auto place = [&](int row, int f) { return a.C + (size_t)(f >> a.c_shift) * a.c_tile + (size_t)row * a.ldc + (f & (a.c_tf - 1)); };
    auto fetch = [&](const float *dst, int f) {
        if (vec_ok && f + 4 <= a.f_store) return *reinterpret_cast<const float4 *>(dst);
        float4 o = make_float4(dst[0], 0.f, 0.f, 0.f);
        if (f + 1 < a.f_store) o.y = dst[1];
        if (f + 2 < a.f_store) o.z = dst[2];
        if (f + 3 < a.f_store) o.w = dst[3];
        return o;
    };
    auto factor = [&](int row) { return !a.finalize ? 1.f : a.mz ? inv_z(a.mz[row].y) : (a.r ? a.r[row] : 1.f); };
    auto finish = [&](float *dst, int f, float sc, float4 v) {
        v.x *= sc; v.y *= sc; v.z *= sc; v.w *= sc;
        if (a.finalize && a.act == SENSEI_ACT_RELU) {
            v.x = v.x > 0.f ? v.x : 0.f; v.y = v.y > 0.f ? v.y : 0.f; v.z = v.z > 0.f ? v.z : 0.f; v.w = v.w > 0.f ? v.w : 0.f;
        }
        if (vec_ok && f + 4 <= a.f_store) {
            *reinterpret_cast<float4 *>(dst) = v;
        } else {
            dst[0] = v.x;
            if (f + 1 < a.f_store) dst[1] = v.y;
            if (f + 2 < a.f_store) dst[2] = v.z;
            if (f + 3 < a.f_store) dst[3] = v.w;
        }
    };
    const int items = fr.n_serial * n_q;
    for (int item = lane; item < items; item += 64) {
        const int r = item / n_q, f = (q0 + item % n_q) * 4;
        const int first = lds.first[wave][r], last = lds.last[wave][r], row = lds.row[wave][r];
        float *dst = place(row, f);
        float4 v = fetch(dst, f);
        const float sc = factor(row);
        for (int cc = first; cc <= last; ++cc) add4(v, *reinterpret_cast<const float4 *>(a.carry + (size_t)cc * a.f_carry + f));
        finish(dst, f, sc, v);
    }
    const int g = lane >> 3;
    while (wide) {
        const int l = __ffsll((long long)wide) - 1;
        wide &= wide - 1;
        const int row = __builtin_amdgcn_readlane(fr.i, l), first = __builtin_amdgcn_readlane(fr.c, l), last = __builtin_amdgcn_readlane(fr.c_last, l);
        for (int q = lane & 7; q < n_q; q += 8) {
            const int f = (q0 + q) * 4;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
            for (int cc = first + g; cc <= last; cc += 8) add4(v, *reinterpret_cast<const float4 *>(a.carry + (size_t)cc * a.f_carry + f));
#pragma unroll
            for (int off = 8; off < 64; off <<= 1)
                add4(v, make_float4(__shfl_xor(v.x, off, 64), __shfl_xor(v.y, off, 64), __shfl_xor(v.z, off, 64), __shfl_xor(v.w, off, 64)));
            if (g == 0) {
                float *dst = place(row, f);
                float4 o = fetch(dst, f);
                add4(o, v);
                finish(dst, f, factor(row), o);
            }
        }
    }
}

// The same for the fused attention mode: the pieces of a row come with their (maximum, sum) pairs and are merged like the
// lanes of a wavefront are - everything rescaled to the largest maximum; then 1 / sum and the activation.
__global__ __launch_bounds__(kBlock) void k_spmm_fixup_attn(SpmmArgs a) {
    __shared__ FixupLds lds;
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
    if (a.head_vec) {   // one head (32 columns) per blockIdx.y
        const int head = blockIdx.y;
        a.f_store = a.head_cols;
        a.C += (size_t)head * a.c_tile;
        a.carry += (size_t)head * 32;
        a.mz_out += head * a.head_mz;
        a.carry_mz += (size_t)head * a.n_chunks;
    }
    const FixupRows fr = fixup_find(a, lds, wave, lane);
    unsigned long long wide = fr.wide;
    auto finish = [&](float *dst, float acc, float iz) {
        float y = acc * iz;
        if (a.act == SENSEI_ACT_RELU) y = y > 0.f ? y : 0.f;
        *dst = y;
    };
    const int items = fr.n_serial * a.f_store;
    for (int item = lane; item < items; item += 64) {
        const int r = item / a.f_store, f = item % a.f_store;
        const int row = lds.row[wave][r], first = lds.first[wave][r], last = lds.last[wave][r];
        float *dst = a.C + (size_t)(f / a.c_tf) * a.c_tile + (size_t)row * a.ldc + (f % a.c_tf);
        float2 own = a.mz_out[row];
        float m = own.x, z = own.y, acc = *dst;
        for (int cc = first; cc <= last; ++cc) {
            const float2 p = a.carry_mz[cc];
            const float mn = p.x > m ? p.x : m;
            const float k0 = __expf(m - mn), k1 = __expf(p.x - mn);
            acc = acc * k0 + a.carry[(size_t)cc * a.f_carry + f] * k1;
            z = z * k0 + p.y * k1;
            m = mn;
        }
        finish(dst, acc, inv_z(z));
    }
    while (wide) {   // one long row at a time: the maximum over its pieces, then lanes over columns
        const int l = __ffsll((long long)wide) - 1;
        wide &= wide - 1;
        const int row = __builtin_amdgcn_readlane(fr.i, l), first = __builtin_amdgcn_readlane(fr.c, l), last = __builtin_amdgcn_readlane(fr.c_last, l);
        const float2 own = a.mz_out[row];
        float m = own.x, z = 0.f;
        for (int cc = first + lane; cc <= last; cc += 64) m = fmaxf(m, a.carry_mz[cc].x);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) m = fmaxf(m, __shfl_xor(m, off, 64));
        for (int cc = first + lane; cc <= last; cc += 64) z += a.carry_mz[cc].y * __expf(a.carry_mz[cc].x - m);
#pragma unroll
        for (int off = 1; off < 64; off <<= 1) z += __shfl_xor(z, off, 64);
        const float k_own = __expf(own.x - m), iz = inv_z(z + own.y * k_own);
        for (int f = lane; f < a.f_store; f += 64) {
            float *dst = a.C + (size_t)(f / a.c_tf) * a.c_tile + (size_t)row * a.ldc + (f % a.c_tf);
            float acc = *dst * k_own;
#pragma unroll 8
            for (int cc = first; cc <= last; ++cc) acc = fmaf(a.carry[(size_t)cc * a.f_carry + f], __expf(a.carry_mz[cc].x - m), acc);
            finish(dst, acc, iz);
        }
    }
}

template <int VEC, int LPG, bool OFF32>
hipError_t spmm_dispatch_mode(const SpmmArgs &a, int mode, dim3 grid, hipStream_t s) {
    switch (mode) {
        case SENSEI_SPMM_PATTERN: hipLaunchKernelGGL((k_spmm<VEC, LPG, SENSEI_SPMM_PATTERN, OFF32>), grid, dim3(kBlock), 0, s, a); break;
        case SENSEI_SPMM_WEIGHTED: hipLaunchKernelGGL((k_spmm<VEC, LPG, SENSEI_SPMM_WEIGHTED, OFF32>), grid, dim3(kBlock), 0, s, a); break;
        case kSpmmSoftmax: hipLaunchKernelGGL((k_spmm<VEC, LPG, kSpmmSoftmax, OFF32>), grid, dim3(kBlock), 0, s, a); break;
        case kSpmmAttnFused: hipLaunchKernelGGL((k_spmm<VEC, LPG, kSpmmAttnFused, OFF32>), grid, dim3(kBlock), 0, s, a); break;
        default: hipLaunchKernelGGL((k_spmm<VEC, LPG, SENSEI_SPMM_SCALED, OFF32>), grid, dim3(kBlock), 0, s, a); break;
    }
    return hipGetLastError();
}

template <bool OFF32>
hipError_t spmm_rows_pattern(const SpmmArgs &a, int lpg, dim3 grid, hipStream_t s) {
    switch (lpg) {
        case 8: hipLaunchKernelGGL((k_spmm<4, 8, SENSEI_SPMM_PATTERN, OFF32>), grid, dim3(kBlock), 0, s, a); break;
        case 16: hipLaunchKernelGGL((k_spmm<4, 16, SENSEI_SPMM_PATTERN, OFF32>), grid, dim3(kBlock), 0, s, a); break;
        case 32: hipLaunchKernelGGL((k_spmm<4, 32, SENSEI_SPMM_PATTERN, OFF32>), grid, dim3(kBlock), 0, s, a); break;
        default: hipLaunchKernelGGL((k_spmm<4, 64, SENSEI_SPMM_PATTERN, OFF32>), grid, dim3(kBlock), 0, s, a); break;
    }
    return hipGetLastError();
}

template <int MODE, int LPG, bool OFF32, bool PLAIN>
hipError_t spmm_flat_per(const SpmmArgs &a, dim3 grid, hipStream_t s) {
    switch (a.chunk_nnz) {
        case 64: hipLaunchKernelGGL((k_spmm_flat<MODE, 1, LPG, OFF32, PLAIN>), grid, dim3(kBlock), 0, s, a); break;
        case 128: hipLaunchKernelGGL((k_spmm_flat<MODE, 2, LPG, OFF32, PLAIN>), grid, dim3(kBlock), 0, s, a); break;
        case 256: hipLaunchKernelGGL((k_spmm_flat<MODE, 4, LPG, OFF32, PLAIN>), grid, dim3(kBlock), 0, s, a); break;
        case 512: hipLaunchKernelGGL((k_spmm_flat<MODE, 8, LPG, OFF32, PLAIN>), grid, dim3(kBlock), 0, s, a); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

// operands with 16-byte loads: 32-column tiles, or wider ones on a row-major operand (spmm_shape)
template <int LPG, bool OFF32, bool PLAIN>
hipError_t spmm_flat_mode(const SpmmArgs &a, int mode, dim3 grid, hipStream_t s) {
    switch (mode) {
        case SENSEI_SPMM_PATTERN: return spmm_flat_per<SENSEI_SPMM_PATTERN, LPG, OFF32, PLAIN>(a, grid, s);
        case SENSEI_SPMM_WEIGHTED: return spmm_flat_per<SENSEI_SPMM_WEIGHTED, LPG, OFF32, PLAIN>(a, grid, s);
        case SENSEI_SPMM_SCALED: return spmm_flat_per<SENSEI_SPMM_SCALED, LPG, OFF32, PLAIN>(a, grid, s);
        case kSpmmSoftmax: return spmm_flat_per<kSpmmSoftmax, LPG, OFF32, PLAIN>(a, grid, s);
        case kSpmmAttnFused: return spmm_flat_per<kSpmmAttnFused, LPG, OFF32, PLAIN>(a, grid, s);
        default: break;
    }
    return hipErrorInvalidValue;
}
template <bool PLAIN>
hipError_t spmm_flat_dispatch(const SpmmArgs &a, int mode, int lpg, bool off32, dim3 grid, hipStream_t s) {
    switch (lpg) {
        case 8: return off32 ? spmm_flat_mode<8, true, PLAIN>(a, mode, grid, s) : spmm_flat_mode<8, false, PLAIN>(a, mode, grid, s);
        case 16: return spmm_flat_mode<16, false, PLAIN>(a, mode, grid, s);
        case 32: return spmm_flat_mode<32, false, PLAIN>(a, mode, grid, s);
        default: return spmm_flat_mode<64, false, PLAIN>(a, mode, grid, s);
    }
}

template <int VEC>
hipError_t spmm_dispatch_lpg(const SpmmArgs &a, int mode, int lpg, bool off32, dim3 grid, hipStream_t s) {
    switch (lpg) {
        case 8: return off32 ? spmm_dispatch_mode<VEC, 8, true>(a, mode, grid, s) : spmm_dispatch_mode<VEC, 8, false>(a, mode, grid, s);
        case 16: return off32 ? spmm_dispatch_mode<VEC, 16, true>(a, mode, grid, s) : spmm_dispatch_mode<VEC, 16, false>(a, mode, grid, s);
        case 32: return off32 ? spmm_dispatch_mode<VEC, 32, true>(a, mode, grid, s) : spmm_dispatch_mode<VEC, 32, false>(a, mode, grid, s);
        default: return off32 ? spmm_dispatch_mode<VEC, 64, true>(a, mode, grid, s) : spmm_dispatch_mode<VEC, 64, false>(a, mode, grid, s);
    }
}

// ------------------------------------------------------- element-wise / degrees

__global__ void k_fill_i32(int32_t *p, long long n, int32_t v) {
    long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) p[t] = v;
}

__global__ void k_deg_row(const int32_t *__restrict__ row_ptr, int n_rows, int32_t *__restrict__ deg_row) {
    int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n_rows) deg_row[i] = row_ptr[i + 1] - row_ptr[i];
}

__global__ void k_deg_col(const int32_t *__restrict__ col_idx, long long nnz, int32_t *__restrict__ deg_col) {
    long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (k < nnz) atomicAdd(&deg_col[col_idx[k]], 1);  // integer atomics: the result is exact in any order
}

// The same count for patterns whose columns fit a few LDS-sized ranges: a workgroup counts the entries of one share of the
// pattern that fall into one range of kDegRange columns in LDS and adds its non-zero counters to deg_col at the end, so the
// global atomics number (shares x columns) instead of one per entry, and the columns that every row refers to no longer
// serialise them.  Workgroup number -> (share, range): the ranges of one share run on one XCD at about the same time
// (workgroups are dealt round-robin to the eight XCDs), so a share is read from memory once and from that L2 afterwards.
constexpr int kDegRange = 32768, kDegThreads = 1024, kDegRangesMax = 16;

__global__ __launch_bounds__(kDegThreads) void k_deg_col_ranges(const int32_t *__restrict__ col_idx, long long nnz, int n_cols, int n_ranges,
                                                                long long per_share, int32_t *__restrict__ deg_col) {
    __shared__ int32_t cnt[kDegRange];
    const int g = blockIdx.x >> 3;
    const int range = g % n_ranges, share = (g / n_ranges) * 8 + (blockIdx.x & 7);
    const int lo_col = range * kDegRange;
    for (int d = threadIdx.x; d < kDegRange; d += kDegThreads) cnt[d] = 0;
    __syncthreads();
    const long long k0 = share * per_share, k1 = k0 + per_share < nnz ? k0 + per_share : nnz;
    long long k = k0 + threadIdx.x;
    for (; k + 3 * kDegThreads < k1; k += 4 * kDegThreads) {
        unsigned d[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) d[u] = (unsigned)(col_idx[k + u * kDegThreads] - lo_col);
#pragma unroll
        for (int u = 0; u < 4; ++u)
            if (d[u] < (unsigned)kDegRange) atomicAdd(&cnt[d[u]], 1);
    }
    for (; k < k1; k += kDegThreads) {
        const unsigned d = (unsigned)(col_idx[k] - lo_col);
        if (d < (unsigned)kDegRange) atomicAdd(&cnt[d], 1);
    }
    __syncthreads();
    const int width = n_cols - lo_col < kDegRange ? n_cols - lo_col : kDegRange;
    for (int d = threadIdx.x; d < width; d += kDegThreads) {
        const int32_t c = cnt[d];
        if (c) atomicAdd(&deg_col[lo_col + d], c);
    }
}

__global__ void k_norm_vec(const int32_t *__restrict__ deg, long long n, float *__restrict__ out) {
    long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) {
        int d = deg[t];
        d = d < 1 ? 1 : d;
        out[t] = 1.0f / sqrtf((float)d);  // IEEE sqrt and divide (hipcc's default), no rsq approximation
    }
}


constexpr int kShortRowElem = 16;  // element-wise kernels: chunks whose rows average fewer non-zeros use one lane per row

// Visits every non-zero of one chunk with one wavefront.  per_row(i) is evaluated once per row (piece) and its
// result handed to per_nnz(k, row_data) for each non-zero k of that row inside the chunk.  Long rows: the
// wavefront walks the rows (row data in scalar registers) and its lanes stride over the non-zeros, so loads
// and stores are coalesced.  Short rows: one lane per row.  Either way no per-non-zero row search is needed.
template <class PerRow, class PerNnz>
__device__ __forceinline__ void walk_chunk(const NnzArgs &a, int chunk, int lane, PerRow per_row, PerNnz per_nnz) {
    const long long lo_ll = (long long)chunk * a.chunk_nnz;
    const int lo = (int)lo_ll;
    const int hi = (int)((lo_ll + a.chunk_nnz < (long long)a.nnz) ? lo_ll + a.chunk_nnz : (long long)a.nnz);
    if (lo >= hi) return;
    const int i0 = a.chunk_row[chunk], i1 = a.chunk_row[chunk + 1];
    const int i_first = (a.row_ptr[i0] > lo) ? i0 - 1 : i0;
    if ((long long)(i1 - i_first) * kShortRowElem > (long long)(hi - lo)) {
        for (int ib = i_first; ib < i1; ib += 64) {
            const int row = ib + lane;
            if (row < i1) {
                int rs = a.row_ptr[row], re = a.row_ptr[row + 1];
                rs = rs > lo ? rs : lo;
                re = re < hi ? re : hi;
                if (rs < re) {
                    const auto rd = per_row(row);
#pragma unroll 4
                    for (int k = rs; k < re; ++k) per_nnz(k, rd);
                }
            }
        }
        return;
    }
    int i = __builtin_amdgcn_readfirstlane(i_first);
    int pos = lo;
    while (pos < hi) {
        const int re = __builtin_amdgcn_readfirstlane(a.row_ptr[i + 1]);
        if (re > pos) {
            const int seg_hi = re < hi ? re : hi;
            const auto rd = per_row(i);
#pragma unroll 4
            for (int k = pos + lane; k < seg_hi; k += 64) per_nnz(k, rd);
            pos = seg_hi;
        }
        i = __builtin_amdgcn_readfirstlane(i + 1);
    }
}

__device__ __forceinline__ int wave_chunk() {
    return blockIdx.x * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// The same with the chunks in one contiguous range per XCD (workgroups go round robin to the eight XCDs): for grids of blocks_by_xcd().
__device__ __forceinline__ int wave_chunk_by_xcd() {
    const int block = (blockIdx.x & (kXcds - 1)) * (gridDim.x / kXcds) + blockIdx.x / kXcds;
    return block * kWavesPerBlock + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
}

// out[k] = op(row value of entry k, column value of entry k): the SDDMM instances with a vector on either side
template <int PER, class Op>
__device__ __forceinline__ void flat_edge_op(const NnzArgs &a, const float *__restrict__ row_vec, const float *__restrict__ col_vec,
                                             float *__restrict__ out, Op op) {
    __shared__ FlatLds<PER> lds;
    const int chunk = wave_chunk(), lane = threadIdx.x & 63;
    if (chunk >= a.n_chunks) return;
    int *rows = lds.row[threadIdx.x >> 6];
    const ChunkSpan<PER> span(a, chunk);
    float y[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) y[u] = col_vec[a.col_idx[span.at(u, lane)]];
    const FlatChunk<PER> c = flat_rows<PER>(a, chunk, lane, rows, [](int, bool) {});
    if (c.lo >= c.hi) return;
    // one value at a time: with all eight read in one branch (row_values) 115 M entries of 494 a row take 365 us instead of 327, 100 M of 1,021 421 instead of
    // 394, and patterns of short rows 3 to 5 % less (2.1 M entries of 21 12.8 instead of 13.4 us)
    const bool in_lanes = c.i1 - c.i_first <= 64;
    const float mine = in_lanes && c.i_first + lane < c.i1 ? row_vec[c.i_first + lane] : 0.f;
    float x[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) x[u] = in_lanes ? lane_read((rows[u * 64 + lane] - c.i_first) * 4, mine) : row_vec[rows[u * 64 + lane]];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int k = c.lo + u * 64 + lane;
        if (k < c.hi) out[k] = op(x[u], y[u]);
    }
}

template <int PER>
__global__ __launch_bounds__(kBlock) void k_sddmm_norm(NnzArgs a, const float *__restrict__ r, const float *__restrict__ c, float *__restrict__ val) {
    flat_edge_op<PER>(a, r, c, val, [](float x, float y) { return x * y; });
}

__device__ __forceinline__ float leaky(float t, float slope) { return t > 0.f ? t : slope * t; }

template <int PER>
__global__ __launch_bounds__(kBlock) void k_score(NnzArgs a, const float *__restrict__ s_l, const float *__restrict__ s_r, float slope,
                                                   float *__restrict__ e) {
    flat_edge_op<PER>(a, s_l, s_r, e, [slope](float x, float y) { return leaky(x + y, slope); });
}

template <int VEC>
__global__ void k_row_broadcast(const float *__restrict__ s, const float *X, long long ldx, long long n, int f, float *Y,
                                long long ldy, int act, const float *__restrict__ mask, long long ldm, SideWork side) {  // Y may be X (in place)
    if ((int)blockIdx.x < side.blocks) return side_block(side, (int)blockIdx.x);
    const int fv = f / VEC;
    long long t = (long long)(blockIdx.x - side.blocks) * blockDim.x + threadIdx.x;
    if (t >= n * fv) return;
    const long long i = t / fv;
    const int q = (int)(t % fv) * VEC;
    const float sc = s ? s[i] : 1.f;
    Vec<VEC> x = Vec<VEC>::load(X + i * ldx + q);
#pragma unroll
    for (int e = 0; e < VEC; ++e) {
        float y = x.v[e] * sc;
        if (act == SENSEI_ACT_RELU) y = y > 0.f ? y : 0.f;
        if (mask && !(mask[i * ldm + q + e] > 0.f)) y = 0.f;  // gradient of ReLU: passes where the forward output is positive
        x.v[e] = y;
    }
    x.store(Y + i * ldy + q);
}

__global__ void k_reciprocal(const float *__restrict__ v, long long n, float *__restrict__ out) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) out[i] = 1.0f / v[i];
}

__global__ void k_stack_weights(const float *__restrict__ W, long long ldw, int hops, int f_in, int fp, int f_out, float *__restrict__ out,
                                long long ldo) {
    const long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= (long long)hops * fp * f_out) return;
    const int m = (int)(i % f_out);
    const long long row = i / f_out;
    const int h = (int)(row / fp), f = (int)(row % fp);
    out[row * ldo + m] = f < f_in ? W[((long long)h * f_in + f) * ldw + m] : 0.f;
}

// Copy of X (n x f, row-major) into slice-major tiles of 32 columns, optionally scaled per row; the pad columns
// up to the next multiple of 32 are written as zeros.  One thread per (row, 4 columns).
// d < f: heads of d columns (at most 32) that get a slice each
__global__ void k_to_slices(const float *__restrict__ s, const float *__restrict__ X, long long ldx, long long n, int f, int d,
                            float *__restrict__ Y, int x_vec_ok, const float *__restrict__ mask, long long ldm, SideWork side) {
    if ((int)blockIdx.x < side.blocks) return side_block(side, (int)blockIdx.x);
    const int fp4 = d < f ? f / d * 8 : ((f + 31) & ~31) / 4;
    const long long t = (long long)(blockIdx.x - side.blocks) * blockDim.x + threadIdx.x;
    if (t >= n * fp4) return;
    // consecutive threads walk the rows of one tile: reads are 16-byte pieces 8 to a row, writes are contiguous
    const long long per_tile = n * 8;
    const int tile = (int)(t / per_tile);
    const long long in_tile = t % per_tile;
    const long long i = in_tile >> 3;
    const int q = (d < f ? tile * d : tile * 32) + (int)(in_tile & 7) * 4;
    if (d < f) f = tile * d + d;   // where this slice's columns end
    const float sc = s ? s[i] : 1.f;
    float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
    const float *x = X + i * ldx + q;
    if (x_vec_ok && q + 4 <= f) {
        v = *reinterpret_cast<const float4 *>(x);
    } else {
        if (q < f) v.x = x[0];
        if (q + 1 < f) v.y = x[1];
        if (q + 2 < f) v.z = x[2];
        if (q + 3 < f) v.w = x[3];
    }
    v.x *= sc; v.y *= sc; v.z *= sc; v.w *= sc;
    if (mask) {  // gradient of ReLU: passes where the forward output is positive
        const float *mk = mask + i * ldm + q;
        if (!(q < f && mk[0] > 0.f)) v.x = 0.f;
        if (!(q + 1 < f && mk[1] > 0.f)) v.y = 0.f;
        if (!(q + 2 < f && mk[2] > 0.f)) v.z = 0.f;
        if (!(q + 3 < f && mk[3] > 0.f)) v.w = 0.f;
    }
    *reinterpret_cast<float4 *>(Y + (size_t)tile * (size_t)n * 32 + (size_t)in_tile * 4) = v;
}

// ------------------------------------------------------------- edge softmax

// (m, z) pairs: z = sum of exp(e - m).  Merge keeps m the larger maximum.
__device__ __forceinline__ void mz_merge(float &m, float &z, float m2, float z2) {
    const float mm = m > m2 ? m : m2;
    if (mm == -INFINITY) { m = mm; z = 0.f; return; }
    z = z * expf(m - mm) + z2 * expf(m2 - mm);
    m = mm;
}

struct SoftmaxArgs {
    NnzArgs n;
    const float *e, *s_l, *s_r;
    float slope;
    float2 *stats, *carry;
    float *alpha;
    float *logits;             // where the statistics pass parks the logits it computed from s_l, s_r
    const int32_t *dst_index;  // optional: the logit of entry k goes to logits[dst_index[k]] (panel or remainder order), nowhere if negative
};

// Row statistics of the logits (read, or formed from the two score vectors and stored on the way): a flat walk whose segmented
// reduction merges (max, sum) pairs.
template <bool FROM_E, int PER, class SrOf>
__device__ __forceinline__ void softmax_stats_chunk(const SoftmaxArgs &a, int chunk, int lane, int *rows, float *val, SrOf s_r_of) {
    float es[PER], e[PER], sr[PER];
    int dst[PER];
    if (a.n.nnz > 0) {
        const ChunkSpan<PER> span(a.n, chunk);
        if (FROM_E) {
#pragma unroll
            for (int u = 0; u < PER; ++u) es[u] = a.e[span.at(u, lane)];
        } else {
            int col[PER];
#pragma unroll
            for (int u = 0; u < PER; ++u) {
                const int k = span.at(u, lane);
                col[u] = a.n.col_idx[k];
                dst[u] = a.dst_index ? a.dst_index[k] : k;
            }
#pragma unroll
            for (int u = 0; u < PER; ++u) sr[u] = s_r_of(col[u]);
        }
    }
    const FlatChunk<PER> c = flat_rows<PER>(a.n, chunk, lane, rows, [&](int r0, bool none) { if (none) a.stats[r0 + lane] = make_float2(-INFINITY, 0.f); });
    if (c.lo >= c.hi) return;
    if (!FROM_E) {
        // (row_values for all eight at once costs the pass over column panels 5 %: 335 -> 352 us on 100 M entries)
        const bool in_lanes = c.i1 - c.i_first <= 64;
        const float mine = in_lanes && c.i_first + lane < c.i1 ? a.s_l[c.i_first + lane] : 0.f;
#pragma unroll
        for (int u = 0; u < PER; ++u) es[u] = in_lanes ? lane_read((rows[u * 64 + lane] - c.i_first) * 4, mine) : a.s_l[rows[u * 64 + lane]];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            es[u] = leaky(es[u] + sr[u], a.slope);
            if (c.lo + u * 64 + lane < c.hi && dst[u] >= 0) a.logits[dst[u]] = es[u];   // kept for the second pass (negative: the entry lies in a dense tile)
        }
    }
    to_blocked<PER>(val, lane, es, e);
    // head, whole rows and tail of this lane as in flat_sum, with (max, sum of exp) pairs: the maximum over the part of a row that
    // lies in this lane first (forwards, then handed back), then one exp per entry
    const int n_mine = c.hi - c.lo - lane * PER;   // entries of this lane inside the chunk (may be more than PER, or negative)
    float mx[PER];   // never below the lowest finite value: entries of -inf (masked out) then weigh exp(-inf) = 0, also where the lane holds no others
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if (q >= n_mine) e[q] = -INFINITY;
        mx[q] = fmaxf((q > 0 && !((c.starts >> q) & 1u)) ? mx[q > 0 ? q - 1 : 0] : -FLT_MAX, e[q]);
    }
#pragma unroll
    for (int q = PER - 2; q >= 0; --q)
        if (!((c.starts >> (q + 1)) & 1u)) mx[q] = mx[q + 1];
    auto write = [&](int i, float m, float z) {
        if (z == 0.f) m = -INFINITY;
        if (c.cont && i == c.i_first) a.carry[chunk] = make_float2(m, z);
        else a.stats[i] = make_float2(m, z);
    };
    float hm = -INFINITY, hz = 0.f, rz = 0.f;
    bool started = false;
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        if ((c.starts >> q) & 1u) {
            const float pm = q > 0 ? mx[q > 0 ? q - 1 : 0] : -INFINITY;
            if (started) write(c.rid[q > 0 ? q - 1 : 0], pm, rz);
            else { hm = pm; hz = rz; }
            started = true;
            rz = 0.f;
        }
        if (q < n_mine) rz += __expf(e[q] - mx[q]);
    }
    float m = mx[PER - 1], z = rz;
    int f = started;
    // by the LDS crossbar: the pass is bound by vector instructions, which moves of three values a step would add to
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const float m2 = __shfl_up(m, off, 64), z2 = __shfl_up(z, off, 64);
        const int of = __shfl_up(f, off, 64);
        if (lane >= off) {
            if (!f) mz_merge(m, z, m2, z2);
            f |= of;
        }
    }
    const float bm = __shfl_up(m, 1, 64), bz = __shfl_up(z, 1, 64);
    const int head_row = (c.starts & 1u) ? c.prev_row : c.rid[0];
    if (started && head_row >= 0 && lane > 0) {
        mz_merge(hm, hz, bm, bz);
        write(head_row, hm, hz);
    }
    if (lane == 63) write(c.rid[PER - 1], m, z);
}

template <bool FROM_E, int PER>
__global__ __launch_bounds__(kBlock) void k_softmax_stats(SoftmaxArgs a) {
    __shared__ FlatLds<PER> lds;
    const int chunk = wave_chunk(), wave = threadIdx.x >> 6;
    if (chunk >= a.n.n_chunks) return;
    softmax_stats_chunk<FROM_E, PER>(a, chunk, threadIdx.x & 63, lds.row[wave], lds.val[wave], [&](int col) { return a.s_r[col]; });
}

// The same over a column-panel copy of the pattern, the logits left in the copy's order.  Over the pattern itself the pass is bound by its 4-byte
// gathers of s_r, which move a 128-byte line from L2 each (100 M entries on 98,000 columns: 12.8 GB, 490 us) and by the places of the entries in
// the copy, read and scattered to.  A panel's share of s_r fits LDS: a workgroup of 16 wavefronts fills it once (up to kPanelStatsCols floats) and
// walks its share of the panel's chunks, one workgroup a compute unit.  A row's statistics come in one pair per panel and chunk and are put
// together by k_panel_stats_join: 490 -> 340 us in all (then bound by the instructions of the segmented scans: fetching the next chunk ahead gains nothing).
constexpr int kPanelStatsWaves = 16, kPanelStatsCols = 20480;
struct PanelStatsArgs {
    SoftmaxArgs s[kMaxPanels];   // stats, carry: the panel's own
    int n_panels, per_panel, width, n_cols;
};
template <int PER>
__global__ __launch_bounds__(64 * kPanelStatsWaves) void k_panel_stats(PanelStatsArgs a) {
    extern __shared__ __attribute__((aligned(16))) float panel_lds[];
    const int q = blockIdx.x / a.per_panel, part = blockIdx.x % a.per_panel, wave = threadIdx.x >> 6;
    const SoftmaxArgs &s = a.s[q];
    int *rows = reinterpret_cast<int *>(panel_lds) + wave * (128 * PER);
    float *val = panel_lds + wave * (128 * PER) + 64 * PER, *sr = panel_lds + kPanelStatsWaves * (128 * PER);
    const int col0 = q * a.width, cols = a.n_cols - col0 < a.width ? a.n_cols - col0 : a.width;
    for (int j = threadIdx.x; j < cols; j += 64 * kPanelStatsWaves) sr[j] = s.s_r[col0 + j];
    __syncthreads();
    const int c0 = (int)((long long)s.n.n_chunks * part / a.per_panel), c1 = (int)((long long)s.n.n_chunks * (part + 1) / a.per_panel);
    for (int chunk = c0 + wave; chunk < c1; chunk += kPanelStatsWaves) {
        softmax_stats_chunk<false, PER>(s, chunk, threadIdx.x & 63, rows, val, [&](int col) { return sr[col - col0]; });
        lds_exchange();   // the next chunk writes where this one read
    }
}

// stats[i] = the pairs of row i over all panels and the chunks it goes on in, in that order
__global__ void k_panel_stats_join(PanelStatsArgs a, float2 *__restrict__ stats, int n_rows) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= n_rows) return;
    float m = -INFINITY, z = 0.f;
    for (int q = 0; q < a.n_panels; ++q) {
        const SoftmaxArgs &s = a.s[q];
        const int rs = s.n.row_ptr[i], re = s.n.row_ptr[i + 1];
        const float2 own = s.stats[i];
        mz_merge(m, z, own.x, own.y);
        if (re <= rs) continue;
#pragma unroll 4
        for (int c = rs / s.n.chunk_nnz + 1; c <= (re - 1) / s.n.chunk_nnz; ++c) {
            const float2 p = s.carry[c];
            mz_merge(m, z, p.x, p.y);
        }
    }
    stats[i] = make_float2(m, z);
}

// merges the carried (m, z) pieces of rows that span several chunks, in chunk order or (long rows) lane by lane and then over the lanes
__global__ __launch_bounds__(kBlock) void k_softmax_fixup(SoftmaxArgs a) {
    const int lane = threadIdx.x & 63;
    fixup_rows(a.n,
               [&](int i, int c, int c_last) {
                   float2 st = a.stats[i];
                   for (int cc = c; cc <= c_last; ++cc) {
                       const float2 p = a.carry[cc];
                       mz_merge(st.x, st.y, p.x, p.y);
                   }
                   a.stats[i] = st;
               },
               [&](int i, int c, int c_last) {
                   float m = -INFINITY, z = 0.f;
                   for (int cc = c + lane; cc <= c_last; cc += 64) {
                       const float2 p = a.carry[cc];
                       mz_merge(m, z, p.x, p.y);
                   }
#pragma unroll
                   for (int off = 1; off < 64; off <<= 1) {
                       const float m2 = __shfl_xor(m, off, 64), z2 = __shfl_xor(z, off, 64);
                       mz_merge(m, z, m2, z2);
                   }
                   if (lane == 0) {
                       float2 st = a.stats[i];
                       mz_merge(st.x, st.y, m, z);
                       a.stats[i] = st;
                   }
               });
}

// alpha = exp(e - m_i) / z_i; `e` may be the alpha array itself (in place)
template <int PER>
__global__ __launch_bounds__(kBlock) void k_softmax_alpha(SoftmaxArgs a) {
    __shared__ FlatLds<PER> lds;
    const int chunk = wave_chunk(), lane = threadIdx.x & 63;
    if (chunk >= a.n.n_chunks) return;
    int *rows = lds.row[threadIdx.x >> 6];
    const ChunkSpan<PER> span(a.n, chunk);
    float e[PER];
    float2 st[PER];
#pragma unroll
    for (int u = 0; u < PER; ++u) e[u] = a.e[span.at(u, lane)];
    const FlatChunk<PER> c = flat_rows<PER>(a.n, chunk, lane, rows, [](int, bool) {});
    if (c.lo >= c.hi) return;
#pragma unroll
    for (int u = 0; u < PER; ++u) st[u] = a.stats[rows[u * 64 + lane]];
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int k = c.lo + u * 64 + lane;
        if (k < c.hi) a.alpha[k] = expf(e[u] - st[u].x) / st[u].y;
    }
}

// ------------------------------------------------------------ column panels

// first position in [lo, hi) of an ascending index run whose column is >= bound
__device__ __forceinline__ int lower_bound_col(const int32_t *__restrict__ col_idx, int lo, int hi, int bound) {
    while (lo < hi) {
        const int mid = (int)(((long long)lo + hi) >> 1);
        if (col_idx[mid] < bound) lo = mid + 1; else hi = mid;
    }
    return lo;
}

struct PanelPtrs {
    int32_t *rp[kMaxPanels];  // per panel: n_rows + 1 entries (counts, then row pointers after the scan)
};

// cnt[q][i] = entries of row i whose column lies in panel q (panel q = columns [q*width, (q+1)*width))
__global__ void k_panel_count(const int32_t *__restrict__ row_ptr, const int32_t *__restrict__ col_idx, int n_rows, int n_panels,
                              int width, PanelPtrs pp) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i > n_rows) return;
    if (i == n_rows) {
        for (int q = 0; q < n_panels; ++q) pp.rp[q][n_rows] = 0;
        return;
    }
    const int hi = row_ptr[i + 1];
    int prev = row_ptr[i];
    for (int q = 0; q < n_panels; ++q) {
        const int pos = (q + 1 < n_panels) ? lower_bound_col(col_idx, prev, hi, (q + 1) * width) : hi;
        pp.rp[q][i] = pos - prev;
        prev = pos;
    }
}

// exclusive prefix sum over int32, in place: per-block scan, sequential scan of the block totals, add back
constexpr int kScanPerBlock = 2048;
__global__ __launch_bounds__(256) void k_scan_local(int32_t *data, int n, int32_t *block_sums) {
    __shared__ int part[256];
    const int base = blockIdx.x * kScanPerBlock + threadIdx.x * 8;
    int v[8], sum = 0;
#pragma unroll
    for (int e = 0; e < 8; ++e) { v[e] = (base + e < n) ? data[base + e] : 0; sum += v[e]; }
    part[threadIdx.x] = sum;
    __syncthreads();
    for (int off = 1; off < 256; off <<= 1) {
        const int add = threadIdx.x >= off ? part[threadIdx.x - off] : 0;
        __syncthreads();
        part[threadIdx.x] += add;
        __syncthreads();
    }
    int run = part[threadIdx.x] - sum;  // exclusive prefix of this thread within the block
#pragma unroll
    for (int e = 0; e < 8; ++e) { if (base + e < n) data[base + e] = run; run += v[e]; }
    if (threadIdx.x == 255) block_sums[blockIdx.x] = part[255];
}
__global__ void k_scan_sums(int32_t *block_sums, int n_blocks) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    int run = 0;
    for (int b = 0; b < n_blocks; ++b) { const int v = block_sums[b]; block_sums[b] = run; run += v; }
}
__global__ __launch_bounds__(256) void k_scan_add(int32_t *data, int n, const int32_t *__restrict__ block_sums) {
    const int add = block_sums[blockIdx.x];
    const int base = blockIdx.x * kScanPerBlock + threadIdx.x * 8;
#pragma unroll
    for (int e = 0; e < 8; ++e) if (base + e < n) data[base + e] += add;
}

// off[q] = number of entries in panels before q (start of panel q in the concatenated column / perm arrays); off[n_panels] = nnz
__global__ void k_panel_offsets(PanelPtrs pp, int n_rows, int n_panels, int32_t *off) {
    if (blockIdx.x != 0 || threadIdx.x != 0) return;
    int run = 0;
    for (int q = 0; q < n_panels; ++q) { off[q] = run; run += pp.rp[q][n_rows]; }
    off[n_panels] = run;
}

struct PanelRow {
    int pos[kMaxPanels];   // first entry of the row that belongs to panel q (original numbering)
    int base[kMaxPanels];  // where the row's panel-q entries start in the panel copy
};

// copies every entry's column into its panel and records where each original entry went
__global__ __launch_bounds__(kBlock) void k_panel_scatter(NnzArgs a, int n_panels, int width, PanelPtrs pp, const int32_t *__restrict__ off,
                                                           int32_t *__restrict__ col_out, int32_t *__restrict__ perm_out) {
    const int chunk = wave_chunk();
    if (chunk >= a.n_chunks) return;
    walk_chunk(a, chunk, threadIdx.x & 63,
               [&](int i) {
                   PanelRow rd;
                   const int hi = a.row_ptr[i + 1];
                   int prev = a.row_ptr[i];
#pragma unroll
                   for (int q = 0; q < kMaxPanels; ++q) {
                       rd.pos[q] = prev;
                       rd.base[q] = 0;
                       if (q < n_panels) {
                           rd.base[q] = off[q] + pp.rp[q][i];
                           prev = (q + 1 < n_panels) ? lower_bound_col(a.col_idx, prev, hi, (q + 1) * width) : hi;
                       }
                   }
                   return rd;
               },
               [&](int k, const PanelRow &rd) {
                   const int col = a.col_idx[k];
                   int p = rd.pos[0], b = rd.base[0];
#pragma unroll
                   for (int q = 1; q < kMaxPanels; ++q)
                       if (q < n_panels && col >= q * width) { p = rd.pos[q]; b = rd.base[q]; }
                   const int d = b + (k - p);
                   col_out[d] = col;
                   perm_out[k] = d;
               });
}

// One row-pointer array over the segments (panel q, row i) -> q * n_rows + i of a panel copy, in global positions: the panel
// copy read as a single CSR with n_panels * n_rows rows, whose entries run panel by panel
__global__ void k_panel_segments(PanelPtrs pp, const int32_t *__restrict__ off, int n_rows, int n_panels, int32_t *__restrict__ seg_ptr) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    const long long total = (long long)n_panels * n_rows;
    if (t > total) return;
    if (t == total) { seg_ptr[t] = off[n_panels]; return; }
    const int q = (int)(t / n_rows), i = (int)(t % n_rows);
    seg_ptr[t] = off[q] + pp.rp[q][i];
}

__global__ void k_replicate_f2(const float2 *__restrict__ src, long long n, int copies, float2 *__restrict__ dst) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n * copies) dst[t] = src[t % n];
}

// ------------------------------------------------------- dense tiles of the hub region (set-up kernels)
//
// Nodes are ranked by degree (rank 0 = the longest row / the most referenced column).  In rank order the pattern of a
// skewed graph is nearly dense at the top left; tiles of 128 x 128 ranks that hold enough entries are stored as bit
// masks and multiplied on the matrix cores, the entries outside such tiles stay in a (smaller) CSR remainder.
struct TileMapArgs {
    NnzArgs n;
    const int32_t *rank_r, *rank_c;  // rank of every row / column node; ranks >= h_r / h_c lie outside the tiled region
    int h_r, h_c, nt_c;
};

__device__ __forceinline__ int tile_of(const TileMapArgs &a, int rr, int col) {
    if (rr >= a.h_r) return -1;
    const int rc = a.rank_c[col];
    if (rc >= a.h_c) return -1;
    return (rr >> 7) * a.nt_c + (rc >> 7);
}

__global__ __launch_bounds__(kBlock) void k_tile_hist(TileMapArgs a, int32_t *__restrict__ hist) {
    const int chunk = wave_chunk();
    if (chunk >= a.n.n_chunks) return;
    walk_chunk(a.n, chunk, threadIdx.x & 63, [&](int i) { return a.rank_r[i]; },
               [&](int k, int rr) {
                   const int t = tile_of(a, rr, a.n.col_idx[k]);
                   if (t >= 0) atomicAdd(&hist[t], 1);
               });
}

// sel[t] = 1 where tile t holds at least min_count entries (sel[n_tiles] = 0, the slot that receives the total of the scan)
__global__ void k_tile_flags(const int32_t *__restrict__ hist, int n_tiles, int min_count, int32_t *__restrict__ sel) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t <= n_tiles) sel[t] = (t < n_tiles && hist[t] >= min_count) ? 1 : 0;
}

// after the exclusive scan of sel: slot numbers of the kept tiles (row-major, so the slots of one row of tiles are
// consecutive), the column tile of every slot, the first slot of every row of tiles
__global__ void k_tile_slots(const int32_t *__restrict__ hist, const int32_t *__restrict__ sel_scan, int n_tiles, int nt_r, int nt_c,
                             int min_count, int32_t *__restrict__ slot_of, int32_t *__restrict__ slot_ct, int32_t *__restrict__ slot_rt,
                             int32_t *__restrict__ rt_ptr) {
    const int t = blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n_tiles) {
        const bool kept = hist[t] >= min_count;
        slot_of[t] = kept ? sel_scan[t] : -1;
        if (kept) {
            slot_ct[sel_scan[t]] = t % nt_c;
            slot_rt[sel_scan[t]] = t / nt_c;
        }
    }
    if (t <= nt_r) rt_ptr[t] = sel_scan[(long long)t * nt_c < n_tiles ? t * nt_c : n_tiles];
}

// bit (row, column) of its tile for every entry inside a kept tile; flag[k] = 1 for the entries that stay sparse;
// where[k] = -(cell + 1) for an entry inside a kept tile, cell = (slot * 128 + row in tile) * 128 + column in tile (-1 when that
// does not fit 31 bits; the entries that stay sparse get their place in the remainder later)
__global__ __launch_bounds__(kBlock) void k_tile_mark(TileMapArgs a, const int32_t *__restrict__ slot_of, unsigned *__restrict__ bits,
                                                       int32_t *__restrict__ flag, int32_t *__restrict__ where) {
    const int chunk = wave_chunk();
    if (chunk >= a.n.n_chunks) return;
    walk_chunk(a.n, chunk, threadIdx.x & 63, [&](int i) { return a.rank_r[i]; },
               [&](int k, int rr) {
                   const int col = a.n.col_idx[k];
                   const int t = tile_of(a, rr, col);
                   const int slot = t >= 0 ? slot_of[t] : -1;
                   if (slot >= 0) {
                       const int rc = a.rank_c[col];
                       atomicOr(&bits[((size_t)slot * 128 + (rr & 127)) * 4 + ((rc & 127) >> 5)], 1u << (rc & 31));
                       where[k] = slot < kMaxCellSlots ? -(((slot * 128 + (rr & 127)) * 128 + (rc & 127)) + 1) : -1;
                   }
                   flag[k] = slot >= 0 ? 0 : 1;
               });
}

// pos = exclusive scan of flag over nnz + 1 slots: entry k stays sparse iff pos[k + 1] != pos[k], at place pos[k]
__global__ __launch_bounds__(kBlock) void k_rem_scatter(NnzArgs a, const int32_t *__restrict__ pos, int32_t *__restrict__ col_rem,
                                                         int32_t *__restrict__ dst_rem) {
    const long long k = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (k >= a.nnz) return;
    const int p = pos[k];
    if (pos[k + 1] != p) {  // stays sparse; the others keep the (negative) cell code k_tile_mark gave them
        col_rem[p] = a.col_idx[k];
        dst_rem[k] = p;
    }
}

__global__ void k_rem_rowptr(const int32_t *__restrict__ row_ptr, int n_rows, const int32_t *__restrict__ pos, int32_t *__restrict__ row_ptr_rem) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i <= n_rows) row_ptr_rem[i] = pos[row_ptr[i]];
}

__global__ void k_zero_f32(float *__restrict__ p, long long n4) {  // n4 groups of four floats, 16-byte aligned
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n4) reinterpret_cast<float4 *>(p)[t] = make_float4(0.f, 0.f, 0.f, 0.f);
}

__global__ void k_zero_rows(float *__restrict__ C, long long n, int f, long long ldc) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n * f) C[(t / f) * ldc + (t % f)] = 0.f;
}

inline unsigned blocks_by_xcd(long long n_chunks) { return (unsigned)((n_chunks + kXcds * kWavesPerBlock - 1) / (kXcds * kWavesPerBlock)) * kXcds; }
inline unsigned blocks_for(long long n, int per_block) { return (unsigned)((n + per_block - 1) / per_block); }

// ------------------------------------------------------- backward of the attention layer

// adds the carried pieces of rows that span several chunks, in the order of k_softmax_fixup
__global__ __launch_bounds__(kBlock) void k_sum_fixup(NnzArgs a, float *__restrict__ out, const float *__restrict__ carry) {
    const int lane = threadIdx.x & 63;
    fixup_rows(a,
               [&](int i, int c, int c_last) {
                   float s = out[i];
                   for (int cc = c; cc <= c_last; ++cc) s += carry[cc];
                   out[i] = s;
               },
               [&](int i, int c, int c_last) {
                   float s = 0.f;
                   for (int cc = c + lane; cc <= c_last; cc += 64) s += carry[cc];
#pragma unroll
                   for (int off = 1; off < 64; off <<= 1) s += __shfl_xor(s, off, 64);
                   if (lane == 0) out[i] += s;
               });
}

// where an entry's weight goes: to its place among the entries outside kept tiles (dst_rem < 0: inside one), itself looked up in `place` where
// those have an order of their own
struct RemWeights {
    const int32_t *dst_rem;
    const int32_t *place;
    float *out;
};

// out[i] = sum of val over the stored entries of row i.  2.1 M values at stride 2, 100,000 rows: 173 -> 7 us.  COMPACT: val is the second of
// the pairs (alpha, ds), and the first is copied into the remainder's order in the same pass; the kernel is bound by the pairs' bytes, which a
// pass for the copy read again (GAT training on 115 M entries, where it runs beside the tiles' products: 17.44 -> 17.37 ms).
template <int PER, bool COMPACT>
__global__ __launch_bounds__(kBlock) void k_row_sum(NnzArgs a, const float *__restrict__ val, int stride, float *__restrict__ out,
                                                     float *__restrict__ carry, RemWeights rem) {
    __shared__ FlatLds<PER> lds;
    const int chunk = wave_chunk(), lane = threadIdx.x & 63;
    if (chunk >= a.n_chunks) return;
    float vs[PER], v[PER], w[COMPACT ? PER : 1];
    int to[COMPACT ? PER : 1];
    if (a.nnz > 0) {
        const ChunkSpan<PER> span(a, chunk);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const size_t k = span.at(u, lane);
            if constexpr (COMPACT) {
                const float2 p = reinterpret_cast<const float2 *>(val)[k];
                w[u] = p.x;
                vs[u] = p.y;
                to[u] = span.lo + u * 64 + lane < span.hi ? rem.dst_rem[k] : -1;
            } else {
                vs[u] = val[k * stride];
            }
        }
        if constexpr (COMPACT) {
            if (rem.place) {
#pragma unroll
                for (int u = 0; u < PER; ++u)
                    if (to[u] >= 0) to[u] = rem.place[to[u]];
            }
#pragma unroll
            for (int u = 0; u < PER; ++u)
                if (to[u] >= 0) rem.out[to[u]] = w[u];
        }
    }
    const FlatChunk<PER> c = flat_rows<PER>(a, chunk, lane, lds.row[threadIdx.x >> 6], [&](int r0, bool none) { if (none) out[r0 + lane] = 0.f; });
    if (c.lo >= c.hi) return;
#pragma unroll
    for (int u = 0; u < PER; ++u)
        if (c.lo + u * 64 + lane >= c.hi) vs[u] = 0.f;
    to_blocked<PER>(lds.val[threadIdx.x >> 6], lane, vs, v);
    flat_sum<PER>(c, lane, v, [&](int i, float t, int) {
        if (c.cont && i == c.i_first) carry[chunk] = t;
        else out[i] = t;
    });
}

// ---- per-entry sums over 32-column slices of a vector of the entry's row and one of its column (the general g-SDDMM of Eq. 2)
//
// Four lanes take one entry: lane `sub` of the four reads columns 4 sub .. 4 sub + 3 and 16 + 4 sub .. 16 + 4 sub + 3 of a slice, so each of the two
// loads of an entry covers 64 contiguous bytes.  A group of four lanes owns a sixteenth of the chunk, consecutive entries (those of its own lanes in
// blocked order), and keeps the vectors of the row it is in in registers, those of the row after it already under way: what is
// gathered per entry is the column's vector alone.  Before, consecutive entries went to neighbouring groups and the row's vector was gathered like the
// column's; it hit the vector cache, but the path from there, 64 bytes a clock and compute unit, is what bounds these kernels once the
// slice sits in the L2s: scores of 3 M entries x 64 columns
// 63 -> 48 us, dot products with the row sums behind them 64 -> 54 (both slices in one launch now).
// LDS words of a chunk lie in flat_at<PER, 4, 16> order (four words free after each group's part).
struct Lane8 { float4 lo, hi; };   // a lane's eight columns of a slice
__device__ __forceinline__ Lane8 load8(const float *slice, int row) {   // slice: offset by 4 sub columns
    const float *p = reinterpret_cast<const float *>(reinterpret_cast<const char *>(slice) + ((size_t)(unsigned)row << 7));
    return {*reinterpret_cast<const float4 *>(p), *reinterpret_cast<const float4 *>(p + 16)};
}
__device__ __forceinline__ float dot8(const Lane8 &a, const Lane8 &b) {
    return fmaf(b.lo.x, a.lo.x, fmaf(b.lo.y, a.lo.y, fmaf(b.lo.z, a.lo.z, fmaf(b.lo.w, a.lo.w, fmaf(b.hi.x, a.hi.x, fmaf(b.hi.y, a.hi.y, fmaf(b.hi.z, a.hi.z, b.hi.w * a.hi.w)))))));
}
template <int PER> constexpr int kPairWords = 64 * PER + 64;
template <int PER> __device__ __forceinline__ int pair_at(int p) { return flat_at<PER, 4, 16>(p); }

// words[pair_at(p)] = the row of entry p, sign bit: it is the first of its row in the chunk.  The place behind the chunk's last entry has the bit too: what
// is read there and after it (some other entry's column) makes up a piece of its own, which no row gets.
template <int PER>
__device__ __forceinline__ void pair_words(const FlatChunk<PER> &c, int lane, int *words) {
    const int end = c.hi - c.lo - lane * PER;
#pragma unroll
    for (int e = 0; e < PER; ++e) words[pair_at<PER>(lane * PER + e)] = (int)((unsigned)c.rid[e] | ((((c.starts >> e) & 1u) | (e == end ? 1u : 0u)) << 31));
}

// total(at, sums) once per entry of the chunk, by the one of its four lanes that owns it (at: its place in LDS): N sums over the slice's 32 columns, of
// what inner(own, column's vector, parts) leaves in each lane.  load_own(row, own) fetches the OWN vectors of a row.
template <int PER, int OWN, int N, class LoadOwn, class Inner, class Total>
__device__ __forceinline__ void pair_dots(const FlatChunk<PER> &c, const int *cols, const int *words, int lane, const float *other, LoadOwn load_own, Inner inner, Total total) {
    constexpr int PART = 4 * PER, H = OWN == 1 ? 4 : 2;   // entries whose vectors are under way: with two of the row's, registers for two
    const int sub = lane & 3, part0 = (lane >> 2) * (PART + 4);
    const bool up = (sub & 2) != 0, odd = (sub & 1) != 0;
    Lane8 own[OWN];
#pragma unroll 1
    for (int s = 0; s < PART; s += 4) {
        const int4 c4 = *reinterpret_cast<const int4 *>(&cols[part0 + s]), w4 = *reinterpret_cast<const int4 *>(&words[part0 + s]);
        const int col[4] = {c4.x, c4.y, c4.z, c4.w};
        const int word[4] = {s > 0 ? w4.x : (int)((unsigned)w4.x | 0x80000000u), w4.y, w4.z, w4.w};   // a part begins with a row to load
        float d[N][4];
#pragma unroll
        for (int h = 0; h < 4; h += H) {
            Lane8 b[H], fresh[H][OWN];   // fresh: read where the row changes, and nowhere else written
#pragma unroll
            for (int q = 0; q < H; ++q) if (word[h + q] < 0) load_own(word[h + q] & 0x7fffffff, fresh[q]);
#pragma unroll
            for (int q = 0; q < H; ++q) b[q] = load8(other, col[h + q]);
#pragma unroll
            for (int q = 0; q < H; ++q) {
                if (word[h + q] < 0) {
#pragma unroll
                    for (int o = 0; o < OWN; ++o) own[o] = fresh[q][o];
                }
                float parts[N];
                inner(own, b[q], parts);
#pragma unroll
                for (int n = 0; n < N; ++n) d[n][h + q] = parts[n];
            }
            if (H < 4) __builtin_amdgcn_sched_barrier(0);
        }
        // lanes 2, 3 of the four will own entries 2, 3: they keep d[2], d[3] and receive the partner's, and hand over d[0], d[1]
        float sums[N];
#pragma unroll
        for (int n = 0; n < N; ++n) {
            const float keep_a = up ? d[n][2] : d[n][0], keep_b = up ? d[n][3] : d[n][1];
            const float send_a = up ? d[n][0] : d[n][2], send_b = up ? d[n][1] : d[n][3];
            const float a2 = keep_a + dpp_f32<0x4E>(send_a);   // from lane ^ 2
            const float b2 = keep_b + dpp_f32<0x4E>(send_b);
            const float keep = odd ? b2 : a2, send = odd ? a2 : b2;
            sums[n] = keep + dpp_f32<0xB1>(send);              // from lane ^ 1: the sum over the four lanes for entry s + sub
        }
        total(part0 + s + sub, sums);
    }
}

// Sums over the rows of the chunk of what add(weights, q, own, column's vector, acc) adds per entry to NA accumulators a lane: a group of four lanes walks its
// part as in pair_dots and closes a row (close(row, extra, acc)) where the next one starts; the first row a group closes waits for what the
// groups before it are left with (a scan over the groups), as does its last one where it ends with the part.  weights(at) fetches what two entries weigh from
// LDS, load_own(row, own, extra) a row's vector and one more number.  The places behind the chunk's n_entries are walked like entries and left out (0 times an infinite
// or undefined vector is no 0).  Two entries at a time: with four the registers leave three wavefronts a SIMD
// (a training pass of four heads on 2.1 M entries 614 us, with two 589; this walk 155 us with eight lanes an entry and the own row gathered per entry, now 124).
template <int PER, int NA, class Weights, class LoadOwn, class Add, class Close>
__device__ __forceinline__ void pair_sums(int n_entries, const int *cols, const int *words, int lane, const float *other, Weights weights, LoadOwn load_own, Add add, Close close) {
    constexpr int PART = 4 * PER, U = 2;
    const int g = lane >> 2, part0 = g * (PART + 4);
    float acc[NA], head[NA], extra = 0.f, head_extra = 0.f;
    int row = 0, head_row = -1;
    Lane8 own;
#pragma unroll
    for (int n = 0; n < NA; ++n) acc[n] = head[n] = 0.f;
    auto finish = [&] {
        if (head_row < 0) {
#pragma unroll
            for (int n = 0; n < NA; ++n) head[n] = acc[n];
            head_extra = extra;
            head_row = row;
        } else {
            close(row, extra, acc);
        }
#pragma unroll
        for (int n = 0; n < NA; ++n) acc[n] = 0.f;
    };
#pragma unroll 1
    for (int s = 0; s < PART; s += U) {
        int col[U], word[U];
        const auto w = weights(part0 + s);
        const int2 c2 = *reinterpret_cast<const int2 *>(&cols[part0 + s]), w2 = *reinterpret_cast<const int2 *>(&words[part0 + s]);
        col[0] = c2.x; col[1] = c2.y;
        word[0] = w2.x; word[1] = w2.y;
        if (s == 0) word[0] = (int)((unsigned)word[0] | 0x80000000u);   // a part begins with a row to load
        Lane8 fresh[U], b[U];   // fresh: read where the row changes, and nowhere else written
        float fresh_extra[U];
#pragma unroll
        for (int q = 0; q < U; ++q) if (word[q] < 0) load_own(word[q] & 0x7fffffff, fresh[q], fresh_extra[q]);
#pragma unroll
        for (int q = 0; q < U; ++q) b[q] = load8(other, col[q]);
#pragma unroll
        for (int q = 0; q < U; ++q) {
            if (word[q] < 0) {
                if (q > 0 || s > 0) finish();
                own = fresh[q];
                extra = fresh_extra[q];
                row = word[q] & 0x7fffffff;
            }
            add(w, q, own, b[q], acc);
        }
    }
    if (g == 15 ? n_entries == 64 * PER : words[part0 + PART + 4] < 0) finish();
    int f = head_row >= 0;
    auto step = [&](float (&x)[NA], int of) {
#pragma unroll
        for (int n = 0; n < NA; ++n) acc[n] += f ? 0.f : x[n];
        f |= of;
    };
    float x[NA];
#pragma unroll
    for (int n = 0; n < NA; ++n) x[n] = dpp_f32<0x114>(acc[n]);
    step(x, dpp_i32<0x114>(f));
#pragma unroll
    for (int n = 0; n < NA; ++n) x[n] = dpp_f32<0x118>(acc[n]);
    step(x, dpp_i32<0x118>(f));
    // the last group of the first and third sixteen lanes to the second and fourth, then that of the second to both behind it
#pragma unroll
    for (int half = 16; half < 64; half <<= 1) {
        const int from = ((half == 16 ? (lane & 48) - 4 : 28) + (lane & 3)) * 4;
        const bool takes = (lane & half) != 0;
#pragma unroll
        for (int n = 0; n < NA; ++n) { const float y = lane_read(from, acc[n]); x[n] = takes ? y : 0.f; }
        const int of = lane_read(from, f);
        step(x, takes ? of : 0);
    }
#pragma unroll
    for (int n = 0; n < NA; ++n) { const float y = __shfl_up(acc[n], 4, 64); if (g > 0) head[n] += y; }
    if (head_row >= 0) close(head_row, head_extra, head);
}

struct GatBwdArgs {
    NnzArgs n;
    const float *theta, *dP;  // slice-major (tiles of 32 columns): Theta over the source nodes, dP over the destinations
    const float *logits;      // e_ij per stored entry
    const float2 *mz;         // per row: (max logit, sum of exp(logit - max))
    float *dalpha;            // out, per stored entry: <dP_i, Theta_j>
    float *rowdot, *carry;    // out, per row: sum_j alpha_ij dalpha_ij (+ per-chunk carry slots)
    long long theta_tile, dp_tile;  // floats from one tile to the next
    int n_tiles;
    int dp_rows;  // rows of dP; row r of the pattern is row r mod dp_rows (r >= dp_rows: a segment of a panel-major pattern)
    float scale;  // factor on every dot product (1 in the attention backward; the 1 / sqrt(d) of a key-query score)
};

// dalpha_ij = <dP[i,:], Theta[j,:]> for every stored entry (Eq. 2 with a dot product as the inner operator) together
// with the row sums sum_j alpha_ij dalpha_ij that the softmax backward needs.  A launch takes the 32-column slices t0 .. t1 - 1 (launch_gat_dalpha:
// one, so that every wavefront of the GPU gathers from the same contiguous slice of Theta, or all of a small Theta) and adds to what the launches before
// it left in dalpha: they follow each other on the stream, so no atomics.  The last launch sees the complete dot products and forms the row sums.
template <bool LAST, int PER>
__global__ __launch_bounds__(kBlock) void k_gat_dalpha(GatBwdArgs a, int t0, int t1) {
    __shared__ __attribute__((aligned(16))) int s_col[kWavesPerBlock][kPairWords<PER>], s_word[kWavesPerBlock][kPairWords<PER>];
    __shared__ __attribute__((aligned(16))) float s_val[kWavesPerBlock][kPairWords<PER>];
    const int chunk = wave_chunk(), wave = threadIdx.x >> 6;
    if (chunk >= a.n.n_chunks) return;
    const int lane = threadIdx.x & 63, sub = lane & 3;
    int *cols = s_col[wave], *words = s_word[wave];
    float *val = s_val[wave];
    float es[LAST ? PER : 1], sum[PER];
    int col[PER];
    if (a.n.nnz > 0) {
        const ChunkSpan<PER> span(a.n, chunk);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int k = span.at(u, lane);
            col[u] = a.n.col_idx[k];
            sum[u] = t0 > 0 ? a.dalpha[k] : 0.f;
            if (LAST) es[LAST ? u : 0] = a.logits[k];
        }
    }
    const FlatChunk<PER> c = flat_rows<PER, 4, 16>(a.n, chunk, lane, words, [&](int r0, bool none) { if (LAST && none) a.rowdot[r0 + lane] = 0.f; });
    if (c.lo >= c.hi) return;
    pair_words<PER>(c, lane, words);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        cols[pair_at<PER>(u * 64 + lane)] = col[u];
        val[pair_at<PER>(u * 64 + lane)] = sum[u];
    }
    lds_exchange();
    const int panel_row = c.i_first / a.dp_rows * a.dp_rows;   // first row of the panel the chunk begins in
    for (int tile = t0; tile < t1; ++tile) {
        const float *dP = a.dP + (size_t)tile * a.dp_tile + sub * 4;
        pair_dots<PER, 1, 1>(c, cols, words, lane, a.theta + (size_t)tile * a.theta_tile + sub * 4,
                             [&](int i, Lane8 (&own)[1]) {
                                 i -= panel_row;
                                 while (i >= a.dp_rows) i -= a.dp_rows;   // only where a chunk runs over the end of its panel
                                 own[0] = load8(dP, i);
                             },
                             [&](const Lane8 (&own)[1], const Lane8 &b, float (&parts)[1]) { parts[0] = dot8(own[0], b) * a.scale; },   // exact when the factor is 1
                             [&](int at, const float (&sums)[1]) { val[at] += sums[0]; });
    }
    lds_exchange();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int at = pair_at<PER>(u * 64 + lane), k = c.lo + u * 64 + lane;
        if (k < c.hi) a.dalpha[k] = val[at];
        if (LAST) cols[at] = __float_as_int(es[LAST ? u : 0]);
    }
    if (LAST) {
        float v[PER];
        lds_exchange();
        const int n_mine = c.hi - c.lo - lane * PER;
#pragma unroll
        for (int e = 0; e < PER; ++e) {
            const int at = pair_at<PER>(lane * PER + e);
            const float2 st = a.mz[c.rid[e]];
            v[e] = e < n_mine ? expf(__int_as_float(cols[at]) - st.x) * inv_z(st.y) * val[at] : 0.f;
        }
        flat_sum<PER>(c, lane, v, [&](int i, float t, int) {
            if (c.cont && i == c.i_first) a.carry[chunk] = t;
            else a.rowdot[i] = t;
        });
    }
}

// dalpha of every stored entry from its two sources when the pattern carries a dense-tile split: where[k] >= 0 is the place of
// entry k in the remainder (dalpha_rem, or with `place` dalpha_rem[place[.]]: the remainder's panel-major order), a negative value -(cell + 1) the cell of the dense product Dt that holds it.  Writes
// dalpha in the order of the pattern and forms the row sums sum_j alpha_ij dalpha_ij.
template <int PER>
__global__ __launch_bounds__(kBlock) void k_gat_dalpha_merge(NnzArgs a, const int32_t *__restrict__ where, const int32_t *__restrict__ place, const float *__restrict__ dalpha_rem,
                                                              const float *__restrict__ Dt, const float *__restrict__ logits,
                                                              const float2 *__restrict__ mz, float *__restrict__ dalpha,
                                                              float *__restrict__ rowdot, float *__restrict__ carry) {
    __shared__ FlatLds<PER> lds;
    const int chunk = wave_chunk(), lane = threadIdx.x & 63;
    if (chunk >= a.n_chunks) return;
    int *rows = lds.row[threadIdx.x >> 6];
    int w[PER];
    float e[PER], v[PER], s[PER];
    if (a.nnz > 0) {
        const ChunkSpan<PER> span(a, chunk);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int k = span.at(u, lane);
            w[u] = where[k];
            e[u] = logits[k];
        }
        if (place) {
#pragma unroll
            for (int u = 0; u < PER; ++u) w[u] = w[u] >= 0 ? place[w[u]] : w[u];
        }
#pragma unroll
        for (int u = 0; u < PER; ++u) v[u] = w[u] >= 0 ? dalpha_rem[w[u]] : Dt[-(long long)w[u] - 1];
    }
    const FlatChunk<PER> c = flat_rows<PER>(a, chunk, lane, rows, [&](int r0, bool none) { if (none) rowdot[r0 + lane] = 0.f; });
    if (c.lo >= c.hi) return;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int k = c.lo + u * 64 + lane;
        const float2 st = mz[rows[u * 64 + lane]];
        s[u] = 0.f;
        if (k < c.hi) {
            dalpha[k] = v[u];
            s[u] = expf(e[u] - st.x) * inv_z(st.y) * v[u];
        }
    }
    float b[PER];
    to_blocked<PER>(lds.val[threadIdx.x >> 6], lane, s, b);
    flat_sum<PER>(c, lane, b, [&](int i, float t, int) {
        if (c.cont && i == c.i_first) carry[chunk] = t;
        else rowdot[i] = t;
    });
}

struct ScoreV2Args {
    NnzArgs n;
    const float *theta_l, *theta_r;  // slice-major: W_l x over the destinations, W_r x over the sources
    const float *att;                // attention vector padded with zeros to a multiple of 32
    float *logits;                   // out, per stored entry
    long long tl_tile, tr_tile;      // floats from one tile to the next
    float slope;
};

// Logits of the GATv2 score, e_ij = sum_m a[m] LeakyReLU(Theta_l[i, m] + Theta_r[j, m]): Eq. 2 with an inner operator
// that is neither a product nor a sum alone.  Slices as in k_gat_dalpha.
template <int PER>
__global__ __launch_bounds__(kBlock) void k_score_v2(ScoreV2Args a, int t0, int t1) {
    __shared__ __attribute__((aligned(16))) int s_col[kWavesPerBlock][kPairWords<PER>], s_word[kWavesPerBlock][kPairWords<PER>];
    __shared__ __attribute__((aligned(16))) float s_val[kWavesPerBlock][kPairWords<PER>];
    const int chunk = wave_chunk(), wave = threadIdx.x >> 6;
    if (chunk >= a.n.n_chunks) return;
    const int lane = threadIdx.x & 63, sub = lane & 3;
    int *cols = s_col[wave], *words = s_word[wave];
    float *val = s_val[wave];
    float sum[PER];
    int col[PER];
    const ChunkSpan<PER> span(a.n, chunk);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int k = span.at(u, lane);
        col[u] = a.n.col_idx[k];
        sum[u] = t0 > 0 ? a.logits[k] : 0.f;
    }
    const FlatChunk<PER> c = flat_rows<PER, 4, 16>(a.n, chunk, lane, words, [](int, bool) {});
    if (c.lo >= c.hi) return;
    pair_words<PER>(c, lane, words);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        cols[pair_at<PER>(u * 64 + lane)] = col[u];
        val[pair_at<PER>(u * 64 + lane)] = sum[u];
    }
    lds_exchange();
    const float slope = a.slope;
    auto term = [&](float wt, float x, float y) {
        const float t = x + y;
        return wt * (t > 0.f ? t : slope * t);
    };
    for (int tile = t0; tile < t1; ++tile) {
        const float *theta_l = a.theta_l + (size_t)tile * a.tl_tile + sub * 4;
        const Lane8 w = load8(a.att + tile * 32 + sub * 4, 0);
        pair_dots<PER, 1, 1>(c, cols, words, lane, a.theta_r + (size_t)tile * a.tr_tile + sub * 4, [&](int i, Lane8 (&own)[1]) { own[0] = load8(theta_l, i); },
                             [&](const Lane8 (&own)[1], const Lane8 &b, float (&parts)[1]) {
                                 const Lane8 &p = own[0];
                                 parts[0] = ((term(w.lo.x, p.lo.x, b.lo.x) + term(w.lo.y, p.lo.y, b.lo.y)) + (term(w.lo.z, p.lo.z, b.lo.z) + term(w.lo.w, p.lo.w, b.lo.w))) +
                                            ((term(w.hi.x, p.hi.x, b.hi.x) + term(w.hi.y, p.hi.y, b.hi.y)) + (term(w.hi.z, p.hi.z, b.hi.z) + term(w.hi.w, p.hi.w, b.hi.w)));
                             },
                             [&](int at, const float (&sums)[1]) { val[at] += sums[0]; });
    }
    lds_exchange();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int k = c.lo + u * 64 + lane;
        if (k < c.hi) a.logits[k] = val[pair_at<PER>(u * 64 + lane)];
    }
}

struct V2ScoresArgs {
    NnzArgs n;
    const float *theta_l, *theta_r, *dP, *att;   // dP over the destinations like theta_l
    float *logits, *dalpha;                      // out, per stored entry
    float2 *stats, *carry_stats;                 // out, per row: (max logit, sum of exp(logit - max)) (+ per-chunk carry slots)
    float *rowdot, *carry;                       // out, per row: sum_j alpha_ij dalpha_ij (+ per-chunk carry slots)
    long long tl_tile, tr_tile;
    float slope;
};

// What the backward of the GATv2 layer needs per entry, logit and <dP_i, Theta_r[j]>, from one gather of Theta_r[j], and the row's statistics and weighted sum
// behind them.  As k_score_v2, k_softmax_stats and k_gat_dalpha these were 123 us on 3 M entries x 64 columns, with their
// fix-ups, so 103.
template <bool LAST, int PER>
__global__ __launch_bounds__(kBlock) void k_v2_scores(V2ScoresArgs a, int t0, int t1) {
    __shared__ __attribute__((aligned(16))) int s_col[kWavesPerBlock][kPairWords<PER>], s_word[kWavesPerBlock][kPairWords<PER>];
    __shared__ __attribute__((aligned(16))) float s_e[kWavesPerBlock][kPairWords<PER>], s_d[kWavesPerBlock][kPairWords<PER>];
    const int chunk = wave_chunk(), wave = threadIdx.x >> 6;
    if (chunk >= a.n.n_chunks) return;
    const int lane = threadIdx.x & 63, sub = lane & 3;
    int *cols = s_col[wave], *words = s_word[wave];
    float *es = s_e[wave], *ds = s_d[wave];
    float e0[PER], d0[PER];
    int col[PER];
    if (a.n.nnz > 0) {
        const ChunkSpan<PER> span(a.n, chunk);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int k = span.at(u, lane);
            col[u] = a.n.col_idx[k];
            e0[u] = t0 > 0 ? a.logits[k] : 0.f;
            d0[u] = t0 > 0 ? a.dalpha[k] : 0.f;
        }
    }
    const FlatChunk<PER> c = flat_rows<PER, 4, 16>(a.n, chunk, lane, words, [&](int r0, bool none) {
        if (LAST && none) {
            a.stats[r0 + lane] = make_float2(-INFINITY, 0.f);
            a.rowdot[r0 + lane] = 0.f;
        }
    });
    if (c.lo >= c.hi) return;
    pair_words<PER>(c, lane, words);
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int at = pair_at<PER>(u * 64 + lane);
        cols[at] = col[u];
        es[at] = e0[u];
        ds[at] = d0[u];
    }
    lds_exchange();
    const float slope = a.slope;
    auto term = [&](float wt, float x, float y) {
        const float t = x + y;
        return wt * (t > 0.f ? t : slope * t);
    };
    for (int tile = t0; tile < t1; ++tile) {
        const float *theta_l = a.theta_l + (size_t)tile * a.tl_tile + sub * 4, *dP = a.dP + (size_t)tile * a.tl_tile + sub * 4;
        const Lane8 w = load8(a.att + tile * 32 + sub * 4, 0);
        pair_dots<PER, 2, 2>(c, cols, words, lane, a.theta_r + (size_t)tile * a.tr_tile + sub * 4,
                             [&](int i, Lane8 (&own)[2]) { own[0] = load8(theta_l, i); own[1] = load8(dP, i); },
                             [&](const Lane8 (&own)[2], const Lane8 &b, float (&parts)[2]) {
                                 const Lane8 &p = own[0];
                                 parts[0] = ((term(w.lo.x, p.lo.x, b.lo.x) + term(w.lo.y, p.lo.y, b.lo.y)) + (term(w.lo.z, p.lo.z, b.lo.z) + term(w.lo.w, p.lo.w, b.lo.w))) +
                                            ((term(w.hi.x, p.hi.x, b.hi.x) + term(w.hi.y, p.hi.y, b.hi.y)) + (term(w.hi.z, p.hi.z, b.hi.z) + term(w.hi.w, p.hi.w, b.hi.w)));
                                 parts[1] = dot8(own[1], b);
                             },
                             [&](int at, const float (&sums)[2]) { es[at] += sums[0]; ds[at] += sums[1]; });
    }
    lds_exchange();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int at = pair_at<PER>(u * 64 + lane), k = c.lo + u * 64 + lane;
        if (k < c.hi) {
            a.logits[k] = es[at];
            a.dalpha[k] = ds[at];
        }
    }
    if (!LAST) return;
    float e[PER], mx[PER], v[2][PER];
    const int n_mine = c.hi - c.lo - lane * PER;
#pragma unroll
    for (int q = 0; q < PER; ++q) e[q] = q < n_mine ? es[pair_at<PER>(lane * PER + q)] : -INFINITY;
    flat_piece_max<PER>(c, lane, e, mx);
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        mx[q] = fmaxf(mx[q], -FLT_MAX);   // entries of -inf weigh 0 also where a piece holds no others
        v[0][q] = q < n_mine ? expf(e[q] - mx[q]) : 0.f;
        v[1][q] = q < n_mine ? v[0][q] * ds[pair_at<PER>(lane * PER + q)] : 0.f;
    }
    const float m_before = lane_before(mx[PER - 1], 0.f);   // every entry of a piece has its maximum: it is taken from the last one
    const int last_row = __builtin_amdgcn_readfirstlane(__shfl(c.rid[PER - 1], 63, 64));
    const bool open = __builtin_amdgcn_readfirstlane(a.n.row_ptr[last_row + 1]) > c.hi;
    flat_sums<PER, 2>(c, lane, v, [&](int i, const float (&sum)[2], int, int last) {
        float m = last_value<PER>(mx, m_before, last);
        if (sum[0] == 0.f) m = -INFINITY;
        if (c.cont && i == c.i_first) {
            a.carry_stats[chunk] = make_float2(m, sum[0]);
            a.carry[chunk] = sum[1];
        } else {   // a row that goes on in the next chunk: its sum waits for the fix-up to be divided
            a.stats[i] = make_float2(m, sum[0]);
            a.rowdot[i] = open && i == last_row ? sum[1] : sum[1] * inv_z(sum[0]);
        }
    });
}

struct V2Piece { float m, z, a; };
__device__ __forceinline__ void merge_v2(V2Piece &p, const V2Piece &q) {
    const float m = p.m > q.m ? p.m : q.m;
    if (m == -INFINITY) { p.m = m; return; }   // neither has entries that weigh anything
    const float kp = expf(p.m - m), kq = expf(q.m - m);
    p.z = p.z * kp + q.z * kq;
    p.a = p.a * kp + q.a * kq;
    p.m = m;
}
// the rows that span several chunks, their pieces in chunk order or (long rows) lane by lane and then over the lanes
__global__ __launch_bounds__(kBlock) void k_v2_scores_fixup(V2ScoresArgs a) {
    const int lane = threadIdx.x & 63;
    auto load = [&](int c) { const float2 p = a.carry_stats[c]; return V2Piece{p.x, p.y, a.carry[c]}; };
    auto finish = [&](int i, const V2Piece &rest) {
        const float2 st = a.stats[i];
        V2Piece p = {st.x, st.y, a.rowdot[i]};
        merge_v2(p, rest);
        a.stats[i] = make_float2(p.z == 0.f ? -INFINITY : p.m, p.z);
        a.rowdot[i] = p.a * inv_z(p.z);
    };
    fixup_rows(a.n,
               [&](int i, int c, int c_last) {
                   V2Piece p = load(c);
                   for (int cc = c + 1; cc <= c_last; ++cc) merge_v2(p, load(cc));
                   finish(i, p);
               },
               [&](int i, int c, int c_last) {
                   V2Piece p = {-INFINITY, 0.f, 0.f};
                   for (int cc = c + lane; cc <= c_last; cc += 64) merge_v2(p, load(cc));
#pragma unroll
                   for (int off = 1; off < 64; off <<= 1) merge_v2(p, V2Piece{__shfl_xor(p.m, off, 64), __shfl_xor(p.z, off, 64), __shfl_xor(p.a, off, 64)});
                   if (lane == 0) finish(i, p);
               });
}

struct GatDtArgs {
    NnzArgs n;
    const float *logits, *dalpha, *rowdot;
    const float2 *mz;
    const int32_t *t_pos;   // place of entry k in the transposed pattern
    float *dt;              // SUMS: not written, may be null
    float2 *adt_t;          // (alpha, dt) at the entry's place in the transposed pattern: one 8-byte scattered store
    float *rowsum, *carry;  // SUMS: row sums of dt (+ per-chunk carry slots)
    float slope;
};

// Softmax and LeakyReLU backward per stored entry: alpha = exp(e - m_i) / z_i, de = alpha (dalpha - rowdot_i),
// dt = de * (e > 0 ? 1 : slope) (e > 0 exactly when the pre-activation is).  (alpha, dt) is written at the entry's place in the transposed
// pattern (for ds_r and alpha^T dP); in row order dt is either kept, or summed over the rows at once (SUMS: ds_l).
// The scattered stores bound it: entries of consecutive rows go to consecutive places of a transposed row, so a line fills up over many
// rows, and with neighbouring chunks on different XCDs every L2 holds a piece of it and writes it out by itself.  Chunks are therefore
// given out so that an XCD has one range of them (2.1 M entries with the row sums 32 + 7 -> 27 us, 3 M entries without 53 -> 47).
template <bool SUMS, int PER>
__global__ __launch_bounds__(kBlock) void k_gat_dt(GatDtArgs a) {
    __shared__ FlatLds<PER> lds;
    const int chunk = wave_chunk_by_xcd(), lane = threadIdx.x & 63;
    if (chunk >= a.n.n_chunks) return;
    int *rows = lds.row[threadIdx.x >> 6];
    float e[PER], da[PER], t[PER];
    int p[PER];
    if (a.n.nnz > 0) {
        const ChunkSpan<PER> span(a.n, chunk);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int k = span.at(u, lane);
            e[u] = a.logits[k];
            da[u] = a.dalpha[k];
            p[u] = a.t_pos[k];
        }
    }
    const FlatChunk<PER> c = flat_rows<PER>(a.n, chunk, lane, rows, [&](int r0, bool none) { if (SUMS && none) a.rowsum[r0 + lane] = 0.f; });
    if (c.lo >= c.hi) return;
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int k = c.lo + u * 64 + lane, i = rows[u * 64 + lane];
        const float2 st = a.mz[i];
        const float al = expf(e[u] - st.x) * inv_z(st.y);
        const float dt = al * (da[u] - a.rowdot[i]) * (e[u] > 0.f ? 1.f : a.slope);
        t[u] = 0.f;
        if (k < c.hi) {
            if (SUMS) t[u] = dt;
            else a.dt[k] = dt;
            a.adt_t[p[u]] = make_float2(al, dt);
        }
    }
    if (SUMS) {
        float v[PER];
        to_blocked<PER>(lds.val[threadIdx.x >> 6], lane, t, v);
        flat_sum<PER>(c, lane, v, [&](int i, float sum, int) {
            if (c.cont && i == c.i_first) a.carry[chunk] = sum;
            else a.rowsum[i] = sum;
        });
    }
}

// ---- backward of attention heads that are one slice wide (at most 32 columns), every head in one launch (blockIdx.y)
//
// Two walks and nothing stored per entry.  Over the rows of the pattern (k_gat_head_rows): logits and softmax statistics of the row, the dot
// products dalpha_ij = <dP_i, Theta_j>, and from them rowdot_i = sum_j alpha_ij dalpha_ij and ds_l[i] = sum_j dt_ij.  Over the rows of the
// transposed pattern (k_gat_head_cols): the coefficients again from the scores and the row's statistics, the dot product of the gathered row of
// dP with the row's own Theta_j, dt_ij = alpha_ij (dalpha_ij - rowdot_i) LeakyReLU'(e_ij), and with them ds_r[j] = sum_i dt_ij and dTheta_j =
// sum_i alpha_ij dP_i + ds_l[j] a_l + ds_r[j] a_r.  Before, dalpha was stored, and a pass over the rows left (alpha, dt) at its place in the transposed pattern for another two
// passes over that: the scattered stores, and 24 bytes per entry and head written and read.
//
// ds_l needs rowdot, a sum over the same row, before it can weigh an entry.  With P and N the entries of the row with a positive logit and the
// others, LeakyReLU' is 1 on P and `slope` on N, and since alpha sums to 1, sum_j alpha (dalpha - rowdot) = 0, so
//   ds_l = (1 - slope) (A_P - rowdot Z_P) = -(1 - slope) (A_N - rowdot Z_N),   A = sum of alpha dalpha, Z = sum of alpha over the set:
// four sums in one walk, and the set that weighs less is used (a row of one sign only gives exactly 0, as it should).
struct GatHeadArgs {
    NnzArgs n;                      // the pattern, or its transpose (k_gat_head_cols)
    const float *theta, *dP;        // slice h belongs to head h: Theta over the sources, dP over the destinations, padded with zeros to 32 columns
    const float *s_l, *s_r;         // per head, n_src floats apart
    float4 *row;                    // per head, n_dst apart: (s_l, maximum, 1 / sum of exp, rowdot) of every destination
    const float *a_l, *a_r;         // d floats a head
    float *ds_l, *ds_r;             // per head, n_src apart
    float *piece;                   // per head, chunk and kind (continued, open): (m, Z_P, Z_N, A_P, A_N) of a piece of a row that spans chunks, 8 floats
    float *dtheta;                  // k_gat_head_cols: head h's columns start at h * d
    float *carry, *ds_carry;        // per head and chunk: the piece of the continued row (32 floats; one float)
    long long n_src, n_dst, ldd;
    int d, store_vec_ok;
    float slope;
};

struct HeadPiece { float m, zp, zn, ap, an; };
__device__ __forceinline__ void merge_piece(HeadPiece &a, const HeadPiece &b) {
    const float m = a.m > b.m ? a.m : b.m;
    if (m == -INFINITY) { a.m = m; return; }   // neither has entries that weigh anything
    const float ka = expf(a.m - m), kb = expf(b.m - m);
    a.zp = a.zp * ka + b.zp * kb;
    a.zn = a.zn * ka + b.zn * kb;
    a.ap = a.ap * ka + b.ap * kb;
    a.an = a.an * ka + b.an * kb;
    a.m = m;
}
__device__ __forceinline__ void finish_head_row(const GatHeadArgs &a, int head, int i, const HeadPiece &p) {
    const float z = p.zp + p.zn, iz = inv_z(z), rowdot = (p.ap + p.an) * iz;
    a.row[head * a.n_dst + i] = make_float4(a.s_l[head * a.n_src + i], z == 0.f ? -INFINITY : p.m, iz, rowdot);
    const float t = p.zn < p.zp ? rowdot * p.zn - p.an : p.ap - rowdot * p.zp;
    a.ds_l[head * a.n_src + i] = (1.f - a.slope) * iz * t;
}

template <int PER>
__global__ __launch_bounds__(kBlock) void k_gat_head_rows(GatHeadArgs a) {
    __shared__ __attribute__((aligned(16))) int s_col[kWavesPerBlock][kPairWords<PER>], s_word[kWavesPerBlock][kPairWords<PER>];
    __shared__ __attribute__((aligned(16))) float s_val[kWavesPerBlock][kPairWords<PER>];
    const int chunk = wave_chunk(), head = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, sub = lane & 3;
    if (chunk >= a.n.n_chunks) return;
    int *cols = s_col[wave], *words = s_word[wave];
    float *val = s_val[wave];
    const float *s_l = a.s_l + head * a.n_src, *s_r = a.s_r + head * a.n_src;
    float es[PER], p[PER], mx[PER];
    int col[PER];
    if (a.n.nnz > 0) {
        const ChunkSpan<PER> span(a.n, chunk);
#pragma unroll
        for (int u = 0; u < PER; ++u) col[u] = a.n.col_idx[span.at(u, lane)];
#pragma unroll
        for (int u = 0; u < PER; ++u) es[u] = s_r[col[u]];
    }
    const FlatChunk<PER> c = flat_rows<PER, 4, 16>(a.n, chunk, lane, words, [&](int r0, bool none) { if (none) a.ds_l[head * a.n_src + r0 + lane] = 0.f; });
    if (c.lo >= c.hi) return;
    unsigned neg = 0u;   // bit q: entry q of this lane (blocked order) has a logit of 0 or below
    {
        float e[PER];
        int rw[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) rw[u] = words[pair_at<PER>(u * 64 + lane)];
        row_values<PER>(c, lane, s_l, rw, e);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int at = pair_at<PER>(u * 64 + lane);
            val[at] = leaky(e[u] + es[u], a.slope);
            cols[at] = col[u];
        }
        lds_exchange();
        pair_words<PER>(c, lane, words);
        const int n_mine = c.hi - c.lo - lane * PER;
#pragma unroll
        for (int q = 0; q < PER; ++q) e[q] = q < n_mine ? val[pair_at<PER>(lane * PER + q)] : -INFINITY;
        flat_piece_max<PER>(c, lane, e, mx);
#pragma unroll
        for (int q = 0; q < PER; ++q) {
            mx[q] = fmaxf(mx[q], -FLT_MAX);   // entries of -inf weigh 0 also where a piece holds no others
            p[q] = q < n_mine ? expf(e[q] - mx[q]) : 0.f;
            neg |= (e[q] > 0.f ? 0u : 1u) << q;
        }
    }
    lds_exchange();
    const float *theta = a.theta + (size_t)head * a.n_src * 32 + sub * 4, *dP = a.dP + (size_t)head * a.n_dst * 32 + sub * 4;
    pair_dots<PER, 1, 1>(c, cols, words, lane, theta, [&](int i, Lane8 (&own)[1]) { own[0] = load8(dP, i); },
                         [](const Lane8 (&own)[1], const Lane8 &b, float (&parts)[1]) { parts[0] = dot8(own[0], b); },
                         [&](int at, const float (&sums)[1]) { val[at] = sums[0]; });
    lds_exchange();
    float v[4][PER];
#pragma unroll
    for (int q = 0; q < PER; ++q) {
        const float t = q < c.hi - c.lo - lane * PER ? p[q] * val[pair_at<PER>(lane * PER + q)] : 0.f;
        const bool n = (neg >> q) & 1u;
        v[0][q] = n ? 0.f : p[q];
        v[1][q] = n ? p[q] : 0.f;
        v[2][q] = n ? 0.f : t;
        v[3][q] = n ? t : 0.f;
    }
    const float m_before = lane_before(mx[PER - 1], 0.f);   // every entry of a piece has its maximum: it is taken from the last one
    const int last_row = __builtin_amdgcn_readfirstlane(__shfl(c.rid[PER - 1], 63, 64));
    const bool open = __builtin_amdgcn_readfirstlane(a.n.row_ptr[last_row + 1]) > c.hi;
    flat_sums<PER, 4>(c, lane, v, [&](int i, const float (&sum)[4], int, int last) {
        const float m = last_value<PER>(mx, m_before, last);
        const HeadPiece piece = {m, sum[0], sum[1], sum[2], sum[3]};
        const bool cont = c.cont && i == c.i_first;
        if (cont || (open && i == last_row)) {
            float *dst = a.piece + (((size_t)head * a.n.n_chunks + chunk) * 2 + (cont ? 0 : 1)) * 8;
            *reinterpret_cast<float4 *>(dst) = make_float4(piece.m, piece.zp, piece.zn, piece.ap);
            dst[4] = piece.an;
        } else {
            finish_head_row(a, head, i, piece);
        }
    });
}

// merges the pieces of rows that span several chunks, in chunk order or (long rows) lane by lane and then over the lanes
__global__ __launch_bounds__(kBlock) void k_gat_head_fixup(GatHeadArgs a) {
    const int head = blockIdx.y, lane = threadIdx.x & 63;
    auto load = [&](int chunk, int kind) {
        const float *src = a.piece + (((size_t)head * a.n.n_chunks + chunk) * 2 + kind) * 8;
        const float4 t = *reinterpret_cast<const float4 *>(src);
        return HeadPiece{t.x, t.y, t.z, t.w, src[4]};
    };
    fixup_rows(a.n,
               [&](int i, int c, int c_last) {
                   HeadPiece p = load(c - 1, 1);
                   for (int cc = c; cc <= c_last; ++cc) merge_piece(p, load(cc, 0));
                   finish_head_row(a, head, i, p);
               },
               [&](int i, int c, int c_last) {
                   HeadPiece p = {-INFINITY, 0.f, 0.f, 0.f, 0.f};
                   for (int cc = c + lane; cc <= c_last; cc += 64) merge_piece(p, load(cc, 0));
#pragma unroll
                   for (int off = 1; off < 64; off <<= 1)
                       merge_piece(p, HeadPiece{__shfl_xor(p.m, off, 64), __shfl_xor(p.zp, off, 64), __shfl_xor(p.zn, off, 64), __shfl_xor(p.ap, off, 64),
                                                __shfl_xor(p.an, off, 64)});
                   if (lane == 0) {
                       HeadPiece q = load(c - 1, 1);
                       merge_piece(q, p);
                       finish_head_row(a, head, i, q);
                   }
               });
}

// The walk over the transposed pattern (pair_sums): the dot product of the gathered row of dP with the row's own Theta_j is reduced over the four
// lanes of a group by DPP moves.
template <int PER>
__global__ __launch_bounds__(kBlock) void k_gat_head_cols(GatHeadArgs a) {
    __shared__ __attribute__((aligned(16))) int s_col[kWavesPerBlock][kPairWords<PER>], s_word[kWavesPerBlock][kPairWords<PER>];
    __shared__ __attribute__((aligned(16))) float s_alpha[kWavesPerBlock][kPairWords<PER>];   // negative: the logit is 0 or below
    __shared__ __attribute__((aligned(16))) float s_dot[kWavesPerBlock][kPairWords<PER>];     // rowdot of the entry's destination
    __shared__ __attribute__((aligned(16))) float s_att[kWavesPerBlock][64];
    const int chunk = wave_chunk(), head = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63, sub = lane & 3;
    if (chunk >= a.n.n_chunks) return;
    int *words = s_word[wave], *cols = s_col[wave];
    float *alpha = s_alpha[wave], *rdot = s_dot[wave];
    const float *theta = a.theta + (size_t)head * a.n_src * 32 + sub * 4, *dP = a.dP + (size_t)head * a.n_dst * 32 + sub * 4;
    float *out = a.dtheta + (size_t)head * a.d, *ds_out = a.ds_r + head * a.n_src;
    float *a_l = s_att[wave], *a_r = a_l + 32;   // the head's attention vectors, zeros behind them
    if ((lane & 31) < a.d) a_l[lane] = (lane < 32 ? a.a_l : a.a_r)[head * a.d + (lane & 31)];
    else a_l[lane] = 0.f;
    const float *ds_l = a.ds_l + head * a.n_src;
    auto own_ds = [&](int row) { return row < a.n_dst ? ds_l[row] : 0.f; };   // sources that are no destination have none
    int cont_row = -1;
    constexpr int NA = 9;   // eight columns of dTheta, ds_r
    // the rank-1 terms ds_l a_l + ds_r a_r: every piece of a row adds its share of ds_r, the first one ds_l
    auto close = [&](int row, float dl, const float (&v)[NA]) {
        const bool cont = row == cont_row;
        const float ds = v[8];
        float *dst = cont ? a.carry + ((size_t)head * a.n.n_chunks + chunk) * 32 : out + (size_t)row * a.ldd;
        if (cont) dl = 0.f;
#pragma unroll
        for (int h = 0; h < 2; ++h) {
            const int q = h * 16 + sub * 4;
            const float4 l4 = *reinterpret_cast<const float4 *>(a_l + q), r4 = *reinterpret_cast<const float4 *>(a_r + q);
            const float l[4] = {l4.x, l4.y, l4.z, l4.w}, r[4] = {r4.x, r4.y, r4.z, r4.w};
            float y[4];
#pragma unroll
            for (int i = 0; i < 4; ++i) y[i] = fmaf(dl, l[i], fmaf(ds, r[i], v[h * 4 + i]));
            if (cont || (a.store_vec_ok && q + 4 <= a.d)) {
                *reinterpret_cast<float4 *>(dst + q) = make_float4(y[0], y[1], y[2], y[3]);
            } else {
#pragma unroll
                for (int i = 0; i < 4; ++i) if (q + i < a.d) dst[q + i] = y[i];
            }
        }
        if (sub == 0) {
            if (cont) a.ds_carry[(size_t)head * a.n.n_chunks + chunk] = ds;
            else ds_out[row] = ds;
        }
    };
    int col[PER];
    float4 st[PER];
    if (a.n.nnz > 0) {
        const ChunkSpan<PER> span(a.n, chunk);
#pragma unroll
        for (int u = 0; u < PER; ++u) col[u] = a.n.col_idx[span.at(u, lane)];
#pragma unroll
        for (int u = 0; u < PER; ++u) st[u] = a.row[head * a.n_dst + col[u]];
    }
    const float none_of[NA] = {};
    const FlatChunk<PER> c = flat_rows<PER, 4, 16>(a.n, chunk, lane, words, [&](int r0, bool none) {
        unsigned long long m = __ballot(none);
        for (int b = 0; m; ++b, m >>= 16) {   // rows without entries: one per group at a time
            if (!((m >> (lane >> 2)) & 1ull)) continue;
            const int row = r0 + b * 16 + (lane >> 2);
            close(row, own_ds(row), none_of);
        }
    });
    if (c.lo >= c.hi) return;
    if (c.cont) cont_row = c.i_first;
    {
        int rw[PER];
        float x[PER];
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int at = pair_at<PER>(u * 64 + lane);
            rw[u] = words[at];
            cols[at] = col[u];
        }
        row_values<PER>(c, lane, a.s_r + head * a.n_src, rw, x);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const int at = pair_at<PER>(u * 64 + lane);
            const float t = st[u].x + x[u];
            float w = expf(leaky(t, a.slope) - st[u].y) * st[u].z;
            if (c.lo + u * 64 + lane >= c.hi) w = 0.f;
            alpha[at] = t > 0.f ? w : __uint_as_float(__float_as_uint(w) | 0x80000000u);
            rdot[at] = st[u].w;
        }
        lds_exchange();
        pair_words<PER>(c, lane, words);
    }
    lds_exchange();
    struct W { float w[2], rd[2]; };
    pair_sums<PER, NA>(
        c.hi - c.lo, cols, words, lane, dP,
        [&](int at) {
            const float2 w4 = *reinterpret_cast<const float2 *>(&alpha[at]), d4 = *reinterpret_cast<const float2 *>(&rdot[at]);
            return W{{w4.x, w4.y}, {d4.x, d4.y}};
        },
        [&](int row, Lane8 &own, float &dl) {
            own = load8(theta, row);
            dl = own_ds(row);
        },
        [&](const W &w, int q, const Lane8 &own, const Lane8 &b, float (&acc)[NA]) {
            float x = dot8(own, b);
            x += dpp_f32<0xB1>(x);    // lane ^ 1
            x += dpp_f32<0x4E>(x);    // lane ^ 2
            const float al = fabsf(w.w[q]);
            acc[8] = fmaf(__float_as_uint(w.w[q]) >> 31 ? a.slope * al : al, x - w.rd[q], acc[8]);
            acc[0] = fmaf(al, b.lo.x, acc[0]); acc[1] = fmaf(al, b.lo.y, acc[1]); acc[2] = fmaf(al, b.lo.z, acc[2]); acc[3] = fmaf(al, b.lo.w, acc[3]);
            acc[4] = fmaf(al, b.hi.x, acc[4]); acc[5] = fmaf(al, b.hi.y, acc[5]); acc[6] = fmaf(al, b.hi.z, acc[6]); acc[7] = fmaf(al, b.hi.w, acc[7]);
        },
        close);
}

// the rows of dTheta and ds_r that span several chunks, their pieces added one after the other in chunk order (eight loads under way): a wavefront
// takes 8 chunks' rows, lanes over the columns (lane 32: ds_r)
__global__ __launch_bounds__(kBlock) void k_gat_head_cols_fixup(GatHeadArgs a) {
    const int head = blockIdx.y, lane = threadIdx.x & 63;
    const int c0 = 1 + (blockIdx.x * kWavesPerBlock + (threadIdx.x >> 6)) * 8;
    int c_last = 0, i = -1;
    if (lane < 8 && c0 + lane < a.n.n_chunks) i = continued_row(a.n, c0 + lane, c_last);
    unsigned long long todo = __ballot(i >= 0);
    const float *carry = a.carry + (size_t)head * a.n.n_chunks * 32, *ds_carry = a.ds_carry + (size_t)head * a.n.n_chunks;
    while (todo) {
        const int l = __ffsll((long long)todo) - 1;
        todo &= todo - 1;
        const int row = __builtin_amdgcn_readlane(i, l), first = c0 + l, last = __builtin_amdgcn_readlane(c_last, l);
        float *dst = lane < a.d ? a.dtheta + (size_t)row * a.ldd + (size_t)head * a.d + lane : lane == 32 ? a.ds_r + head * a.n_src + row : nullptr;
        if (!dst) continue;
        float s = 0.f;
#pragma unroll 8
        for (int cc = first; cc <= last; ++cc) s += lane == 32 ? ds_carry[cc] : carry[(size_t)cc * 32 + lane];
        *dst += s;
    }
}

// ---- backward of the GATv2 score e_ij = a . LeakyReLU(U_ij), U_ij = Theta_l[i, :] + Theta_r[j, :]: the sums with a vector per entry, one slice of 32
// columns per wavefront, k_spmm_flat's walk with the row's own vector gathered per entry while rows change.
//   COLS = false, over the pattern (own: Theta_l, gathered: Theta_r, weights de): dTheta_l[i] = a (x) sum_j de_ij LeakyReLU'(U_ij) and the sums
//     R[i] = sum_j de_ij LeakyReLU(U_ij), whose column sums are da;
//   COLS = true, over its transpose (own: Theta_r, gathered: Theta_l and dP, weights (alpha, de) pairs): dTheta_r[j] = sum_i alpha_ij dP_i +
//     a (x) sum_i de_ij LeakyReLU'(U_ij).
// a multiplies the finished pieces.  Bound by the gathers of both vectors; as four walks of one sum each with a pass to multiply by a they took
// 297 us on 3 M entries x 64 columns, as two 179.
struct V2WalkArgs {
    NnzArgs n;
    const float *own, *other, *dP;   // slice-major: over the rows of n, over its columns, over its columns
    const float *w, *att;            // per entry; padded with zeros to whole slices
    float *C, *R;                    // row-major (ldc); slice-major over the rows
    float *carry, *carry_r;          // f_carry floats a chunk
    long long own_tile, other_tile, ldc;
    int f, f_carry, n_tiles, tiles_live, n_groups, store_vec_ok;
    float slope;
};

template <bool COLS, int PER>
__global__ __launch_bounds__(kBlock) void k_v2_walk(V2WalkArgs a) {
    constexpr int LPG = 8, G = 64 / LPG, T = 64 * PER, PART = T / G, PAD = 4, U = 4;
    __shared__ __attribute__((aligned(16))) int s_col[kWavesPerBlock][T + G * PAD];
    __shared__ __attribute__((aligned(16))) int s_row[kWavesPerBlock][T + G * PAD];
    __shared__ __attribute__((aligned(16))) float s_de[kWavesPerBlock][T + G * PAD];
    __shared__ __attribute__((aligned(16))) float s_al[COLS ? kWavesPerBlock : 1][COLS ? T + G * PAD : 4];
    const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63, g = lane / LPG, li = lane % LPG;
    const int per_set = a.n_groups * a.tiles_live, in_set = blockIdx.x % per_set;
    const int tile = blockIdx.x / per_set * a.tiles_live + in_set % a.tiles_live;
    if (tile >= a.n_tiles) return;
    const int chunk = in_set / a.tiles_live * kWavesPerBlock + __builtin_amdgcn_readfirstlane(wave);
    if (chunk >= a.n.n_chunks) return;
    const int f0 = tile * 32 + li * 4;
    int *rows = s_row[wave], *cols = s_col[wave];
    float *de = s_de[wave], *al = s_al[COLS ? wave : 0];
    const float *own = a.own + (size_t)tile * a.own_tile + li * 4, *other = a.other + (size_t)tile * a.other_tile + li * 4;
    const float *dP = COLS ? a.dP + (size_t)tile * a.other_tile + li * 4 : nullptr;
    const float4 at4 = *reinterpret_cast<const float4 *>(a.att + f0);
    int cont_row = -1;
    auto write_row = [&](int row, float4 v, float4 r) {   // v: the sums that a multiplies; r: the others
        v.x *= at4.x; v.y *= at4.y; v.z *= at4.z; v.w *= at4.w;
        if (COLS) { v.x += r.x; v.y += r.y; v.z += r.z; v.w += r.w; }
        if (row == cont_row) {
            *reinterpret_cast<float4 *>(a.carry + (size_t)chunk * a.f_carry + f0) = v;
            if (!COLS) *reinterpret_cast<float4 *>(a.carry_r + (size_t)chunk * a.f_carry + f0) = r;
            return;
        }
        float *dst = a.C + (size_t)row * a.ldc + f0;
        if (a.store_vec_ok && f0 + 4 <= a.f) {
            *reinterpret_cast<float4 *>(dst) = v;
        } else {
            if (f0 < a.f) dst[0] = v.x;
            if (f0 + 1 < a.f) dst[1] = v.y;
            if (f0 + 2 < a.f) dst[2] = v.z;
            if (f0 + 3 < a.f) dst[3] = v.w;
        }
        if (!COLS) *reinterpret_cast<float4 *>(a.R + (size_t)tile * a.own_tile + (size_t)row * 32 + li * 4) = r;
    };
    float we[PER], wa[COLS ? PER : 1];
    int col[PER];
    if (a.n.nnz > 0) {
        const ChunkSpan<PER> span(a.n, chunk);
#pragma unroll
        for (int u = 0; u < PER; ++u) {
            const size_t k = span.at(u, lane);
            col[u] = a.n.col_idx[k];
            if (COLS) {
                const float2 p = reinterpret_cast<const float2 *>(a.w)[k];
                wa[COLS ? u : 0] = p.x;
                we[u] = p.y;
            } else {
                we[u] = a.w[k];
            }
        }
    }
    const float4 zero = make_float4(0.f, 0.f, 0.f, 0.f);
    const FlatChunk<PER> c = flat_rows<PER, PAD, G>(a.n, chunk, lane, rows, [&](int r0, bool none) {
        unsigned long long m = __ballot(none);
        for (int b = 0; m; ++b, m >>= G)   // rows without entries: one per group at a time
            if ((m >> g) & 1ull) write_row(r0 + b * G + g, zero, zero);
    });
    if (c.lo >= c.hi) return;
    const int n = c.hi - c.lo;
    if (c.cont) cont_row = c.i_first;
    {   // the last entry of every row piece is flagged (sign bit of its column)
        unsigned ends = (c.starts >> 1) | ((unsigned)lane_behind((int)(c.starts & 1u), 0) << (PER - 1));
        const int e_last = n - 1 - lane * PER;
        if (e_last >= 0 && e_last < PER) ends |= 1u << e_last;
#pragma unroll
        for (int e = 0; e < PER; ++e) cols[flat_at<PER, PAD, G>(lane * PER + e)] = (int)(((ends >> e) & 1u) << 31);
    }
    lds_exchange();
#pragma unroll
    for (int u = 0; u < PER; ++u) {
        const int at = flat_at<PER, PAD, G>(u * 64 + lane);
        const bool live = c.lo + u * 64 + lane < c.hi;
        cols[at] |= col[u];
        de[at] = live ? we[u] : 0.f;
        if (COLS) al[at] = live ? wa[COLS ? u : 0] : 0.f;
    }
    lds_exchange();
    float4 acc = zero, accr = zero, head = zero, headr = zero, mine = zero;
    int head_at = -1, mine_row = -1;
    const int part0 = g * (PART + PAD);
    for (int s = 0; s < PART && s < n; s += U) {
        const int4 c4 = *reinterpret_cast<const int4 *>(&cols[part0 + s]), r4 = *reinterpret_cast<const int4 *>(&rows[part0 + s]);
        const float4 e4 = *reinterpret_cast<const float4 *>(&de[part0 + s]);
        float4 a4 = zero;
        if (COLS) a4 = *reinterpret_cast<const float4 *>(&al[part0 + s]);
        const int cf[U] = {c4.x, c4.y, c4.z, c4.w}, rf[U] = {r4.x, r4.y, r4.z, r4.w};
        const float e[U] = {e4.x, e4.y, e4.z, e4.w}, w[U] = {a4.x, a4.y, a4.z, a4.w};
        float4 b[U], d[COLS ? U : 1], o[U];
#pragma unroll
        for (int q = 0; q < U; ++q) {
            const size_t j = (size_t)(cf[q] & 0x7fffffff) * 32;
            b[q] = *reinterpret_cast<const float4 *>(other + j);
            if (COLS) d[COLS ? q : 0] = *reinterpret_cast<const float4 *>(dP + j);
        }
        if (__all(rf[U - 1] == mine_row)) {   // (rows ascend) every group stays in its row
#pragma unroll
            for (int q = 0; q < U; ++q) o[q] = mine;
        } else {
#pragma unroll
            for (int q = 0; q < U; ++q) o[q] = *reinterpret_cast<const float4 *>(own + (size_t)rf[q] * 32);
            mine_row = rf[U - 1];
            mine = o[U - 1];
        }
#pragma unroll
        for (int q = 0; q < U; ++q) {
            auto add = [&](float &s1, float &s2, float x, float y, float p) {
                const float t = x + y, dt = t > 0.f ? 1.f : a.slope;
                s1 = fmaf(e[q], dt, s1);   // the product is not rounded: a rounded de * slope costs rows of two to ten entries 9 to 1 % of precision
                s2 = COLS ? fmaf(w[q], p, s2) : fmaf(e[q], dt * t, s2);
            };
            const float4 p = d[COLS ? q : 0];
            add(acc.x, accr.x, o[q].x, b[q].x, p.x);
            add(acc.y, accr.y, o[q].y, b[q].y, p.y);
            add(acc.z, accr.z, o[q].z, b[q].z, p.z);
            add(acc.w, accr.w, o[q].w, b[q].w, p.w);
            if (cf[q] < 0) {
                if (head_at < 0) {
                    head = acc;
                    headr = accr;
                    head_at = part0 + s + q;
                } else {
                    write_row(rf[q], acc, accr);
                }
                acc = accr = zero;
            }
        }
    }
    int f = head_at >= 0;
    auto up = [&](const float4 &v, int off) { return make_float4(__shfl_up(v.x, off, 64), __shfl_up(v.y, off, 64), __shfl_up(v.z, off, 64), __shfl_up(v.w, off, 64)); };
#pragma unroll
    for (int off = LPG; off < 64; off <<= 1) {
        const float4 x = up(acc, off), y = up(accr, off);
        const int of = __shfl_up(f, off, 64);
        if (lane >= off) {
            if (!f) {
                acc.x += x.x; acc.y += x.y; acc.z += x.z; acc.w += x.w;
                accr.x += y.x; accr.y += y.y; accr.z += y.z; accr.w += y.w;
            }
            f |= of;
        }
    }
    acc = up(acc, LPG);
    accr = up(accr, LPG);
    if (head_at >= 0) {
        if (g > 0) {
            head.x += acc.x; head.y += acc.y; head.z += acc.z; head.w += acc.w;
            headr.x += accr.x; headr.y += accr.y; headr.z += accr.z; headr.w += accr.w;
        }
        write_row(rows[head_at], head, headr);
    }
}

// dTheta[j, :] += ds_l[j] a_l + ds_r[j] a_r (ds_l counts only for j < n_l)
__global__ void k_rank1_add(float *__restrict__ D, long long ldd, long long n, int f, const float *__restrict__ ds_l, long long n_l,
                            const float *__restrict__ ds_r, const float *__restrict__ a_l, const float *__restrict__ a_r) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * f) return;
    const long long j = t / f;
    const int q = (int)(t % f);
    const float l = j < n_l ? ds_l[j] : 0.f;
    D[j * ldd + q] += l * a_l[q] + ds_r[j] * a_r[q];
}

// D[i, m] = (accumulate ? D[i, m] : 0) + v[m] G[i, m]: a column scaling, on its own or added to what D holds (G may be D itself)
__global__ void k_scale_cols(float *D, long long ldd, const float *G, long long ldg, const float *__restrict__ v, long long n, int f,
                             int accumulate) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= n * f) return;
    const long long i = t / f;
    const int m = (int)(t % f);
    const float g = v[m] * G[i * ldg + m];
    D[i * ldd + m] = accumulate ? D[i * ldd + m] + g : g;
}

__global__ void k_set_f32(float *p, long long n, float v) {
    const long long t = (long long)blockIdx.x * blockDim.x + threadIdx.x;
    if (t < n) p[t] = v;
}

// part[slab][0][q] = sum_j Theta[j, q] v_l[j], part[slab][1][q] = sum_j Theta[j, q] v_r[j] over the rows of the slab,
// Theta slice-major, sums in fp64.  One workgroup per (tile, slab): eight lanes read a row's 32 columns as 16-byte words, 32 rows per
// pass, four passes in flight.  Bound by the read of Theta once there are enough workgroups: with one row in flight per thread and 25
// slabs a 100,000 x 32 slice took 234 us at 55 GB/s; now 7 us (both kernels: 11).
__global__ __launch_bounds__(256) void k_theta_t_vec(const float *__restrict__ theta, long long n, int f_pad, const float *__restrict__ v_l,
                                                     long long n_l, const float *__restrict__ v_r, int rows_per_slab,
                                                     double *__restrict__ part, long long head_stride) {
    __shared__ double red[2][4][32];   // per wavefront
    const int tile = blockIdx.x, slab = blockIdx.y;
    if (v_l) v_l += tile * head_stride;   // heads of one slice: a pair of vectors per tile
    if (v_r) v_r += tile * head_stride;
    const int q = threadIdx.x & 7, rr = threadIdx.x >> 3;
    const long long j_lo = (long long)slab * rows_per_slab;
    const long long j_hi = (j_lo + rows_per_slab < n) ? j_lo + rows_per_slab : n;
    const float *th = theta + (size_t)tile * (size_t)n * 32 + q * 4;
    double sl[4] = {0.0, 0.0, 0.0, 0.0}, sr[4] = {0.0, 0.0, 0.0, 0.0};
#pragma unroll 4
    for (long long j = j_lo + rr; j < j_hi; j += 32) {
        const float4 x = *reinterpret_cast<const float4 *>(th + j * 32);
        const double l = j >= n_l ? 0.0 : v_l ? (double)v_l[j] : 1.0, r = v_r ? (double)v_r[j] : 0.0;   // null: column sums; nothing
        sl[0] += (double)x.x * l; sl[1] += (double)x.y * l; sl[2] += (double)x.z * l; sl[3] += (double)x.w * l;
        sr[0] += (double)x.x * r; sr[1] += (double)x.y * r; sr[2] += (double)x.z * r; sr[3] += (double)x.w * r;
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
#pragma unroll
        for (int off = 8; off < 64; off <<= 1) {
            sl[e] += __shfl_xor(sl[e], off, 64);
            sr[e] += __shfl_xor(sr[e], off, 64);
        }
        if ((threadIdx.x & 63) < 8) {
            red[0][threadIdx.x >> 6][q * 4 + e] = sl[e];
            red[1][threadIdx.x >> 6][q * 4 + e] = sr[e];
        }
    }
    __syncthreads();
    if (threadIdx.x < 64) {
        const int w = threadIdx.x >> 5, c = threadIdx.x & 31;
        part[((size_t)slab * 2 + w) * f_pad + tile * 32 + c] = ((red[w][0][c] + red[w][1][c]) + red[w][2][c]) + red[w][3][c];
    }
}

// adds the slabs: 16 columns a workgroup, the slabs dealt to 16 lanes each whose partial sums are added in lane order
__global__ __launch_bounds__(256) void k_sum_slabs(const double *__restrict__ part, int slabs, int f_pad, int f, float *__restrict__ out_l,
                                                   float *__restrict__ out_r, int d) {
    __shared__ double red[2][16][16];
    const int c = threadIdx.x & 15, y = threadIdx.x >> 4;
    const int q = blockIdx.x * 16 + c;
    const int out = d < f ? q / 32 * d + q % 32 : q;            // heads of d columns in slices of 32
    const bool on = q < f && (d >= f || q % 32 < d);
    double l = 0.0, r = 0.0;
    if (q < f) {
#pragma unroll 8
        for (int s = y; s < slabs; s += 16) {
            l += part[((size_t)s * 2 + 0) * f_pad + q];
            r += part[((size_t)s * 2 + 1) * f_pad + q];
        }
    }
    red[0][y][c] = l;
    red[1][y][c] = r;
    __syncthreads();
    if (y > 1 || !on) return;
    double t = 0.0;
#pragma unroll
    for (int u = 0; u < 16; ++u) t += red[y][u][c];
    float *dst = y == 0 ? out_l : out_r;
    if (dst) dst[out] = (float)t;
}

// pos[k] = index in the transposed pattern of the entry (i, j) stored at k: the place of i among the ascending
// columns of row j of At.  miss counts entries that are not there (At is not the transpose of A).
__global__ __launch_bounds__(kBlock) void k_transpose_pos(NnzArgs a, const int32_t *__restrict__ t_row_ptr, const int32_t *__restrict__ t_col_idx,
                                                           int32_t *__restrict__ pos, int32_t *__restrict__ miss) {
    const int chunk = wave_chunk();
    if (chunk >= a.n_chunks) return;
    walk_chunk(a, chunk, threadIdx.x & 63, [&](int i) { return i; },
               [&](int k, int i) {
                   const int j = a.col_idx[k];
                   int lo = t_row_ptr[j], hi = t_row_ptr[j + 1];
                   const int end = hi;
                   while (lo < hi) {
                       const int mid = (int)(((long long)lo + hi) >> 1);
                       if (t_col_idx[mid] < i) lo = mid + 1; else hi = mid;
                   }
                   const bool found = lo < end && t_col_idx[lo] == i;
                   pos[k] = found ? lo : 0;
                   if (!found) atomicAdd(miss, 1);
               });
}

// graph feature extractor: out[0] = largest row length, out[1] = sum of squared row lengths (as two 32-bit halves are
// not needed: 64-bit integer atomics), both exact
__global__ void k_row_moments(const int32_t *__restrict__ row_ptr, int n_rows, unsigned long long *__restrict__ out) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    unsigned long long d = 0;
    if (i < n_rows) d = (unsigned long long)(row_ptr[i + 1] - row_ptr[i]);
    unsigned long long mx = d, sq = d * d;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
        const unsigned long long m2 = __shfl_xor(mx, off, 64), s2 = __shfl_xor(sq, off, 64);
        mx = mx > m2 ? mx : m2;
        sq += s2;
    }
    if ((threadIdx.x & 63) == 0) {
        atomicMax(&out[0], mx);
        atomicAdd(&out[1], sq);
    }
}

__global__ void k_fill_u64(unsigned long long *p, int n, unsigned long long v) {
    const int i = blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = v;
}

// calls f with the chunk length of a plan (64 PER entries) as a compile-time constant
template <class F>
hipError_t with_per(int chunk_nnz, F f) {
    switch (chunk_nnz) {
        case 64: f(std::integral_constant<int, 1>()); break;
        case 128: f(std::integral_constant<int, 2>()); break;
        case 256: f(std::integral_constant<int, 4>()); break;
        case 512: f(std::integral_constant<int, 8>()); break;
        default: return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

NnzArgs nnz_args(const sensei_csr &A, const ChunkPlan &p) {
    NnzArgs n;
    n.row_ptr = A.row_ptr; n.col_idx = A.col_idx; n.chunk_row = p.chunk_row;
    n.n_rows = A.n_rows; n.nnz = (int)A.nnz; n.chunk_nnz = p.chunk_nnz; n.n_chunks = p.n_chunks;
    return n;
}

}  // namespace

// ----------------------------------------------------------------- host side

// Non-zeros per chunk (= per wavefront): 64 times the entries a lane of the flat walks owns, at most eight (more would not fit its registers
// and LDS).  Large graphs: 512.  With 512 / 256 / 128 on 115 M non-zeros, ms: GCN layer 602 -> 256 on the tile split 3.40 / 3.47 / 3.86, unsplit
// 6.32 / 6.56 / 7.59, 256 -> 41 0.90 / 0.92 / 1.07, GAT backward 13.5 / 13.9 / 14.9; 62 M non-zeros, GAT layer 4.65 / 4.72 / 4.95; on 2 to 4 M
// non-zeros the three are within 3 %.
int choose_chunk_nnz(int64_t nnz) {
    if (nnz >= (1LL << 19)) return 512;
    if (nnz >= (1LL << 18)) return 256;
    if (nnz >= (1LL << 17)) return 128;
    return 64;  // small graphs are latency bound: more, shorter wavefronts
}

// The two walks of the narrow heads' backward hold more per entry: chunks of 512 leave them three wavefronts a SIMD.  Training passes with chunks of 64 / 128 /
// 256 / 512 there, us: 4 heads, 2.1 M entries 670 / 612 / 589 / 604, 2.4 M on a grid, 2 heads 1,437 / 1,413 / 1,433 / 1,463, 8 heads, 20 M 10,935 / 9,710 / 8,993 /
// 8,986, 2 heads, 99 M 26,575 / 26,213 / 26,081 / 25,959, one head, 292,000 103 / 106 / 106 / 117, 2 heads, 170,000 146 / 139 / 144 / 157.
int choose_head_chunk_nnz(int64_t nnz) { return choose_chunk_nnz(nnz) < 256 ? choose_chunk_nnz(nnz) : 256; }

static int n_chunks_for(int64_t nnz, int t) { return nnz <= 0 ? 1 : (int)((nnz + t - 1) / t); }

size_t plan_bytes(int64_t nnz) {
    return align_up(((size_t)n_chunks_for(nnz, choose_chunk_nnz(nnz)) + 1) * sizeof(int32_t), 256);
}

hipError_t launch_side(SideWork *side, hipStream_t s) {
    if (!side || side->blocks <= 0) return hipSuccess;
    const SideWork w = side->take();
    hipLaunchKernelGGL(k_side, dim3((unsigned)w.blocks), dim3(kSideThreads), 0, s, w);
    return hipGetLastError();
}

hipError_t launch_chunk_rows(const sensei_csr &A, const ChunkPlan &p, hipStream_t s) {
    SideWork w;
    w.add_plan(A, p);
    return launch_side(&w, s);
}

SpmmShape spmm_shape(const float *B, int64_t ldb, int f) {
    SpmmShape sh;
    const uintptr_t addr = reinterpret_cast<uintptr_t>(B);
    if (f % 4 == 0 && ldb % 4 == 0 && addr % 16 == 0) sh.vec = 4;
    else if (f % 2 == 0 && ldb % 2 == 0 && addr % 8 == 0) sh.vec = 2;
    else sh.vec = 1;
    const int fv = (f + sh.vec - 1) / sh.vec;  // vector columns
    // A neighbour group reads one 128-byte line per neighbour (32 floats) and the feature tiles are spread over the XCDs.  Rows that do not
    // fill whole groups use one wider group instead when that covers the row in a single tile (measured faster than leaving a nearly empty
    // last tile).  Very wide rows use wider groups so that the number of tiles stays moderate: every tile of a chunk finds the rows and reads
    // the columns again (50,000 rows of 12 entries, 4,096 columns: 1,635 us in 128 tiles of 8 lanes, 1,378 in 32 of 32), and the grid, tiles
    // times chunks, has to stay below 2^32 threads.  Rows of a few 8- or 4-byte words take the narrowest group that covers them: more
    // neighbours per step (1 M nodes of a grid, one column: 156 us with 32 lanes a neighbour, 57 with 8).
    int lpg = 32 / sh.vec;
    while (lpg > 8 && lpg / 2 >= fv) lpg >>= 1;
    if (fv > lpg && fv <= 32 && fv % lpg != 0) while (lpg < fv) lpg <<= 1;
    while (lpg < 64 && (fv + lpg - 1) / lpg > 32) lpg <<= 1;
    sh.lpg = lpg;
    sh.n_tiles = (fv + lpg - 1) / lpg;
    sh.f_carry = sh.n_tiles * lpg * sh.vec;
    return sh;
}

// Value-less SpMM on rows of two and a half to five entries on average: a row to every lane group of k_spmm, so that the groups of a wavefront
// read and write neighbouring rows, where the flat walk has them an eighth of a chunk apart and its 26 KB of LDS a workgroup cost a quarter
// of the wavefronts.  Times flat / by rows, us: 4 M nodes of a grid, 4 columns 245 / 192, 20 columns 448 / 315, 64 columns 807 / 702, 128
// columns 1,737 / 1,405; 2 M rows of three random entries, 4 / 20 / 128 columns 146 / 132, 233 / 218, 870 / 809.  Where a tile is all of the row
// and fills its line, only if the operand exceeds the 256 MB of the last-level cache (32 columns, 4 M nodes 407 / 362; a GCN layer on 1 M nodes
// 249 / 259).  Not where most rows are empty or nearly so (300,000 rows of 2, 4 columns 52 / 59; training on sampled blocks, 103,000 rows of
// 0.6, 151 / 156), not from five entries on (300,000 rows of 5, 8 columns 44 / 47; of 16, 58 / 116), nor with weights, where the rows of hubs
// cost the most (power-law pattern of 300,000 rows, 64 columns: 238 / 370, value-less 296 / 355).
static bool spmm_by_rows(const sensei_csr &A, int mode, int f, bool b_sliced, int n_tiles) {
    if (mode != SENSEI_SPMM_PATTERN || A.nnz >= 5 * (int64_t)A.n_rows || 2 * A.nnz < 5 * (int64_t)A.n_rows) return false;
    return n_tiles > 1 || !(b_sliced || f == 32) || (int64_t)A.n_cols * 128 > (256LL << 20);
}

size_t spmm_carry_bytes(int64_t nnz, int f) {
    const int t = choose_chunk_nnz(nnz);
    // tiles are at most 256 floats wide, so the padded width stays below f + 256
    const size_t f_carry = align_up((size_t)(f > 0 ? f : 1), 32) + 256;
    return align_up((size_t)n_chunks_for(nnz, t) * f_carry * sizeof(float), 256);
}

hipError_t launch_spmm(const sensei_csr &A, int mode, const float *r, const float *c, const float *B, int64_t ldb,
                       int f, float *C, int64_t ldc, int f_store, int act, const ChunkPlan &p, float *carry,
                       hipStream_t s, KernelTimer *timer, bool accumulate, bool finalize, const float2 *mz, bool b_sliced, int val_stride,
                       bool c_sliced, bool defer_fixup, const AttnFusedArgs *fused) {
    SpmmShape sh = spmm_shape(B, ldb, f);
    if (b_sliced) {  // slices of 32 floats per row: one 128-byte line per neighbour and tile
        sh.vec = 4; sh.lpg = 8; sh.n_tiles = (f + 31) / 32; sh.f_carry = sh.n_tiles * 32;
        ldb = 32;
    }
    SpmmArgs a;
    a.tile_stride_b = b_sliced ? (long long)(A.n_cols > 0 ? A.n_cols : 1) * 128 : (long long)sh.vec * sh.lpg * 4;
    a.mz = (mode == kSpmmSoftmax) ? mz : nullptr;
    a.val_stride = val_stride;
    if (c_sliced) ldc = 32;  // requires b_sliced (tiles of 32 columns) and f_store == pad32(f): checked by the callers
    a.c_tf = sh.vec * sh.lpg;
    a.c_shift = __builtin_ctz((unsigned)a.c_tf);
    a.c_tile = c_sliced ? (long long)(A.n_rows > 0 ? A.n_rows : 1) * 32 : (long long)a.c_tf;
    a.row_ptr = A.row_ptr; a.col_idx = A.col_idx; a.chunk_row = p.chunk_row;
    a.val = A.val; a.r = r; a.c = c; a.B = B; a.C = C; a.carry = carry;
    a.ldb = ldb; a.ldc = ldc;
    a.n_rows = A.n_rows; a.nnz = (int)A.nnz; a.chunk_nnz = p.chunk_nnz; a.n_chunks = p.n_chunks;
    a.f = f; a.f_store = f_store; a.f_carry = sh.f_carry; a.n_tiles = sh.n_tiles; a.act = act;
    a.store_vec_ok = (ldc % sh.vec == 0) && (reinterpret_cast<uintptr_t>(C) % (4 * sh.vec) == 0);
    a.accumulate = accumulate ? 1 : 0; a.finalize = finalize ? 1 : 0;
    a.scale_weights = defer_fixup ? 0 : 1;   // deferred fix-up: the caller wants raw sums
    a.s_l = nullptr; a.s_r = nullptr; a.slope = 0.f; a.mz_out = nullptr; a.carry_mz = nullptr; a.head_vec = 0; a.head_mz = 0; a.head_cols = 0;
    if (mode == kSpmmAttnFused) {
        if (!fused || accumulate || !finalize || defer_fixup) return hipErrorInvalidValue;
        a.s_l = fused->s_l; a.s_r = fused->s_r; a.slope = fused->slope; a.mz_out = fused->row_mz; a.carry_mz = fused->chunk_mz;
        if (fused->heads > 1) {
            if (!b_sliced || c_sliced || f != fused->heads * 32 || fused->cols > 32 || f_store != fused->heads * fused->cols) return hipErrorInvalidValue;
            a.head_vec = A.n_cols; a.head_mz = A.n_rows + 1; a.head_cols = fused->cols;
            a.c_tile = fused->cols;
            if (fused->cols % 4 != 0) a.store_vec_ok = 0;   // a head's columns begin anywhere
        }
    }
    const unsigned groups = blocks_for(p.n_chunks, kWavesPerBlock);
    // Feature tiles worked on at the same time (consecutive XCDs take consecutive tiles of the live set): all eight
    // while a 128-byte slice of the gathered matrix is small, four beyond that (233 k-node R-MAT graph at F = 256, ms with 1 / 2 / 4 / 8 live
    // tiles: 6.13 / 5.91 / 5.85 / 6.04; GAT layer that aggregates 602 columns of it over a panel-major remainder, 2 / 4 / 8: 10.8 / 10.5 / 11.6;
    // 2.45 M nodes at F = 512: 27.9 / 27.9 / 27.4 / 27.6; 98 k nodes of 1,021 random entries at F = 512: 19.5 / 19.0 / 19.0 / 18.9).
    const double slice_bytes = (double)(A.n_cols > 0 ? A.n_cols : 1) * sh.lpg * sh.vec * 4.0;
    a.tiles_live = slice_bytes > 8e6 ? 4 : 8;
    if (a.tiles_live > sh.n_tiles) a.tiles_live = sh.n_tiles;
    a.n_groups = (int)groups;
    const unsigned n_sets = (unsigned)((sh.n_tiles + a.tiles_live - 1) / a.tiles_live);
    dim3 grid(groups * (unsigned)a.tiles_live * n_sets);
    // byte offsets of the gathered matrix fit 32 bits?
    const bool off32 = (unsigned long long)(A.n_cols > 0 ? A.n_cols : 1) * (unsigned long long)ldb * 4ull + 4ull * (unsigned long long)f <= 0xffffffffull &&
                       A.n_cols < (1 << 24) && ldb * 4 < (1 << 24);
    hipError_t err;
    const bool by_rows = sh.vec == 4 && spmm_by_rows(A, mode, f, b_sliced, sh.n_tiles), flat = sh.vec == 4 && !by_rows;
    a.find_rows = p.pending && flat && A.nnz > 0 ? p.chunk_row : nullptr;
    if (p.pending && !a.find_rows && (err = launch_chunk_rows(A, p, s)) != hipSuccess) return err;
    hipEvent_t t0 = timer ? timer->next() : nullptr, t1 = t0 ? timer->next() : nullptr;
    if (t1 && hipEventRecord(t0, s) != hipSuccess) return hipErrorUnknown;
    if (by_rows) err = off32 ? spmm_rows_pattern<true>(a, sh.lpg, grid, s) : spmm_rows_pattern<false>(a, sh.lpg, grid, s);
    // plain: whole 16-byte pieces of a row, written and not added to.  Without the code for the others in its loop the kernel is 1 to 3 % faster.
    else if (flat) err = a.store_vec_ok && f_store % 4 == 0 && !accumulate ? spmm_flat_dispatch<true>(a, mode, sh.lpg, off32, grid, s)
                                                                           : spmm_flat_dispatch<false>(a, mode, sh.lpg, off32, grid, s);
    else switch (sh.vec) {
        case 2: err = spmm_dispatch_lpg<2>(a, mode, sh.lpg, off32, grid, s); break;
        default: err = spmm_dispatch_lpg<1>(a, mode, sh.lpg, off32, grid, s); break;
    }
    if (err != hipSuccess) return err;
    if (t1 && hipEventRecord(t1, s) != hipSuccess) return hipErrorUnknown;
    if (p.n_chunks > 1 && !(defer_fixup && b_sliced && !finalize)) {
        const unsigned fg = blocks_for(p.n_chunks - 1, kWavesPerBlock * kFixupChunks);
        if (mode == kSpmmAttnFused) hipLaunchKernelGGL(k_spmm_fixup_attn, dim3(fg, a.head_vec ? sh.n_tiles : 1), dim3(kBlock), 0, s, a);
        else {
            a.fix_quads = p.n_chunks < 8192 ? 8 : 32;
            if (flat && a.scale_weights && mode != SENSEI_SPMM_PATTERN) { a.r = nullptr; a.mz = nullptr; }   // the pieces are scaled already
            hipLaunchKernelGGL(k_spmm_fixup, dim3(fg, blocks_for(f_store, 4 * a.fix_quads)), dim3(kBlock), 0, s, a);
        }
        err = hipGetLastError();
    }
    return err;
}

hipError_t launch_degrees(const sensei_csr &A, int32_t *deg_row, int32_t *deg_col, hipStream_t s) {
    if (A.n_rows > 0) hipLaunchKernelGGL(k_deg_row, dim3(blocks_for(A.n_rows, kBlock)), dim3(kBlock), 0, s, A.row_ptr, A.n_rows, deg_row);
    if (A.n_cols > 0) hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(A.n_cols, kBlock)), dim3(kBlock), 0, s, deg_col, (long long)A.n_cols, 0);
    const int n_ranges = (int)((A.n_cols + kDegRange - 1) / kDegRange);
    if (A.nnz >= (1 << 18) && n_ranges <= kDegRangesMax) {
        int shares = 256 / n_ranges / 8 * 8;  // about one workgroup per compute unit, a multiple of eight shares
        if (shares < 8) shares = 8;
        const long long per_share = (A.nnz + shares - 1) / shares;
        hipLaunchKernelGGL(k_deg_col_ranges, dim3(shares * n_ranges), dim3(kDegThreads), 0, s, A.col_idx, (long long)A.nnz, (int)A.n_cols, n_ranges,
                           per_share, deg_col);
    } else if (A.nnz > 0) {
        hipLaunchKernelGGL(k_deg_col, dim3(blocks_for(A.nnz, kBlock)), dim3(kBlock), 0, s, A.col_idx, (long long)A.nnz, deg_col);
    }
    return hipGetLastError();
}

hipError_t launch_norm_vectors(const int32_t *deg, int64_t n, float *out, hipStream_t s) {
    if (n > 0) hipLaunchKernelGGL(k_norm_vec, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, s, deg, (long long)n, out);
    return hipGetLastError();
}

hipError_t launch_sddmm_norm(const sensei_csr &A, const float *r, const float *c, float *val, const ChunkPlan &p, hipStream_t s) {
    if (A.nnz <= 0) return hipSuccess;
    return with_per(p.chunk_nnz, [&](auto per) {
        hipLaunchKernelGGL(k_sddmm_norm<per()>, dim3(blocks_for(p.n_chunks, kWavesPerBlock)), dim3(kBlock), 0, s, nnz_args(A, p), r, c, val);
    });
}

hipError_t launch_score(const sensei_csr &A, const float *s_l, const float *s_r, float slope, float *e, const ChunkPlan &p, hipStream_t s) {
    if (A.nnz <= 0) return hipSuccess;
    return with_per(p.chunk_nnz, [&](auto per) {
        hipLaunchKernelGGL(k_score<per()>, dim3(blocks_for(p.n_chunks, kWavesPerBlock)), dim3(kBlock), 0, s, nnz_args(A, p), s_l, s_r, slope, e);
    });
}

hipError_t launch_row_broadcast(const float *s_vec, const float *X, int64_t ldx, int64_t n, int f, float *Y, int64_t ldy, int act, hipStream_t s,
                                const float *mask, int64_t ldm, SideWork *side) {
    if (n <= 0 || f <= 0) return launch_side(side, s);
    const SideWork sw = take_side(side);
    const bool a16 = reinterpret_cast<uintptr_t>(X) % 16 == 0 && reinterpret_cast<uintptr_t>(Y) % 16 == 0;
    if (f % 4 == 0 && ldx % 4 == 0 && ldy % 4 == 0 && a16)
        hipLaunchKernelGGL((k_row_broadcast<4>), dim3(blocks_for(n * (f / 4), kBlock) + sw.blocks), dim3(kBlock), 0, s, s_vec, X, (long long)ldx, (long long)n, f, Y, (long long)ldy, act, mask, (long long)ldm, sw);
    else
        hipLaunchKernelGGL((k_row_broadcast<1>), dim3(blocks_for(n * f, kBlock) + sw.blocks), dim3(kBlock), 0, s, s_vec, X, (long long)ldx, (long long)n, f, Y, (long long)ldy, act, mask, (long long)ldm, sw);
    return hipGetLastError();
}

hipError_t launch_reciprocal(const float *v, int64_t n, float *out, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_reciprocal, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, s, v, (long long)n, out);
    return hipGetLastError();
}

hipError_t launch_stack_weights(const float *W, int64_t ldw, int hops, int f_in, int f_out, float *out, int64_t ldo, hipStream_t s) {
    const long long total = (long long)hops * pad32(f_in) * f_out;
    if (total <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_stack_weights, dim3(blocks_for(total, kBlock)), dim3(kBlock), 0, s, W, (long long)ldw, hops, f_in, pad32(f_in), f_out, out, (long long)ldo);
    return hipGetLastError();
}

hipError_t launch_to_slices(const float *s_vec, const float *X, int64_t ldx, int64_t n, int f, float *Y, hipStream_t s, const float *mask,
                            int64_t ldm, SideWork *side, int n_heads) {
    if (n <= 0 || f <= 0) return launch_side(side, s);
    const SideWork sw = take_side(side);
    const int d = f / n_heads;
    const int x_vec_ok = (ldx % 4 == 0 && (n_heads == 1 || d % 4 == 0) && reinterpret_cast<uintptr_t>(X) % 16 == 0) ? 1 : 0;
    const long long threads = n * (long long)(n_heads > 1 ? n_heads * 8 : pad32(f) / 4);
    hipLaunchKernelGGL(k_to_slices, dim3(blocks_for(threads, kBlock) + sw.blocks), dim3(kBlock), 0, s, s_vec, X, (long long)ldx, (long long)n, f, d, Y, x_vec_ok, mask, (long long)ldm, sw);
    return hipGetLastError();
}

size_t softmax_ws_bytes(const sensei_csr &A) {
    const int t = choose_chunk_nnz(A.nnz);
    return align_up((size_t)(A.n_rows + 1) * sizeof(float2), 256) + align_up((size_t)n_chunks_for(A.nnz, t) * sizeof(float2), 256);
}

hipError_t launch_softmax(const sensei_csr &A, const float *e, float *alpha, const ChunkPlan &p, float2 *stats, float2 *carry_stats,
                          hipStream_t s) {
    SoftmaxArgs a;
    a.n = nnz_args(A, p);
    a.e = e; a.s_l = nullptr; a.s_r = nullptr; a.slope = 0.f; a.stats = stats; a.carry = carry_stats; a.alpha = alpha;
    a.logits = nullptr; a.dst_index = nullptr;
    dim3 g1(blocks_for(p.n_chunks, kWavesPerBlock));
    return with_per(p.chunk_nnz, [&](auto per) {
        hipLaunchKernelGGL((k_softmax_stats<true, per()>), g1, dim3(kBlock), 0, s, a);
        if (p.n_chunks > 1) hipLaunchKernelGGL(k_softmax_fixup, dim3(blocks_for(p.n_chunks - 1, kBlock)), dim3(kBlock), 0, s, a);
        if (A.nnz > 0 && alpha) hipLaunchKernelGGL(k_softmax_alpha<per()>, g1, dim3(kBlock), 0, s, a);
    });
}

hipError_t launch_attention_stats(const sensei_csr &A, const float *s_l, const float *s_r, float slope, float *logits,
                                  const int32_t *dst_index, const ChunkPlan &p, float2 *stats, float2 *carry_stats, hipStream_t s) {
    SoftmaxArgs a;
    a.n = nnz_args(A, p);
    a.e = nullptr; a.s_l = s_l; a.s_r = s_r; a.slope = slope; a.stats = stats; a.carry = carry_stats; a.alpha = nullptr;
    a.logits = logits; a.dst_index = dst_index;
    return with_per(p.chunk_nnz, [&](auto per) {
        hipLaunchKernelGGL((k_softmax_stats<false, per()>), dim3(blocks_for(p.n_chunks, kWavesPerBlock)), dim3(kBlock), 0, s, a);
        if (p.n_chunks > 1) hipLaunchKernelGGL(k_softmax_fixup, dim3(blocks_for(p.n_chunks - 1, kBlock)), dim3(kBlock), 0, s, a);
    });
}


bool panel_stats_usable(int width, int chunk_nnz) { return width <= kPanelStatsCols && chunk_nnz == 512; }

hipError_t launch_panel_stats(const PanelWalk *panels, int n_panels, int width, int n_rows, int n_cols, const float *s_l, const float *s_r, float slope,
                              float2 *seg_stats, float2 *seg_carry, float2 *stats, hipStream_t s) {
    PanelStatsArgs a;
    a.n_panels = n_panels; a.width = width; a.n_cols = n_cols;
    a.per_panel = 256 / n_panels;   // one workgroup a compute unit
    int chunk_nnz = 0;
    for (int q = 0; q < n_panels; ++q) {
        SoftmaxArgs &p = a.s[q];
        p.n = nnz_args(panels[q].A, panels[q].plan);
        p.e = nullptr; p.s_l = s_l; p.s_r = s_r; p.slope = slope; p.alpha = nullptr; p.dst_index = nullptr;
        p.logits = const_cast<float *>(panels[q].A.val);
        p.stats = seg_stats + (size_t)q * n_rows;
        p.carry = seg_carry;
        seg_carry += panels[q].plan.n_chunks;
        chunk_nnz = panels[q].plan.chunk_nnz;
    }
    if (chunk_nnz != 512 || width > kPanelStatsCols) return hipErrorInvalidValue;
    const size_t lds = (size_t)kPanelStatsWaves * 1024 * sizeof(float) + (size_t)width * sizeof(float);
    hipLaunchKernelGGL(k_panel_stats<8>, dim3((unsigned)(a.per_panel * n_panels)), dim3(64 * kPanelStatsWaves), lds, s, a);
    if (n_rows > 0) hipLaunchKernelGGL(k_panel_stats_join, dim3(blocks_for(n_rows, kBlock)), dim3(kBlock), 0, s, a, stats, n_rows);
    return hipGetLastError();
}

// ------------------------------------------------------------ backward of the attention layer (host side)

hipError_t launch_row_sum(const sensei_csr &A, const float *val, int stride, float *out, const ChunkPlan &p, float *carry, hipStream_t s,
                          const int32_t *dst_rem, const int32_t *place, float *first_rem) {
    const NnzArgs n = nnz_args(A, p);
    const RemWeights rem = {dst_rem, place, first_rem};
    return with_per(p.chunk_nnz, [&](auto per) {
        const dim3 grid(blocks_for(p.n_chunks, kWavesPerBlock));
        if (dst_rem) hipLaunchKernelGGL((k_row_sum<per(), true>), grid, dim3(kBlock), 0, s, n, val, 2, out, carry, rem);
        else hipLaunchKernelGGL((k_row_sum<per(), false>), grid, dim3(kBlock), 0, s, n, val, stride, out, carry, rem);
        if (p.n_chunks > 1) hipLaunchKernelGGL(k_sum_fixup, dim3(blocks_for(p.n_chunks - 1, kBlock)), dim3(kBlock), 0, s, n, out, carry);
    });
}

// 32-column slices of the gathered matrix that one launch of the per-entry sums takes: all of a small matrix, which saves finding the rows again and the sums
// written and read in between (3 M entries on 50,000 columns, 64 wide, 54 us in one launch of two slices, 61 in two), one of a larger one, so that what the L2s hold
// is one slice (a gathered line, in launches of one slice / of four: 50,000 columns 7.3 / 6.9 ps, 100,000 8.4 / 10.1, 233,000 7.6 / 13.3).
static int slices_a_walk(int64_t n_cols, int n_tiles) {
    const int64_t most = (32LL << 20) / (128 * (n_cols > 0 ? n_cols : 1));
    return most >= n_tiles ? n_tiles : 1;
}

hipError_t launch_gat_dalpha(const sensei_csr &A, const float *theta, const float *dP, int f, const float *logits, const float2 *mz,
                             float *dalpha, float *rowdot, const ChunkPlan &p, float *carry, hipStream_t s, float scale, int dp_rows) {
    GatBwdArgs a;
    a.scale = scale;
    a.n = nnz_args(A, p);
    a.theta = theta; a.dP = dP; a.logits = logits; a.mz = mz; a.dalpha = dalpha; a.rowdot = rowdot; a.carry = carry;
    a.theta_tile = (long long)(A.n_cols > 0 ? A.n_cols : 1) * 32;
    a.dp_tile = (long long)(dp_rows > 0 ? dp_rows : A.n_rows > 0 ? A.n_rows : 1) * 32;
    a.n_tiles = (f + 31) / 32;
    a.dp_rows = dp_rows > 0 ? dp_rows : A.n_rows > 0 ? A.n_rows : 1;
    const dim3 grid(blocks_for(p.n_chunks, kWavesPerBlock));
    if (A.nnz <= 0 && !rowdot) return hipSuccess;
    return with_per(p.chunk_nnz, [&](auto per) {
        const int step = slices_a_walk(A.n_cols, a.n_tiles);
        for (int t = 0; t < a.n_tiles; t += step) {
            const int t1 = t + step < a.n_tiles ? t + step : a.n_tiles;
            if (t1 == a.n_tiles && rowdot) hipLaunchKernelGGL((k_gat_dalpha<true, per()>), grid, dim3(kBlock), 0, s, a, t, t1);
            else hipLaunchKernelGGL((k_gat_dalpha<false, per()>), grid, dim3(kBlock), 0, s, a, t, t1);
        }
        if (rowdot && p.n_chunks > 1)
            hipLaunchKernelGGL(k_sum_fixup, dim3(blocks_for(p.n_chunks - 1, kBlock)), dim3(kBlock), 0, s, a.n, rowdot, carry);
    });
}

hipError_t launch_gat_dalpha_merge(const sensei_csr &A, const int32_t *where, const float *dalpha_rem, const float *Dt, const float *logits,
                                   const float2 *mz, float *dalpha, float *rowdot, const ChunkPlan &p, float *carry, hipStream_t s, const int32_t *place) {
    const NnzArgs n = nnz_args(A, p);
    return with_per(p.chunk_nnz, [&](auto per) {
        hipLaunchKernelGGL(k_gat_dalpha_merge<per()>, dim3(blocks_for(p.n_chunks, kWavesPerBlock)), dim3(kBlock), 0, s, n, where, place, dalpha_rem, Dt, logits,
                           mz, dalpha, rowdot, carry);
        if (p.n_chunks > 1) hipLaunchKernelGGL(k_sum_fixup, dim3(blocks_for(p.n_chunks - 1, kBlock)), dim3(kBlock), 0, s, n, rowdot, carry);
    });
}

hipError_t launch_score_v2(const sensei_csr &A, const float *theta_l, const float *theta_r, int f, const float *att_padded, float slope,
                           float *logits, const ChunkPlan &p, hipStream_t s) {
    if (A.nnz <= 0) return hipSuccess;
    ScoreV2Args a;
    a.n = nnz_args(A, p);
    a.theta_l = theta_l; a.theta_r = theta_r; a.att = att_padded; a.logits = logits; a.slope = slope;
    a.tl_tile = (long long)(A.n_rows > 0 ? A.n_rows : 1) * 32;
    a.tr_tile = (long long)(A.n_cols > 0 ? A.n_cols : 1) * 32;
    const dim3 grid(blocks_for(p.n_chunks, kWavesPerBlock));
    const int n_tiles = (f + 31) / 32;
    return with_per(p.chunk_nnz, [&](auto per) {
        const int step = slices_a_walk(A.n_cols, n_tiles);
        for (int t = 0; t < n_tiles; t += step) hipLaunchKernelGGL(k_score_v2<per()>, grid, dim3(kBlock), 0, s, a, t, t + step < n_tiles ? t + step : n_tiles);
    });
}

hipError_t launch_v2_scores(const sensei_csr &A, const float *theta_l, const float *theta_r, const float *dP, int f, const float *att_padded, float slope,
                            float *logits, float *dalpha, float2 *stats, float2 *carry_stats, float *rowdot, float *carry, const ChunkPlan &p, hipStream_t s) {
    V2ScoresArgs a;
    a.n = nnz_args(A, p);
    a.theta_l = theta_l; a.theta_r = theta_r; a.dP = dP; a.att = att_padded; a.logits = logits; a.dalpha = dalpha; a.slope = slope;
    a.stats = stats; a.carry_stats = carry_stats; a.rowdot = rowdot; a.carry = carry;
    a.tl_tile = (long long)(A.n_rows > 0 ? A.n_rows : 1) * 32;
    a.tr_tile = (long long)(A.n_cols > 0 ? A.n_cols : 1) * 32;
    const dim3 grid(blocks_for(p.n_chunks, kWavesPerBlock));
    const int n_tiles = (f + 31) / 32, step = slices_a_walk(A.n_cols, n_tiles);
    return with_per(p.chunk_nnz, [&](auto per) {
        for (int t = 0; t < n_tiles; t += step) {
            const int t1 = t + step < n_tiles ? t + step : n_tiles;
            if (t1 == n_tiles) hipLaunchKernelGGL((k_v2_scores<true, per()>), grid, dim3(kBlock), 0, s, a, t, t1);
            else hipLaunchKernelGGL((k_v2_scores<false, per()>), grid, dim3(kBlock), 0, s, a, t, t1);
        }
        if (p.n_chunks > 1) hipLaunchKernelGGL(k_v2_scores_fixup, dim3(blocks_for(p.n_chunks - 1, kBlock)), dim3(kBlock), 0, s, a);
    });
}

hipError_t launch_gat_dt(const sensei_csr &A, const float *logits, const float *dalpha, const float *rowdot, const float2 *mz,
                         const int32_t *t_pos, float slope, float *dt, float2 *adt_t, const ChunkPlan &p, hipStream_t s, float *rowsum, float *carry) {
    if (A.nnz <= 0 && !rowsum) return hipSuccess;
    GatDtArgs a;
    a.n = nnz_args(A, p);
    a.logits = logits; a.dalpha = dalpha; a.rowdot = rowdot; a.mz = mz; a.t_pos = t_pos; a.dt = dt; a.adt_t = adt_t;
    a.rowsum = rowsum; a.carry = carry;
    a.slope = slope;
    const dim3 grid(blocks_by_xcd(p.n_chunks));
    return with_per(p.chunk_nnz, [&](auto per) {
        if (rowsum) hipLaunchKernelGGL((k_gat_dt<true, per()>), grid, dim3(kBlock), 0, s, a);
        else hipLaunchKernelGGL((k_gat_dt<false, per()>), grid, dim3(kBlock), 0, s, a);
        if (rowsum && p.n_chunks > 1)
            hipLaunchKernelGGL(k_sum_fixup, dim3(blocks_for(p.n_chunks - 1, kBlock)), dim3(kBlock), 0, s, a.n, rowsum, carry);
    });
}

hipError_t launch_rank1_add(float *D, int64_t ldd, int64_t n, int f, const float *ds_l, int64_t n_l, const float *ds_r, const float *a_l,
                            const float *a_r, hipStream_t s) {
    if (n <= 0 || f <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_rank1_add, dim3(blocks_for(n * f, kBlock)), dim3(kBlock), 0, s, D, (long long)ldd, (long long)n, f, ds_l, (long long)n_l,
                       ds_r, a_l, a_r);
    return hipGetLastError();
}

// the two walks of the GATv2 backward (see k_v2_walk); carry, carry_r: spmm_carry_bytes of the pattern at pad32(f) columns
hipError_t launch_v2_walk(const sensei_csr &A, const ChunkPlan &p, bool cols, const float *own, const float *other, const float *dP, const float *w,
                          const float *att_padded, float slope, int f, float *C, int64_t ldc, float *R, float *carry, float *carry_r, hipStream_t s) {
    V2WalkArgs a;
    a.n = nnz_args(A, p);
    a.own = own; a.other = other; a.dP = dP; a.w = w; a.att = att_padded; a.C = C; a.R = R; a.carry = carry; a.carry_r = carry_r;
    a.own_tile = (long long)(A.n_rows > 0 ? A.n_rows : 1) * 32;
    a.other_tile = (long long)(A.n_cols > 0 ? A.n_cols : 1) * 32;
    a.ldc = ldc; a.f = f; a.n_tiles = (f + 31) / 32; a.f_carry = a.n_tiles * 32; a.slope = slope;
    a.store_vec_ok = ldc % 4 == 0 && reinterpret_cast<uintptr_t>(C) % 16 == 0;
    a.tiles_live = a.other_tile * 4 > 8000000 ? 4 : 8;   // as in launch_spmm
    if (a.tiles_live > a.n_tiles) a.tiles_live = a.n_tiles;
    a.n_groups = (int)blocks_for(p.n_chunks, kWavesPerBlock);
    const dim3 grid((unsigned)(a.n_groups * a.tiles_live * ((a.n_tiles + a.tiles_live - 1) / a.tiles_live)));
    const hipError_t e = with_per(p.chunk_nnz, [&](auto per) {
        if (cols) hipLaunchKernelGGL((k_v2_walk<true, per()>), grid, dim3(kBlock), 0, s, a);
        else hipLaunchKernelGGL((k_v2_walk<false, per()>), grid, dim3(kBlock), 0, s, a);
    });
    if (e != hipSuccess || p.n_chunks <= 1) return e;
    SpmmArgs x = {};   // the carry slots of rows that span chunks: raw sums
    x.row_ptr = A.row_ptr; x.chunk_row = p.chunk_row; x.n_rows = A.n_rows; x.nnz = (int)A.nnz; x.chunk_nnz = p.chunk_nnz; x.n_chunks = p.n_chunks;
    x.f_carry = a.f_carry; x.c_tf = 32; x.c_shift = 5; x.act = SENSEI_ACT_NONE; x.fix_quads = p.n_chunks < 8192 ? 8 : 32;
    for (int out = 0; out < (cols ? 1 : 2); ++out) {
        x.C = out ? R : C; x.carry = out ? carry_r : carry;
        x.ldc = out ? 32 : ldc; x.c_tile = out ? a.own_tile : 32; x.f_store = out ? a.f_carry : f;
        x.store_vec_ok = out ? 1 : a.store_vec_ok;
        hipLaunchKernelGGL(k_spmm_fixup, dim3(blocks_for(p.n_chunks - 1, kWavesPerBlock * kFixupChunks), blocks_for(x.f_store, 4 * x.fix_quads)), dim3(kBlock), 0, s, x);
    }
    return hipGetLastError();
}

hipError_t launch_scale_cols(float *D, int64_t ldd, const float *G, int64_t ldg, const float *v, int64_t n, int f, bool accumulate, hipStream_t s) {
    if (n <= 0 || f <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_scale_cols, dim3(blocks_for(n * f, kBlock)), dim3(kBlock), 0, s, D, (long long)ldd, G, (long long)ldg, v, (long long)n, f,
                       accumulate ? 1 : 0);
    return hipGetLastError();
}

hipError_t launch_fill_f32(float *p, int64_t n, float v, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_set_f32, dim3(blocks_for(n, kBlock)), dim3(kBlock), 0, s, p, (long long)n, v);
    return hipGetLastError();
}

static int theta_t_slabs(int64_t n) {   // at least 128 rows (four passes of a workgroup) a slab, at most 512 slabs
    const int64_t slabs = (n + 127) / 128;
    return (int)(slabs < 1 ? 1 : slabs > 512 ? 512 : slabs);
}

size_t theta_t_vec_bytes(int64_t n, int f) { return align_up((size_t)theta_t_slabs(n) * 2 * (size_t)pad32(f) * sizeof(double), 256); }

hipError_t launch_theta_t_vec(const float *theta_sliced, int64_t n, int f, const float *v_l, int64_t n_l, const float *v_r, float *out_l,
                              float *out_r, double *part, hipStream_t s, int n_heads) {
    if (f <= 0) return hipSuccess;
    const int d = f / n_heads, width = n_heads > 1 ? n_heads * 32 : f;   // several heads: one slice each
    const int slabs = theta_t_slabs(n), f_pad = pad32(width);
    const int rows_per_slab = (int)((((n > 0 ? n : 1) + slabs - 1) / slabs + 31) / 32 * 32);
    hipLaunchKernelGGL(k_theta_t_vec, dim3((unsigned)(f_pad / 32), (unsigned)slabs), dim3(256), 0, s, theta_sliced, (long long)n, f_pad, v_l,
                       (long long)n_l, v_r, rows_per_slab, part, n_heads > 1 ? (long long)n : 0LL);
    hipLaunchKernelGGL(k_sum_slabs, dim3(blocks_for(width, 16)), dim3(256), 0, s, part, slabs, f_pad, width, out_l, out_r, n_heads > 1 ? d : width);
    return hipGetLastError();
}

// The two walks of the heads' backward (see k_gat_head_rows); `row` is scratch, written by the first and read by the second.
hipError_t launch_gat_heads_backward(const sensei_csr &A, const ChunkPlan &p, const sensei_csr &At, const ChunkPlan &pt, const GatHeadsBackward &b,
                                     hipStream_t s) {
    GatHeadArgs a;
    a.n = nnz_args(A, p);
    a.theta = b.theta; a.dP = b.dP; a.s_l = b.s_l; a.s_r = b.s_r; a.row = b.row; a.ds_l = b.ds_l; a.ds_r = b.ds_r; a.piece = b.piece;
    a.a_l = b.a_l; a.a_r = b.a_r;
    a.dtheta = b.dtheta; a.carry = b.carry; a.ds_carry = b.ds_carry;
    a.n_src = A.n_cols; a.n_dst = A.n_rows; a.ldd = b.ldd; a.d = b.d; a.slope = b.slope;
    a.store_vec_ok = b.ldd % 4 == 0 && b.d % 4 == 0 && reinterpret_cast<uintptr_t>(b.dtheta) % 16 == 0;
    const unsigned heads = (unsigned)b.heads;
    hipError_t e = with_per(p.chunk_nnz, [&](auto per) {
        hipLaunchKernelGGL(k_gat_head_rows<per()>, dim3(blocks_for(p.n_chunks, kWavesPerBlock), heads), dim3(kBlock), 0, s, a);
        if (p.n_chunks > 1) hipLaunchKernelGGL(k_gat_head_fixup, dim3(blocks_for(p.n_chunks - 1, kBlock), heads), dim3(kBlock), 0, s, a);
    });
    if (e != hipSuccess) return e;
    a.n = nnz_args(At, pt);
    return with_per(pt.chunk_nnz, [&](auto per) {
        hipLaunchKernelGGL(k_gat_head_cols<per()>, dim3(blocks_for(pt.n_chunks, kWavesPerBlock), heads), dim3(kBlock), 0, s, a);
        if (pt.n_chunks > 1)
            hipLaunchKernelGGL(k_gat_head_cols_fixup, dim3(blocks_for(pt.n_chunks - 1, kWavesPerBlock * 8), heads), dim3(kBlock), 0, s, a);
    });
}

hipError_t launch_transpose_pos(const sensei_csr &A, const sensei_csr &At, const ChunkPlan &p, int32_t *pos, int32_t *miss, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, s, miss, 1LL, 0);  // a fill kernel, not a memset: safe under stream capture too
    if (A.nnz <= 0) return hipGetLastError();
    hipLaunchKernelGGL(k_transpose_pos, dim3(blocks_for(p.n_chunks, kWavesPerBlock)), dim3(kBlock), 0, s, nnz_args(A, p), At.row_ptr, At.col_idx,
                       pos, miss);
    return hipGetLastError();
}


hipError_t launch_row_moments(const sensei_csr &A, unsigned long long *out2, hipStream_t s) {
    hipLaunchKernelGGL(k_fill_u64, dim3(1), dim3(64), 0, s, out2, 2, 0ull);
    if (A.n_rows > 0) hipLaunchKernelGGL(k_row_moments, dim3(blocks_for(A.n_rows, kBlock)), dim3(kBlock), 0, s, A.row_ptr, A.n_rows, out2);
    return hipGetLastError();
}

// ------------------------------------------------------------ column panels (host side)

hipError_t launch_exclusive_scan(int32_t *data, int n, int32_t *block_sums, hipStream_t s) {
    const unsigned nb = blocks_for(n, kScanPerBlock);
    hipLaunchKernelGGL(k_scan_local, dim3(nb), dim3(256), 0, s, data, n, block_sums);
    hipLaunchKernelGGL(k_scan_sums, dim3(1), dim3(64), 0, s, block_sums, (int)nb);
    hipLaunchKernelGGL(k_scan_add, dim3(nb), dim3(256), 0, s, data, n, (const int32_t *)block_sums);
    return hipGetLastError();
}

size_t scan_temp_bytes(int n) { return align_up(((size_t)blocks_for(n, kScanPerBlock) + 1) * sizeof(int32_t), 256); }

hipError_t launch_panel_build(const sensei_csr &A, const ChunkPlan &plan, int n_panels, int width, int32_t *const *rp, int32_t *off,
                              int32_t *col_out, int32_t *perm_out, int32_t *scan_temp, hipStream_t s) {
    PanelPtrs pp;
    for (int q = 0; q < kMaxPanels; ++q) pp.rp[q] = q < n_panels ? rp[q] : nullptr;
    hipLaunchKernelGGL(k_panel_count, dim3(blocks_for((long long)A.n_rows + 1, kBlock)), dim3(kBlock), 0, s, A.row_ptr, A.col_idx, A.n_rows,
                       n_panels, width, pp);
    hipError_t err = hipGetLastError();
    for (int q = 0; q < n_panels && err == hipSuccess; ++q) err = launch_exclusive_scan(rp[q], A.n_rows + 1, scan_temp, s);
    if (err != hipSuccess) return err;
    hipLaunchKernelGGL(k_panel_offsets, dim3(1), dim3(64), 0, s, pp, A.n_rows, n_panels, off);
    if (A.nnz > 0)
        hipLaunchKernelGGL(k_panel_scatter, dim3(blocks_for(plan.n_chunks, kWavesPerBlock)), dim3(kBlock), 0, s, nnz_args(A, plan), n_panels,
                           width, pp, (const int32_t *)off, col_out, perm_out);
    return hipGetLastError();
}

hipError_t launch_panel_segments(int32_t *const *rp, const int32_t *off, int n_rows, int n_panels, int32_t *seg_ptr, hipStream_t s) {
    PanelPtrs pp;
    for (int q = 0; q < kMaxPanels; ++q) pp.rp[q] = q < n_panels ? rp[q] : nullptr;
    hipLaunchKernelGGL(k_panel_segments, dim3(blocks_for((long long)n_panels * n_rows + 1, kBlock)), dim3(kBlock), 0, s, pp, off, n_rows, n_panels, seg_ptr);
    return hipGetLastError();
}

hipError_t launch_replicate_stats(const float2 *src, int64_t n, int copies, float2 *dst, hipStream_t s) {
    if (n <= 0 || copies <= 0) return hipSuccess;
    hipLaunchKernelGGL(k_replicate_f2, dim3(blocks_for(n * copies, kBlock)), dim3(kBlock), 0, s, src, (long long)n, copies, dst);
    return hipGetLastError();
}

// ------------------------------------------------------------ dense tiles (host side)

// exclusive scan of up to 2^31 ints: the block totals are scanned by the same three kernels instead of one thread
size_t scan_large_temp_bytes(long long n) {
    const long long nb = (n + kScanPerBlock - 1) / kScanPerBlock;
    return align_up((size_t)(nb + 1) * sizeof(int32_t), 256) + scan_temp_bytes((int)(nb + 1));
}

hipError_t launch_exclusive_scan_large(int32_t *data, long long n, int32_t *temp, hipStream_t s) {
    if (n <= 0) return hipSuccess;
    const unsigned nb = blocks_for(n, kScanPerBlock);
    int32_t *sums = temp;
    int32_t *temp2 = temp + align_up((size_t)(nb + 1) * sizeof(int32_t), 256) / sizeof(int32_t);
    hipLaunchKernelGGL(k_scan_local, dim3(nb), dim3(256), 0, s, data, (int)n, sums);
    const hipError_t e = launch_exclusive_scan(sums, (int)nb, temp2, s);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(k_scan_add, dim3(nb), dim3(256), 0, s, data, (int)n, (const int32_t *)sums);
    return hipGetLastError();
}

static TileMapArgs tile_map_args(const sensei_csr &A, const ChunkPlan &p, const int32_t *rank_r, const int32_t *rank_c, int h_r, int h_c, int nt_c) {
    TileMapArgs a;
    a.n = nnz_args(A, p);
    a.rank_r = rank_r; a.rank_c = rank_c; a.h_r = h_r; a.h_c = h_c; a.nt_c = nt_c;
    return a;
}

hipError_t launch_tile_select(const sensei_csr &A, const ChunkPlan &p, const int32_t *rank_r, const int32_t *rank_c, int h_r, int h_c,
                              int nt_r, int nt_c, int min_count, int32_t *hist, int32_t *sel_scan, int32_t *slot_of, int32_t *slot_ct,
                              int32_t *slot_rt, int32_t *rt_ptr, int32_t *scan_temp, hipStream_t s) {
    const int n_tiles = nt_r * nt_c;
    hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for(n_tiles, kBlock)), dim3(kBlock), 0, s, hist, (long long)n_tiles, 0);
    if (A.nnz > 0)
        hipLaunchKernelGGL(k_tile_hist, dim3(blocks_for(p.n_chunks, kWavesPerBlock)), dim3(kBlock), 0, s,
                           tile_map_args(A, p, rank_r, rank_c, h_r, h_c, nt_c), hist);
    hipLaunchKernelGGL(k_tile_flags, dim3(blocks_for(n_tiles + 1, kBlock)), dim3(kBlock), 0, s, (const int32_t *)hist, n_tiles, min_count, sel_scan);
    const hipError_t e = launch_exclusive_scan(sel_scan, n_tiles + 1, scan_temp, s);
    if (e != hipSuccess) return e;
    const int span = n_tiles > nt_r + 1 ? n_tiles : nt_r + 1;
    hipLaunchKernelGGL(k_tile_slots, dim3(blocks_for(span, kBlock)), dim3(kBlock), 0, s, (const int32_t *)hist, (const int32_t *)sel_scan, n_tiles,
                       nt_r, nt_c, min_count, slot_of, slot_ct, slot_rt, rt_ptr);
    return hipGetLastError();
}

hipError_t launch_tile_split(const sensei_csr &A, const ChunkPlan &p, const int32_t *rank_r, const int32_t *rank_c, int h_r, int h_c, int nt_c,
                             const int32_t *slot_of, int n_slots, unsigned *bits, int32_t *pos, int32_t *scan_temp, int32_t *col_rem,
                             int32_t *dst_rem, int32_t *row_ptr_rem, hipStream_t s) {
    if (n_slots > 0) hipLaunchKernelGGL(k_fill_i32, dim3(blocks_for((long long)n_slots * 512, kBlock)), dim3(kBlock), 0, s,
                                        reinterpret_cast<int32_t *>(bits), (long long)n_slots * 512, 0);
    hipLaunchKernelGGL(k_fill_i32, dim3(1), dim3(64), 0, s, pos + A.nnz, 1LL, 0);
    if (A.nnz > 0)
        hipLaunchKernelGGL(k_tile_mark, dim3(blocks_for(p.n_chunks, kWavesPerBlock)), dim3(kBlock), 0, s,
                           tile_map_args(A, p, rank_r, rank_c, h_r, h_c, nt_c), slot_of, bits, pos, dst_rem);
    const hipError_t e = launch_exclusive_scan_large(pos, (long long)A.nnz + 1, scan_temp, s);
    if (e != hipSuccess) return e;
    if (A.nnz > 0) hipLaunchKernelGGL(k_rem_scatter, dim3(blocks_for(A.nnz, kBlock)), dim3(kBlock), 0, s, nnz_args(A, p), (const int32_t *)pos, col_rem, dst_rem);
    hipLaunchKernelGGL(k_rem_rowptr, dim3(blocks_for((long long)A.n_rows + 1, kBlock)), dim3(kBlock), 0, s, A.row_ptr, A.n_rows, (const int32_t *)pos,
                       row_ptr_rem);
    return hipGetLastError();
}

// C (n x f, row-major with ldc, or slice-major when `sliced`) = 0
hipError_t launch_zero_matrix(float *C, int64_t n, int f, int64_t ldc, bool sliced, hipStream_t s) {
    if (n <= 0 || f <= 0) return hipSuccess;
    if (sliced || ldc == f) {
        const long long total = (long long)n * (sliced ? pad32(f) : f);
        if (total % 4 == 0 && reinterpret_cast<uintptr_t>(C) % 16 == 0) {
            hipLaunchKernelGGL(k_zero_f32, dim3(blocks_for(total / 4, kBlock)), dim3(kBlock), 0, s, C, total / 4);
            return hipGetLastError();
        }
        hipLaunchKernelGGL(k_zero_rows, dim3(blocks_for(total, kBlock)), dim3(kBlock), 0, s, C, total, 1, 1LL);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(k_zero_rows, dim3(blocks_for((long long)n * f, kBlock)), dim3(kBlock), 0, s, C, (long long)n, f, (long long)ldc);
    return hipGetLastError();
}

}  // namespace sensei
