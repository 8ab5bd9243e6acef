// Several levels of the merges in one kernel (included by hrc_kernels.hip,
// inside namespace hrc).
//
// Why.  Level by level, each merge reads and writes whole levels: 1.1 GB of
// traffic for a 1024^2 forward whose inputs and output are 12 MB, and one
// launch per level.  But the levels decompose: cone ii of level n and all its
// descendants read only directions ii and ii + 1 of T_n, and everything a
// lookup along a direction reaches lies on that direction's line.  So a block
// takes one cone ii of level n of one quadrant, a run of probe columns, and a
// window of rows that is sheared along the cone's lower edge, loads its part of
// T_n once into LDS and builds several levels from it on chip.
//
// Sheared windows.  The lower edge of cone ii climbs sb = 2 ii - 2^n rows per
// column of level n.  Window row r at column position p (in columns of level n
// from the block's anchor) is the grid row (y0 + r + p sb) mod S.  In these
// coordinates a lookup along direction K' = K - ii 2^j of level n + j moves
// 2 K' rows at the next column (0 <= K' <= 2^j), so all a window of W output
// rows needs is W + 2 d rows at distance d.  The windows are cyclic in y, so
// every grid row belongs to one window at every column and no block is half
// empty; a lookup whose row leaves the grid is replaced by a select on the
// unsheared row, as in the level-by-level passes.  An LDS row holds L = 128
// window rows; the last ones, whose lookups run into the next LDS row, hold no
// valid values and feed no stored one.
//
// Column 0 of a level is read by nothing but column 0 of the levels below,
// and the gather never reads that: the top and the down kernels leave it out.
//
// Measured at 1024^2 (FP32, four quadrants, per forward): T_2 -> T_4, T_6 23.7 us
// (four single levels 40), 107 MB at 4.5 TB/s; T_6 -> R_6 29.2 us (three levels up
// and four down: 76), bound by vector and scalar issue (35 and 40 thousand
// instructions a CU in 58 thousand cycles); R_6 -> R_4 -> R_2 21.2 us each (two
// single levels 24, but those need T_3 and T_5 stored), 67 MB, half HBM and half
// issue.  Forward 217.7 -> 119 us, 64^2 37 -> 18 us (3 launches for 11).  Block
// sizes: the LDS of a top or four-level block (78 and 58 KB) leaves two on a CU,
// so FP32 blocks of 1024 threads fill its 32 waves (512: 32 and 25.6 us); the
// 16-bit ones fit three to five (1024: 30.5 and 23.8 us, 512: 28.2 and 20.4), and
// a merge down four (512 threads: 24.0 and 24.8 us, 256: 24.0 and 22.6).  RGB
// intervals take twice the LDS, so twice the threads fill the chip again: merges
// up 85.5 -> 81.5 us, top 40.6 -> 37, one adjoint of two levels at 512^2 21.4 -> 17.5.
// Its merge down has 10 or 12 items per level: 12 waves take one each (256 threads: 97
// us, 512: 81 and 86, 768: 71 and 76, 1024: 76 and 82).  Wave counts that are no
// multiple of the CU's four SIMDs lose more than they save (one channel down:
// 256 threads 23 us, 320: 28.6, 384: 28.0).
//
// The arithmetic of every element, and its order, is that of the
// level-by-level bodies, and 16-bit intervals are rounded at the same points
// (LDS holds the storage type), so the results are bitwise the same.

// ---- interval storage types -------------------------------------------------

template <typename TS> struct Store;
template <> struct Store<float2> { using C = float2; static constexpr int ch = 1; };
template <> struct Store<half2_t> { using C = float2; static constexpr int ch = 1; };
template <> struct Store<float4> { using C = float4; static constexpr int ch = 3; };
template <> struct Store<half4_t> { using C = float4; static constexpr int ch = 3; };

// (native vectors: arrays of HIP's vector classes went to scratch memory)
template <int BYTES> struct RawVec {
    typedef unsigned type __attribute__((ext_vector_type(BYTES / 4)));
};
template <> struct RawVec<4> { using type = unsigned; };

__device__ __forceinline__ float trans(float2 v) { return v.y; }
__device__ __forceinline__ float trans(float4 v) { return v.w; }
__device__ __forceinline__ float rad(float2 v, int) { return v.x; }
__device__ __forceinline__ float rad(float4 v, int c) { return c == 0 ? v.x : c == 1 ? v.y : v.z; }
__device__ __forceinline__ float2 half_sum(float2 a, float2 b) {
    return make_float2(0.5f * (a.x + b.x), 0.5f * (a.y + b.y));
}
__device__ __forceinline__ float4 half_sum(float4 a, float4 b) {
    return make_float4(0.5f * (a.x + b.x), 0.5f * (a.y + b.y), 0.5f * (a.z + b.z),
                       0.5f * (a.w + b.w));
}

constexpr int kWindow = 128;  // window rows of an LDS row

// V consecutive intervals of a row as one vector access.
template <int V> __device__ __forceinline__ void ld_row(const float2 *p, float2 (&o)[V]) {
    if constexpr (V == 2) {
        const float4 v = *reinterpret_cast<const float4 *>(p);
        o[0] = lo(v);
        o[1] = hi(v);
    } else {
        o[0] = *p;
    }
}
template <int V> __device__ __forceinline__ void ld_row(const half2_t *p, float2 (&o)[V]) {
    if constexpr (V == 2) {
        const float4 v = ld_pair(p);
        o[0] = lo(v);
        o[1] = hi(v);
    } else {
        const half2_t v = *p;
        o[0] = make_float2((float)v.x, (float)v.y);
    }
}
template <int V> __device__ __forceinline__ void ld_row(const float4 *p, float4 (&o)[V]) {
#pragma unroll
    for (int i = 0; i < V; ++i) o[i] = p[i];
}
template <int V> __device__ __forceinline__ void ld_row(const half4_t *p, float4 (&o)[V]) {
    if constexpr (V == 2) {
        const half8_t v = *reinterpret_cast<const half8_t *>(p);
        cvt_quad(v, o[0], o[1]);
    } else {
        o[0] = ld4(p);
    }
}
template <int V> __device__ __forceinline__ void st_row(float2 *p, const float2 (&v)[V]) {
    if constexpr (V == 2)
        st_pair(p, pair(v[0], v[1]));
    else
        *p = v[0];
}
template <int V> __device__ __forceinline__ void st_row(half2_t *p, const float2 (&v)[V]) {
    if constexpr (V == 2)
        st_pair(p, pair(v[0], v[1]));
    else
        st_iv(p, v[0]);
}
template <int V> __device__ __forceinline__ void st_row(float4 *p, const float4 (&v)[V]) {
#pragma unroll
    for (int i = 0; i < V; ++i) p[i] = v[i];
}
template <int V> __device__ __forceinline__ void st_row(half4_t *p, const float4 (&v)[V]) {
    if constexpr (V == 2)
        st_quad(reinterpret_cast<half2_t *>(p), v[0], v[1]);
    else
        st_iv(p, v[0]);
}
// V consecutive floats of an angular fluence row.
template <int V> __device__ __forceinline__ void ld_f(const float *p, float (&o)[V]) {
    if constexpr (V == 2) {
        const float2 v = *reinterpret_cast<const float2 *>(p);
        o[0] = v.x;
        o[1] = v.y;
    } else {
        o[0] = *p;
    }
}
template <int V> __device__ __forceinline__ void st_f(float *p, const float (&v)[V]) {
    if constexpr (V == 2)
        *reinterpret_cast<float2 *>(p) = make_float2(v[0], v[1]);
    else
        *p = v[0];
}
// A computed interval as it reads back once stored.
__device__ __forceinline__ float2 stored(float2 v, const float2 *) { return v; }
__device__ __forceinline__ float4 stored(float4 v, const float4 *) { return v; }
__device__ __forceinline__ float2 stored(float2 v, const half2_t *) {
    return make_float2((float)to_half(v.x), (float)to_half(v.y));
}
__device__ __forceinline__ float4 stored(float4 v, const half4_t *) {
    return make_float4((float)to_half(v.x), (float)to_half(v.y), (float)to_half(v.z),
                       (float)to_half(v.w));
}

// ---- one block's window -------------------------------------------------------

// The block's quadrant (of the group), cone of level n, chunk of columns and
// first window row.
struct FuseTile {
    int q, ii, x, y0;
};

// Tiles in the order cone (its low three bits), window, cone, chunk, quadrant:
// neighbours in cone share a direction of T_n and neighbours in window their
// halo rows, so they run side by side on one XCD (each takes a contiguous
// eighth) and meet in its L2.  Every wave decodes its block's tile in the
// scalar unit, which the kernels keep nearly as busy as the vector units:
// shifts, and a multiplication in place of the division by the windows.
__device__ __forceinline__ FuseTile fuse_tile(const FuseArgs &a) {
    unsigned t = blockIdx.x;
    if (a.eighth) t = (t & 7u) * (unsigned)a.eighth + (t >> 3);
    const int lb = a.n < 3 ? a.n : 3;
    FuseTile f;
    f.ii = (int)(t & ((1u << lb) - 1));
    t >>= lb;
    const unsigned d = a.inv_nwin ? (unsigned)(((unsigned long long)t * a.inv_nwin) >> 32) : t;
    f.y0 = (int)(t - d * (unsigned)a.nwin) * a.win;
    f.ii |= (int)(d & ((1u << (a.n - lb)) - 1)) << lb;
    t = d >> (a.n - lb);
    f.x = (int)(t & ((1u << a.lchunks) - 1));
    f.q = (int)(t >> a.lchunks);
    return f;
}

// Row state of one lane: window row r (V consecutive ones), and the grid row
// of r at column position p.
template <int V> struct Rows {
    int r, base, sb, mask;
    __device__ __forceinline__ Rows(int r_, int y0, int sb_, int S)
        : r(r_), base(y0 + r_), sb(sb_), mask(S - 1) {}
    __device__ __forceinline__ int y(int p) const { return (base + p * sb) & mask; }
    __device__ __forceinline__ bool in(int yt) const { return (unsigned)yt <= (unsigned)mask; }
};
// Whether the rows of a whole window at every column position 0 .. p lie in the
// grid, unwrapped: then no lookup of the block leaves it, and none needs a select.
__device__ __forceinline__ bool window_inside(int y0, int p, int sb, int S) {
    const int d = p * sb;
    return y0 + (d < 0 ? d : 0) >= 0 && y0 + (d > 0 ? d : 0) + kWindow <= S;
}

// Directions 2k and 2k + 1 (relative to the block's lower edge) of one column
// of level m: Eq. 18, and the mean of Eq. 19-20.  nb: the lane's interval of
// direction k of the near column at level m - 1 (directions L apart), far: how
// far behind it the far column's direction k lies.  yv: the output's grid row
// plus the rows a column of level m - 1 climbs along the lower edge.  The far
// lookups run 2k rows up for direction k and 2k + 2 for k + 1, so apart from
// two bases each every LDS offset is an immediate.  next: the offset of direction
// k + 1, L, or 0 at the column's last direction (no 2k + 1 there, odd is not used):
// the row after that one is the next column's first, or at the last column one past
// the level.  (1024^2 forward 119 us so, 143 with a branch around the three reads.)
template <typename TS, int V, int L, bool ODD, bool IN>
__device__ __forceinline__ void fused_up(const TS *nb, int far, int k, const Rows<V> &w, int yv,
                                         typename Store<TS>::C (&even)[V],
                                         typename Store<TS>::C (&odd)[V], int next) {
    using C = typename Store<TS>::C;
    const TS *fb = nb + far + 2 * k;
    C n0[V], n1[V], f00[V], f02[V], f10[V];
    ld_row<V>(nb, n0);
    ld_row<V>(fb, f00);  // direction k, 2k rows up
    if constexpr (ODD) {
        ld_row<V>(nb + next, n1);
        ld_row<V>(fb + 2, f02);  // direction k, 2k + 2 rows up
        ld_row<V>(fb + next, f10);  // direction k + 1, 2k rows up
    }
    const bool in0 = IN || w.in(yv + 2 * k), in1 = IN || w.in(yv + 2 * k + 2);
    if constexpr (!IN) {
        // every read issued before the selects (else each far read becomes a
        // branch that waits for it)
#pragma unroll
        for (int i = 0; i < V; ++i) {
            pin(f00[i]);
            if constexpr (ODD) {
                pin(f02[i]);
                pin(f10[i]);
            }
        }
        // most waves have every lookup in the grid: one branch spares them the
        // selects
        if (!__all(in0 && in1)) {
#pragma unroll
            for (int i = 0; i < V; ++i) {
                f00[i] = in0 ? f00[i] : empty_interval<C>();
                if constexpr (ODD) {
                    f02[i] = in1 ? f02[i] : empty_interval<C>();
                    f10[i] = in0 ? f10[i] : empty_interval<C>();
                }
            }
        }
    }
#pragma unroll
    for (int i = 0; i < V; ++i) {
        even[i] = merge(n0[i], f00[i]);
        if constexpr (ODD) odd[i] = half_sum(merge(n1[i], f02[i]), merge(n0[i], f10[i]));
    }
}

// The light from beyond the grid (wt.y, wt.w) for the looked-up fluences of the
// two cones whose probe (far) or row (in0, in1) lies outside.
template <int CH, int V, bool IN>
__device__ __forceinline__ void select_light(float (&f)[2][CH][V], bool far, bool in0, bool in1,
                                             float4 wt) {
    if (IN && far) return;
#pragma unroll
    for (int i = 0; i < 2 * CH * V; ++i) pin(f[i / (CH * V)][i / V % CH][i % V]);
    in0 = far && (IN || in0);
    in1 = far && (IN || in1);
    if (__all(in0 && in1)) return;
#pragma unroll
    for (int c = 0; c < CH; ++c)
#pragma unroll
        for (int j = 0; j < V; ++j) {
            f[0][c][j] = in0 ? f[0][c][j] : wt.y;
            f[1][c][j] = in1 ? f[1][c][j] : wt.w;
        }
}

// Eq. 14 (odd column): R_{m-1} of cone k (relative).  t: the lane's interval of
// direction k of T_{m-1} at this column; rm: the lane's row of cone 2k of R_m at
// the next probe, 2k rows up (NULL where that probe lies beyond the grid); wt:
// cone weights and light from beyond the grid of the cones 2k, 2k + 1 (A, E, A, E).
template <typename TS, int V, int L, bool IN>
__device__ __forceinline__ void fused_down_odd(const TS *t, const float *rm, bool far, int k,
                                               float4 wt, const Rows<V> &w, int yv,
                                               float (&o)[Store<TS>::ch][V]) {
    using C = typename Store<TS>::C;
    constexpr int CH = Store<TS>::ch;
    C tv[2][V];
    float f[2][CH][V];
#pragma unroll
    for (int up = 0; up < 2; ++up) {
        ld_row<V>(t + up * L, tv[up]);
#pragma unroll
        for (int c = 0; c < CH; ++c) ld_f<V>(rm + (up * CH + c) * L + 2 * up, f[up][c]);
    }
    select_light<CH, V, IN>(f, far, w.in(yv + 2 * k), w.in(yv + 2 * k + 2), wt);
#pragma unroll
    for (int up = 0; up < 2; ++up) {
        const float A = up ? wt.z : wt.x;
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int j = 0; j < V; ++j) {
                const float v = fmaf(trans(tv[up][j]), f[up][c][j], A * rad(tv[up][j], c));
                o[c][j] = up ? o[c][j] + v : v;
            }
    }
}

// Eq. 15-17 (even column 2c): the co-located probe c of R_m averaged with the
// doubled edges T_m(c, 2k), T_m(c, 2k + 2) (e: already in registers) to the
// probe c + 1.  rn: the lane's row of cone 2k at probe c; rf: of cone 2k at probe
// c + 1, 4k rows up (far: that probe lies in the grid).
template <typename TS, int V, int L, bool IN>
__device__ __forceinline__ void fused_down_even(const typename Store<TS>::C (&e)[2][V],
                                                const float *rn, const float *rf, bool far, int k,
                                                float4 wt, const Rows<V> &w, int yv,
                                                float (&o)[Store<TS>::ch][V]) {
    constexpr int CH = Store<TS>::ch;
    float f0[2][CH][V], f1[2][CH][V];
#pragma unroll
    for (int up = 0; up < 2; ++up)
#pragma unroll
        for (int c = 0; c < CH; ++c) {
            ld_f<V>(rn + (up * CH + c) * L, f0[up][c]);
            ld_f<V>(rf + (up * CH + c) * L + 4 * up, f1[up][c]);
        }
    select_light<CH, V, IN>(f1, far, w.in(yv + 4 * k), w.in(yv + 4 * k + 4), wt);
#pragma unroll
    for (int up = 0; up < 2; ++up) {
        const float A = up ? wt.z : wt.x;
#pragma unroll
        for (int c = 0; c < CH; ++c)
#pragma unroll
            for (int j = 0; j < V; ++j) {
                const float v = 0.5f * (f0[up][c][j] +
                                        fmaf(trans(e[up][j]), f1[up][c][j], A * rad(e[up][j], c)));
                o[c][j] = up ? o[c][j] + v : v;
            }
    }
}

// Cone weights and light from beyond the grid of every cone pair of the levels
// n .. n + M - 1 of the block's cone: entry 2^j - 1 + k for cone k of level n + j,
// thread t's entry t (the threads past the last repeat it).
template <int M>
__device__ __forceinline__ float4 load_weight(int n, int ii, const float *envq, int tid) {
    const int t = tid < (1 << M) - 1 ? tid : (1 << M) - 2;
    const int j = 31 - __clz(t + 1), k = t + 1 - (1 << j);
    const int cone = (2 << (n + j)) - 1 + (((ii << j) + k) << 1);
    float4 w = make_float4(c_cone[cone], 0.f, c_cone[cone + 1], 0.f);
    if (envq) {
        w.y = envq[cone];
        w.w = envq[cone + 1];
    }
    return w;
}
// Entries of padding after a level in LDS: lookups of rows past the valid ones run up
// to 16 entries past their row (direction 8 of the fourth level up), and behind the
// last row of a level come rows that other waves are storing, or the array's end.
constexpr int kFusePad = 16;

// Two directions of COLS columns of T_n into LDS, in two halves so that other
// loads can be issued between: load() takes the columns first_col .. into
// registers, store() puts direction ii + d of column i into LDS row
// 2 slot(i) + d.  The loads take no branch (a wave past the last row loads it
// again), so that every one is in flight before the first wait; its store is left
// out, behind a pin that keeps the load out of that branch.  Columns past the grid's last
// repeat it (and feed no stored value).
template <typename TS, int V, int L, int NT, int COLS> struct TnLoad {
    using Raw = typename RawVec<sizeof(TS) * V>::type;
    static constexpr int H = L / (64 * V), ROWS = COLS * 2 * H, NW = NT / 64, IT = (ROWS + NW - 1) / NW;
    Raw v[IT];
    __device__ __forceinline__ static int row(int it, int wave) {
        const int i = it * NW + wave;
        return (it + 1) * NW <= ROWS ? i : i < ROWS ? i : ROWS - 1;
    }
    __device__ __forceinline__ void load(const TS *T, int N, int n, int ii, int first_col, int y0,
                                         int sb, int wave, int lane) {
        const int S = 1 << N, dirs = (1 << n) + 1, C = S >> n;
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int i = row(it, wave), h = i % H, rd = i / H, x = first_col + (rd >> 1), d = rd & 1;
            const Rows<V> w((h * 64 + lane) * V, y0, sb, S);
            const int xc = x < C ? x : C - 1;
            v[it] = *reinterpret_cast<const Raw *>(
                T + (((unsigned)(xc * dirs + ii + d) << N) + (unsigned)w.y(rd >> 1)));
        }
    }
    template <typename Slot>
    __device__ __forceinline__ void store(TS *lds, int wave, int lane, Slot slot) {
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            if ((it + 1) * NW > ROWS) {
                pin_raw(v[it]);
                if (it * NW + wave >= ROWS) break;
            }
            const int i = row(it, wave), h = i % H, rd = i / H, d = rd & 1;
            *reinterpret_cast<Raw *>(lds + (slot(rd >> 1) * 2 + d) * L + (h * 64 + lane) * V) = v[it];
        }
    }
};

// ---- merge up of G levels: T_n -> T_{n+G} ----------------------------------------

// A block builds one column X of T_{n+G} for one cone of level n from the 2^G
// columns of T_n below it.  Levels alternate between two LDS regions.  Every
// level with a destination in a.T is stored (the last one always).
template <typename TS, int G> struct FuseUp {
    static constexpr int L = kWindow, V = sizeof(TS) == 16 ? 1 : 2, H = L / (64 * V);
    static constexpr int NT = (G == 2 ? 256 : G == 3 || sizeof(TS) == 4 ? 512 : 1024) << (sizeof(TS) == 16);
    static constexpr int NW = NT / 64;
    static constexpr int win = L - (2 << G);  // 2 (2^G - 1) rows of halo
    static constexpr int rows(int j) { return (1 << (G - j)) * ((1 << j) + 1); }
    static constexpr int region(int p) {
        int m = 0;
        for (int j = p; j < G; j += 2) m = rows(j) > m ? rows(j) : m;
        return m;
    }
    static constexpr int reg1 = region(0) * L + kFusePad;  // first entry of the second region
    static constexpr int lds = (reg1 + region(1) * L + kFusePad) * (int)sizeof(TS);
    static_assert((2 << (G - 1)) <= kFusePad, "the last level's lookups");
};

template <typename TS, int G, int j, bool IN>
__device__ __forceinline__ void fuse_up_level(const FuseArgs &a, const FuseTile &t, char *lds,
                                              int own, int sb, int tid) {
    using F = FuseUp<TS, G>;
    using C = typename Store<TS>::C;
    constexpr int V = F::V, L = F::L, H = F::H, NW = F::NW;
    constexpr int dirs = (1 << j) + 1, pdirs = (1 << (j - 1)) + 1, cols = 1 << (G - j);
    const int N = a.N, S = 1 << N, m = a.n + j;
    TS *reg0 = reinterpret_cast<TS *>(lds), *reg1 = reg0 + F::reg1;
    const TS *src = (j & 1) ? reg0 : reg1;
    TS *dst = (j & 1) ? reg1 : reg0;
    TS *out = reinterpret_cast<TS *>(a.T[j]);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    // the last direction is the next cone's first: stored by the last cone only
    const bool last = t.ii == (1 << a.n) - 1;
    for (int i = wave; i < cols * pdirs * H; i += NW) {
        const int h = i % H, e = i / H, X = e & (cols - 1), k = e >> (G - j);
        const bool two = k + 1 < pdirs;  // direction 2k + 1 as well
        const Rows<V> w((h * 64 + lane) * V, t.y0, sb, S);
        const int y = w.y(X << j);
        C ev[V], od[V];
        fused_up<TS, V, L, true, IN>(src + (2 * X * pdirs + k) * L + w.r, pdirs * L, k, w,
                                     y + (sb << (j - 1)), ev, od, two ? L : 0);
        if constexpr (j < G) {
            TS *d = dst + (X * dirs + 2 * k) * L + w.r;
            st_row<V>(d, ev);
            if (two) st_row<V>(d + L, od);
        }
        if ((j == G || out) && w.r < own) {
            TS *o = out + ((unsigned)t.q * a.te[j] +
                           ((unsigned)(((t.x << (G - j)) + X) * ((1 << m) + 1) + (t.ii << j) + 2 * k)
                            << N));
            if (two || last) st_row<V>(o + (unsigned)y, ev);
            if (two) st_row<V>(o + (unsigned)(y + S), od);
        }
    }
}

template <typename TS, int G, bool IN>
__device__ __forceinline__ void fuse_up_levels(const FuseArgs &a, const FuseTile &t, char *lds,
                                               int own, int sb, int tid) {
    fuse_up_level<TS, G, 1, IN>(a, t, lds, own, sb, tid);
    __syncthreads();
    fuse_up_level<TS, G, 2, IN>(a, t, lds, own, sb, tid);
    if constexpr (G >= 3) {
        __syncthreads();
        fuse_up_level<TS, G, 3, IN>(a, t, lds, own, sb, tid);
    }
    if constexpr (G >= 4) {
        __syncthreads();
        fuse_up_level<TS, G, 4, IN>(a, t, lds, own, sb, tid);
    }
}

template <typename TS, int G>
__device__ __forceinline__ void fuse_up_block(const FuseArgs &a, char *lds, int tid) {
    using F = FuseUp<TS, G>;
    const int N = a.N, S = 1 << N, n = a.n;
    const FuseTile t = fuse_tile(a);
    const int sb = 2 * t.ii - (1 << n);
    const int own = a.win < S - t.y0 ? a.win : S - t.y0;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    TnLoad<TS, F::V, F::L, F::NT, (1 << G)> ld;
    ld.load(reinterpret_cast<const TS *>(a.T[0]) + (unsigned)t.q * a.te[0], N, n, t.ii, t.x << G, t.y0,
            sb, wave, lane);
    ld.store(reinterpret_cast<TS *>(lds), wave, lane, [](int i) { return i; });
    __syncthreads();
    if (window_inside(t.y0, (1 << G) - 1, sb, S)) fuse_up_levels<TS, G, true>(a, t, lds, own, sb, tid);
    else fuse_up_levels<TS, G, false>(a, t, lds, own, sb, tid);
}

// ---- the top M levels: T_n -> R_n, n = N - M -------------------------------------

// A block holds every column but 0 of one cone's T_n .. T_{N-1}, then merges
// down from R_N to R_n.  The R levels alternate between two regions; where
// they fit, those lie over T_n's even columns, which only the merge up of
// T_{n+1} reads (T_n's odd columns come first in LDS).
template <typename TS, int M> struct FuseTop {
    static constexpr int L = kWindow, ch = Store<TS>::ch;
    static constexpr int V = sizeof(TS) == 16 ? 1 : 2, H = L / (64 * V);
    static constexpr int NT = (M == 4 && sizeof(TS) == 8) || sizeof(TS) == 16 ? 1024 : 512, NW = NT / 64;
    static constexpr int win = L - 2 * ((1 << M) - 1);  // halo: from column 1 to the far edge
    static constexpr int cols(int j) { return (1 << (M - j)) - 1; }
    static constexpr int t_rows(int j) { return cols(j) * ((1 << j) + 1); }
    static constexpr int t_off(int j) {  // first entry of T_{n+j}
        int o = 0;
        for (int i = 0; i < j; ++i) o += t_rows(i) * L + kFusePad;
        return o;
    }
    static constexpr int r_rows(int j) { return cols(j) * (1 << j) * ch; }
    static constexpr int r_region(int p) {  // float rows of the levels j >= 1 of parity p
        int m = 0;
        for (int j = p == 0 ? 2 : 1; j < M; j += 2) m = r_rows(j) > m ? r_rows(j) : m;
        return m;
    }
    static constexpr int t_bytes = t_off(M) * (int)sizeof(TS);
    static constexpr int r1_at = r_region(0) * L + kFusePad;  // the odd levels' region
    static constexpr int r_bytes = (r1_at + r_region(1) * L + kFusePad) * 4;
    static constexpr int odd_bytes = (1 << (M - 1)) * 2 * L * (int)sizeof(TS);
    static constexpr bool overlay = t_rows(0) * L * (int)sizeof(TS) - odd_bytes >= r_bytes;
    static constexpr int r_off = overlay ? odd_bytes : t_bytes;
    static constexpr int w_off = overlay ? t_bytes : t_bytes + r_bytes;
    static constexpr int lds = w_off + 16 * ((1 << M) - 1);
    // LDS column of T_n's column x: odd columns first
    __device__ __forceinline__ static int slot(int x) {
        return (x & 1) ? x >> 1 : (1 << (M - 1)) + (x >> 1) - 1;
    }
};

// First entry (direction 0, cone 0) of column x of T_{n+j}; of R_{n+j}.
template <typename TS, int M, int j> __device__ __forceinline__ TS *top_t(char *lds, int x) {
    using F = FuseTop<TS, M>;
    const int c = j == 0 ? F::slot(x) : x - 1;
    return reinterpret_cast<TS *>(lds) + F::t_off(j) + c * ((1 << j) + 1) * F::L;
}
template <typename TS, int M, int j> __device__ __forceinline__ float *top_r(char *lds, int x) {
    using F = FuseTop<TS, M>;
    return reinterpret_cast<float *>(lds + F::r_off) +
           ((j & 1) ? F::r1_at : 0) + (x - 1) * (1 << j) * F::ch * F::L;
}

template <typename TS, int M, int j, bool IN>
__device__ __forceinline__ void fuse_top_up(const FuseArgs &a, const FuseTile &t, char *lds, int own,
                                            int sb, int tid) {
    using F = FuseTop<TS, M>;
    using C = typename Store<TS>::C;
    constexpr int V = F::V, L = F::L, H = F::H, NW = F::NW, pdirs = (1 << (j - 1)) + 1;
    const int N = a.N, S = 1 << N, m = a.n + j;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const bool last = t.ii == (1 << a.n) - 1;
    TS *out = reinterpret_cast<TS *>(a.T[j]);
    for (int i = wave; i < F::cols(j) * pdirs * H; i += NW) {
        const int h = i % H, e = i / H, X = 1 + e / pdirs, k = e % pdirs;
        const bool two = k + 1 < pdirs;
        const Rows<V> w((h * 64 + lane) * V, t.y0, sb, S);
        const int y = w.y((X << j) - 1);
        // T_n's odd columns lie first, so its far column is 2^(M-1) - 1 columns back
        constexpr int far = j == 1 ? (1 - (1 << (M - 1))) * 2 * L : pdirs * L;
        C ev[V], od[V];
        fused_up<TS, V, L, true, IN>(top_t<TS, M, j - 1>(lds, 2 * X) + k * L + w.r, far, k, w,
                                     y + (sb << (j - 1)), ev, od, two ? L : 0);
        TS *d = top_t<TS, M, j>(lds, X) + 2 * k * L + w.r;
        st_row<V>(d, ev);
        if (two) st_row<V>(d + L, od);
        if (out && w.r < own) {
            TS *o = out + ((unsigned)t.q * a.te[j] +
                           ((unsigned)(X * ((1 << m) + 1) + (t.ii << j) + 2 * k) << N));
            if (two || last) st_row<V>(o + (unsigned)y, ev);
            if (two) st_row<V>(o + (unsigned)(y + S), od);
        }
    }
}

template <typename TS, int M, int j, bool IN>
__device__ __forceinline__ void fuse_top_down(const FuseArgs &a, const FuseTile &t, char *lds,
                                              int own, int sb, int tid) {
    using F = FuseTop<TS, M>;
    using C = typename Store<TS>::C;
    constexpr int V = F::V, L = F::L, H = F::H, NW = F::NW, CH = F::ch, cones = 1 << j;
    const int N = a.N, S = 1 << N, nn = a.n + j;  // output level
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    const float4 *wl = reinterpret_cast<const float4 *>(lds + F::w_off) + cones - 1;
    float *out = a.R[j];
    const size_t plane = (size_t)a.nq << (2 * N);
    for (int i = wave; i < F::cols(j) * cones * H; i += NW) {
        const int h = i % H, e = i / H, x = 1 + e / cones, k = e % cones;
        const Rows<V> w((h * 64 + lane) * V, t.y0, sb, S);
        const int y = w.y((x << j) - 1);
        const float4 wt = wl[k];
        float o[CH][V];
        if (x & 1) {
            const TS *tb = top_t<TS, M, j>(lds, x) + k * L + w.r;
            if constexpr (j + 1 < M) {
                // a probe past the last column is the light from beyond the grid
                const int c = (x + 1) >> 1, cc = c <= F::cols(j + 1) ? c : c - 1;
                const float *rm = top_r<TS, M, j + 1>(lds, cc > 0 ? cc : 1) + (2 * CH * L + 2) * k + w.r;
                fused_down_odd<TS, V, L, IN>(tb, rm, c <= F::cols(j + 1), k, wt, w, y + (sb << j), o);
            } else {
                // R_N is the light from beyond the grid
                C tv[2][V];
#pragma unroll
                for (int up = 0; up < 2; ++up) ld_row<V>(tb + up * L, tv[up]);
#pragma unroll
                for (int c = 0; c < CH; ++c)
#pragma unroll
                    for (int v = 0; v < V; ++v) {
                        o[c][v] = fmaf(trans(tv[0][v]), wt.y, wt.x * rad(tv[0][v], c));
                        o[c][v] += fmaf(trans(tv[1][v]), wt.w, wt.z * rad(tv[1][v], c));
                    }
            }
        } else {
            if constexpr (j + 1 < M) {
                const int cc = x >> 1;
                const bool far = cc + 1 <= F::cols(j + 1);
                C ed[2][V];
#pragma unroll
                for (int up = 0; up < 2; ++up)
                    ld_row<V>(top_t<TS, M, j + 1>(lds, cc) + 2 * (k + up) * L + w.r, ed[up]);
                const float *rn = top_r<TS, M, j + 1>(lds, cc) + 2 * CH * L * k + w.r;
                const float *rf = rn + (far ? (2 << j) * CH * L : 0) + 4 * k;
                fused_down_even<TS, V, L, IN>(ed, rn, rf, far, k, wt, w, y + 2 * (sb << j), o);
            }
        }
        if constexpr (j > 0) {
            float *dst = top_r<TS, M, j>(lds, x) + k * CH * L + w.r;
#pragma unroll
            for (int c2 = 0; c2 < CH; ++c2) st_f<V>(dst + c2 * L, o[c2]);
        }
        if ((j == 0 || out) && w.r < own) {
            float *op = out + (((unsigned)t.q << (2 * N)) +
                               ((unsigned)((x << nn) | ((t.ii << j) + k)) << N));
#pragma unroll
            for (int c2 = 0; c2 < CH; ++c2) st_f<V>(op + c2 * plane + (unsigned)y, o[c2]);
        }
    }
}

template <typename TS, int M, bool IN>
__device__ __forceinline__ void fuse_top_levels(const FuseArgs &a, const FuseTile &t, char *lds,
                                                int own, int sb, int tid) {
    fuse_top_up<TS, M, 1, IN>(a, t, lds, own, sb, tid);
    __syncthreads();
    if constexpr (M >= 3) {
        fuse_top_up<TS, M, 2, IN>(a, t, lds, own, sb, tid);
        __syncthreads();
    }
    if constexpr (M >= 4) {
        fuse_top_up<TS, M, 3, IN>(a, t, lds, own, sb, tid);
        __syncthreads();
        fuse_top_down<TS, M, 3, IN>(a, t, lds, own, sb, tid);
        __syncthreads();
    }
    if constexpr (M >= 3) {
        fuse_top_down<TS, M, 2, IN>(a, t, lds, own, sb, tid);
        __syncthreads();
    }
    fuse_top_down<TS, M, 1, IN>(a, t, lds, own, sb, tid);
    __syncthreads();
    fuse_top_down<TS, M, 0, IN>(a, t, lds, own, sb, tid);
}

template <typename TS, int M>
__device__ __forceinline__ void fuse_top_block(const FuseArgs &a, char *lds, int tid) {
    using F = FuseTop<TS, M>;
    const int N = a.N, S = 1 << N, n = a.n;
    const FuseTile t = fuse_tile(a);
    const int sb = 2 * t.ii - (1 << n);
    const int own = a.win < S - t.y0 ? a.win : S - t.y0;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    TnLoad<TS, F::V, F::L, F::NT, F::cols(0)> ld;
    ld.load(reinterpret_cast<const TS *>(a.T[0]) + (unsigned)t.q * a.te[0], N, n, t.ii, 1, t.y0, sb, wave,
            lane);
    const float4 wt = load_weight<M>(
        n, t.ii, a.env ? a.env + (size_t)(a.q0 + t.q) * kConeTable : nullptr, tid);
    ld.store(reinterpret_cast<TS *>(lds), wave, lane, [](int i) { return F::slot(i + 1); });
    if (tid < (1 << M) - 1) reinterpret_cast<float4 *>(lds + F::w_off)[tid] = wt;
    __syncthreads();
    if (window_inside(t.y0, (1 << M) - 2, sb, S)) fuse_top_levels<TS, M, true>(a, t, lds, own, sb, tid);
    else fuse_top_levels<TS, M, false>(a, t, lds, own, sb, tid);
}

// ---- merge down of two levels: (T_n, R_{n+2}) -> R_n, n >= 2 -------------------------

// A block computes R_n at the columns x0 + 1 .. x0 + CC (x0 a multiple of CC) of
// one cone: these read columns 1 .. CC/2 + 1 (from x0/2) of R_{n+1} and 1 ..
// CC/4 + 1 (from x0/4) of R_{n+2}; T_{n+1}, and the even directions of
// T_{n+2}, are rebuilt from T_n's columns x0 + 1 .. x0 + CC + 3.  R_{n+2} and
// R_{n+1} lie over the columns of T_n that only the rebuild reads, where they fit
// (R_{n+2} waits for its place in registers).
template <typename TS> struct FuseDown {
    static constexpr int L = kWindow, V = sizeof(TS) == 16 ? 1 : 2, H = L / (64 * V);
    static constexpr int ch = Store<TS>::ch, NT = ch == 3 ? 768 : 256, NW = NT / 64;
    static constexpr int CC = sizeof(TS) == 16 ? 4 : 8;
    // R_n looks up to 4 rows into R_{n+1}, that up to 8 into R_{n+2}: six columns on
    static constexpr int win = L - 12;
    static constexpr int c0 = CC + 3, c1 = CC / 2 + 1, c2 = CC / 4 + 1;  // columns per level
    static constexpr int t0_rows = 2 * c0, t1_rows = 3 * c1;
    static constexpr int odd_bytes = (CC / 2) * 2 * L * (int)sizeof(TS);
    static constexpr int t1_at = t0_rows * L + kFusePad;  // first entry of T_{n+1}
    static constexpr int t_bytes = (t1_at + t1_rows * L + kFusePad) * (int)sizeof(TS);
    static constexpr int r2_bytes = c2 * 4 * ch * L * 4, r1_bytes = c1 * 2 * ch * L * 4;
    static constexpr bool overlay =
        t0_rows * L * (int)sizeof(TS) - odd_bytes >= r1_bytes + r2_bytes;
    static constexpr int r1_off = overlay ? odd_bytes : t_bytes, r2_off = r1_off + r1_bytes;
    static constexpr int w_off =
        t_bytes + (overlay ? 0 : r1_bytes + r2_bytes + kFusePad * 4);
    static constexpr int lds = w_off + 16 * 3;
    // LDS column of T_n's column x0 + i: the odd ones below CC first, then the
    // rest in order
    __device__ __forceinline__ static int slot(int i) {
        return i >= CC ? i - 1 : (i & 1) ? i >> 1 : CC / 2 + (i >> 1) - 1;
    }
};

// R_{n+2} of the block's window: into registers, later into LDS (as TnLoad).
template <typename TS> struct R2Load {
    using F = FuseDown<TS>;
    static constexpr int V = F::V, H = F::H, CH = F::ch, ROWS = F::c2 * 4 * CH * H;
    static constexpr int IT = (ROWS + F::NW - 1) / F::NW;
    using Raw = typename RawVec<4 * V>::type;
    Raw v[IT];
    __device__ __forceinline__ static int row(int it, int wave) {
        const int i = it * F::NW + wave;
        return (it + 1) * F::NW <= ROWS ? i : i < ROWS ? i : ROWS - 1;
    }
    __device__ __forceinline__ void load(const FuseArgs &a, const FuseTile &t, int sb, int wave, int lane) {
        const int N = a.N, S = 1 << N, n = a.n, x0 = t.x * F::CC, last = (S >> (n + 2)) - 1;
        const size_t plane = (size_t)a.nq << (2 * N);
        const float *R2 = a.R[2] + ((unsigned)t.q << (2 * N));
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            const int i = row(it, wave), h = i % H, e = i / H, pl = e % CH, k = (e / CH) & 3;
            const int c = 1 + e / (4 * CH), X = (x0 >> 2) + c;
            const Rows<V> w((h * 64 + lane) * V, t.y0, sb, S);
            v[it] = *reinterpret_cast<const Raw *>(
                R2 + pl * plane +
                (((unsigned)(((X < last ? X : last) << (n + 2)) | (4 * t.ii + k)) << N) +
                 (unsigned)w.y(4 * c - 1)));
        }
    }
    __device__ __forceinline__ void store(float *r2, int wave, int lane) {
#pragma unroll
        for (int it = 0; it < IT; ++it) {
            if ((it + 1) * F::NW > ROWS) {
                pin_raw(v[it]);
                if (it * F::NW + wave >= ROWS) break;
            }
            const int i = row(it, wave);
            *reinterpret_cast<Raw *>(r2 + (i / H) * F::L + ((i % H) * 64 + lane) * V) = v[it];
        }
    }
};

template <typename TS, bool IN>
__device__ __forceinline__ void fuse_down_levels(const FuseArgs &a, const FuseTile &t, char *lds,
                                                 R2Load<TS> &rl, int own, int sb, int tid) {
    using F = FuseDown<TS>;
    using C = typename Store<TS>::C;
    constexpr int V = F::V, L = F::L, H = F::H, NW = F::NW, CH = F::ch, CC = F::CC;
    const int N = a.N, S = 1 << N, n = a.n, x0 = t.x * CC, cols = S >> n;
    const size_t plane = (size_t)a.nq << (2 * N);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    TS *t0 = reinterpret_cast<TS *>(lds), *t1 = t0 + F::t1_at;
    float *r2 = reinterpret_cast<float *>(lds + F::r2_off);
    float *r1 = reinterpret_cast<float *>(lds + F::r1_off);
    const float4 *wl = reinterpret_cast<const float4 *>(lds + F::w_off);
    auto t0_col = [&](int i) { return t0 + F::slot(i) * 2 * L; };
    auto t1_col = [&](int i) { return t1 + (i - 1) * 3 * L; };
    auto r2_col = [&](int i) { return r2 + (i - 1) * 4 * CH * L; };
    auto r1_col = [&](int i) { return r1 + (i - 1) * 2 * CH * L; };
    // A wave's items at the levels with two cones: one row part h and cone k, and
    // every DX-th column from xw; the unrolled loops then address by immediates and a
    // column's parity is the wave's (22.3 -> 20.9 us a pair, 21.2 with next).
    constexpr int DX = NW / (2 * H), IX = (F::c1 + DX - 1) / DX;
    static_assert(NW % (2 * H) == 0, "waves");
    const int h = wave % H, k = wave / H & 1, xw = 1 + wave / (2 * H);
    const Rows<V> w((h * 64 + lane) * V, t.y0, sb, S);
    // T_{n+1}: directions 0, 1 and direction 2 of every column
#pragma unroll
    for (int it = 0; it < IX; ++it) {
        const int X = xw + DX * it;
        if (X > F::c1) break;
        const int far = (int)(t0_col(2 * X + 1) - t0_col(2 * X));
        C ev[V], od[V];
        fused_up<TS, V, L, true, IN>(t0_col(2 * X) + k * L + w.r, far, k, w, w.y(2 * X - 1) + sb, ev, od,
                                     k == 0 ? L : 0);
        TS *d = t1_col(X) + 2 * k * L + w.r;
        st_row<V>(d, ev);
        if (k == 0) st_row<V>(d + L, od);
    }
    __syncthreads();
    if constexpr (F::overlay) {
        rl.store(r2, wave, lane);
        __syncthreads();
    }
    // R_{n+1}
    const float4 wt1 = wl[1 + k];
#pragma unroll
    for (int it = 0; it < IX; ++it) {
        const int x = xw + DX * it;
        if (x > F::c1 || (x0 >> 1) + x >= (cols >> 1)) break;  // beyond the grid: read by no one
        const int y = w.y(2 * x - 1);
        const float4 wt = wt1;
        const int c = (x + 1) >> 1;
        float o[CH][V];
        if (x & 1) {
            fused_down_odd<TS, V, L, IN>(t1_col(x) + k * L + w.r, r2_col(c) + (2 * CH * L + 2) * k + w.r,
                                         (x0 >> 2) + c < (cols >> 2), k, wt, w, y + 2 * sb, o);
        } else {
            const int cc = x >> 1;
            C ed[2][V], none[V];
#pragma unroll
            for (int up = 0; up < 2; ++up) {
                fused_up<TS, V, L, false, IN>(t1_col(2 * cc) + (k + up) * L + w.r, 3 * L, k + up, w,
                                              y + 2 * sb, ed[up], none, 0);
#pragma unroll
                for (int j = 0; j < V; ++j) ed[up][j] = stored(ed[up][j], static_cast<const TS *>(nullptr));
            }
            const float *rn = r2_col(cc) + 2 * CH * L * k + w.r;
            fused_down_even<TS, V, L, IN>(ed, rn, rn + 4 * CH * L + 4 * k,
                                          (x0 >> 2) + cc + 1 < (cols >> 2), k, wt, w, y + 4 * sb, o);
        }
        float *dst = r1_col(x) + k * CH * L + w.r;
#pragma unroll
        for (int c2 = 0; c2 < CH; ++c2) st_f<V>(dst + c2 * L, o[c2]);
        if (a.R[1] && x <= CC / 2 && w.r < own) {
            float *out = a.R[1] + (((unsigned)t.q << (2 * N)) +
                                   ((unsigned)((((x0 >> 1) + x) << (n + 1)) | (2 * t.ii + k)) << N));
#pragma unroll
            for (int c2 = 0; c2 < CH; ++c2) st_f<V>(out + c2 * plane + (unsigned)y, o[c2]);
        }
    }
    __syncthreads();
    // R_n
    const float4 wt0 = wl[0];
    // (not unrolled: its stores then came in one burst at the end, 25 us more a
    // pair at 4096^2)
#pragma unroll 1
    for (int it = 0; it < (CC * H + NW - 1) / NW; ++it) {
        const int x = 1 + wave / H + NW / H * it;
        if (x > CC || x0 + x >= cols) break;
        const int y = w.y(x - 1);
        const float4 wt = wt0;
        const int c = (x + 1) >> 1;
        float o[CH][V];
        if (x & 1) {
            fused_down_odd<TS, V, L, IN>(t0_col(x) + w.r, r1_col(c) + w.r, (x0 >> 1) + c < (cols >> 1),
                                         0, wt, w, y + sb, o);
        } else {
            const int cc = x >> 1;
            C ed[2][V];
#pragma unroll
            for (int up = 0; up < 2; ++up) ld_row<V>(t1_col(cc) + 2 * up * L + w.r, ed[up]);
            const float *rn = r1_col(cc) + w.r;
            fused_down_even<TS, V, L, IN>(ed, rn, rn + 2 * CH * L, (x0 >> 1) + cc + 1 < (cols >> 1), 0,
                                          wt, w, y + 2 * sb, o);
        }
        if (w.r < own) {
            float *out = a.R[0] + (((unsigned)t.q << (2 * N)) +
                                   ((unsigned)(((x0 + x) << n) | t.ii) << N));
#pragma unroll
            for (int c2 = 0; c2 < CH; ++c2) st_f<V>(out + c2 * plane + (unsigned)y, o[c2]);
        }
    }
}

template <typename TS>
__device__ __forceinline__ void fuse_down_block(const FuseArgs &a, char *lds, int tid) {
    using F = FuseDown<TS>;
    constexpr int V = F::V, L = F::L, CC = F::CC;
    const int N = a.N, S = 1 << N, n = a.n;
    const FuseTile t = fuse_tile(a);
    const int x0 = t.x * CC;
    const int sb = 2 * t.ii - (1 << n);
    const int own = a.win < S - t.y0 ? a.win : S - t.y0;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    TS *t0 = reinterpret_cast<TS *>(lds);
    float4 *wl = reinterpret_cast<float4 *>(lds + F::w_off);
    TnLoad<TS, V, L, F::NT, F::c0> ld;
    ld.load(reinterpret_cast<const TS *>(a.T[0]) + (unsigned)t.q * a.te[0], N, n, t.ii, x0 + 1, t.y0, sb,
            wave, lane);
    R2Load<TS> rl;
    rl.load(a, t, sb, wave, lane);
    const float4 wt = load_weight<2>(
        n, t.ii, a.env ? a.env + (size_t)(a.q0 + t.q) * kConeTable : nullptr, tid);
    ld.store(t0, wave, lane, [](int i) { return F::slot(i + 1); });
    if constexpr (!F::overlay) rl.store(reinterpret_cast<float *>(lds + F::r2_off), wave, lane);
    if (tid < 3) wl[tid] = wt;
    __syncthreads();
    if (window_inside(t.y0, CC + 3, sb, S)) fuse_down_levels<TS, true>(a, t, lds, rl, own, sb, tid);
    else fuse_down_levels<TS, false>(a, t, lds, rl, own, sb, tid);
}

// ---- adjoint of the merge down, two levels: (T_n, dR_n) -> dR_{n+1}, dR_{n+2}, n >= 2 ----

// A block takes one cone ii of level n and the columns x0 .. x0 + CC - 1 (as seen
// from below): it writes dR_{n+1} at CC/2 columns from x0/2 and dR_{n+2} at CC/4
// from x0/4.  In gather form these read back along the lower edge: dR_n and
// T_n's transmittances from column x0 - 6 on, and two columns of dR_{n+1} more
// than the block writes.  The transmittances of T_{n+1} and T_{n+2} are rebuilt.
// Lookups run down the window, at most 4 + 8 rows, so the first 12 rows of a
// window hold no valid results.  1024^2: 21 to 26 us a pair (24 on average), 90-93 MB
// from and to HBM (the levels hold 67-71; 13 columns of dR_n are loaded for 8), for
// 34 us of two single levels; vector and scalar issue (20 and 24 thousand
// instructions a CU) and the loads' latency share the time (512 threads: 24).
// Without the second store of a repeated row a 1024^2 forward and reverse takes 604
// us for 600, in RGB 1530 for 1544.
template <typename TS> struct FuseDr {
    static constexpr int L = kWindow, V = 2, ch = Store<TS>::ch;
    static constexpr int NT = ch == 3 ? 512 : 256, NW = NT / 64;
    static constexpr int CC = 8, win = L - 12, skip = 12;
    static constexpr int d0_cols = CC + 5, t0_cols = CC + 4, t1_cols = 4, d1_cols = CC / 2 + 2;
    static constexpr int pad = 16;  // floats before the first row
    static constexpr int d0_off = pad, t0_off = d0_off + d0_cols * ch * L, t1_off = t0_off + t0_cols * 2 * L;
    static constexpr int d1_off = t1_off + t1_cols * 3 * L;
    static constexpr int lds = (d1_off + d1_cols * 2 * ch * L) * 4;
};

__device__ __forceinline__ float stored_t(float v, const float2 *) { return v; }
__device__ __forceinline__ float stored_t(float v, const float4 *) { return v; }
__device__ __forceinline__ float stored_t(float v, const half2_t *) { return (float)to_half(v); }
__device__ __forceinline__ float stored_t(float v, const half4_t *) { return (float)to_half(v); }
__device__ __forceinline__ float raw_t(float2 v) { return v.y; }
__device__ __forceinline__ float raw_t(float4 v) { return v.w; }
__device__ __forceinline__ float raw_t(half2_t v) { return (float)v.y; }
__device__ __forceinline__ float raw_t(half4_t v) { return (float)v.w; }

// One entry of dR_{m} (cone jj = 2 i + up, relative) of column c for V rows, from
// LDS rows of the level below: own, the co-located probe's cone i; g, the odd
// column's, at its shift; g2, the column before's, at twice that; t, t2 the
// transmittances of Eq. 14 and of the doubled edge, as the level-by-level body
// combines them.
template <int V>
__device__ __forceinline__ void fused_dr(const float (&own)[V], const float (&g)[V], const float (&t)[V],
                                         bool in, const float (&g2)[V], const float (&t2)[V], bool in2,
                                         float (&o)[V]) {
#pragma unroll
    for (int j = 0; j < V; ++j) {
        o[j] = 0.5f * own[j];
        o[j] = fmaf(in ? g[j] : 0.f, in ? t[j] : 0.f, o[j]);
        o[j] = fmaf(0.5f * (in2 ? g2[j] : 0.f), in2 ? t2[j] : 0.f, o[j]);
    }
}

template <typename TS>
__device__ __forceinline__ void fuse_dr_block(const FuseArgs &a, char *lds, int tid) {
    using F = FuseDr<TS>;
    constexpr int V = F::V, L = F::L, NW = F::NW, CH = F::ch, CC = F::CC;
    const int N = a.N, S = 1 << N, n = a.n;
    const FuseTile t = fuse_tile(a);
    const int x0 = t.x * CC, cols = S >> n, sb = 2 * t.ii - (1 << n);
    const int own = F::skip + (a.win < S - t.y0 ? a.win : S - t.y0);
    const size_t plane = (size_t)4 << (2 * N);
    const unsigned q0 = (unsigned)t.q << (2 * N);
    const int ii = t.ii;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), lane = tid & 63;
    float *l = reinterpret_cast<float *>(lds);
    float *d0 = l + F::d0_off, *t0 = l + F::t0_off, *t1 = l + F::t1_off, *d1 = l + F::d1_off;
    // window rows from 12 before the first stored one
    const Rows<V> w(lane * V, t.y0 - F::skip, sb, S);
    const TS *none = nullptr;
    // dR_n and T_n's transmittances (directions ii, ii + 1), columns x0 - 6 on; all
    // loads first
    {
        constexpr int DR = F::d0_cols * CH, DI = (DR + NW - 1) / NW;
        constexpr int TR = F::t0_cols * 2, TI = (TR + NW - 1) / NW;
        typename RawVec<8>::type dv[DI];
        typename RawVec<sizeof(TS) * V == 32 ? 16 : sizeof(TS) * V>::type tv[TI][sizeof(TS) * V == 32 ? 2 : 1];
        const float *D = a.R[0] + ((unsigned)t.q << (2 * N));
        const TS *T = reinterpret_cast<const TS *>(a.T[0]) + (unsigned)t.q * a.te[0];
#pragma unroll
        for (int it = 0; it < DI; ++it) {
            int i = it * NW + wave;
            i = i < DR ? i : DR - 1;
            const int p = i / CH, c = i % CH;
            int x = x0 - 6 + p;
            x = x < 0 ? 0 : x < cols ? x : cols - 1;
            dv[it] = *reinterpret_cast<const typename RawVec<8>::type *>(
                D + c * plane + (((unsigned)((x << n) | t.ii) << N) + (unsigned)w.y(p)));
        }
#pragma unroll
        for (int it = 0; it < TI; ++it) {
            int i = it * NW + wave;
            i = i < TR ? i : TR - 1;
            const int p = i >> 1, d = i & 1;
            int x = x0 - 6 + p;
            x = x < 0 ? 0 : x < cols ? x : cols - 1;
            using R = std::remove_reference_t<decltype(tv[0][0])>;
            const R *src = reinterpret_cast<const R *>(
                T + (((unsigned)(x * ((1 << n) + 1) + t.ii + d) << N) + (unsigned)w.y(p)));
            tv[it][0] = src[0];
            if constexpr (sizeof(TS) * V == 32) tv[it][1] = src[1];
        }
#pragma unroll
        for (int it = 0; it < DI; ++it) {
            const int i = it * NW + wave;
            if ((it + 1) * NW > DR) {
                pin_raw(dv[it]);
                if (i >= DR) break;
            }
            *reinterpret_cast<typename RawVec<8>::type *>(d0 + i * L + w.r) = dv[it];
        }
#pragma unroll
        for (int it = 0; it < TI; ++it) {
            const int i = it * NW + wave;
            if ((it + 1) * NW > TR) {
                pin_raw(tv[it][0]);
                if constexpr (sizeof(TS) * V == 32) pin_raw(tv[it][1]);
                if (i >= TR) break;
            }
            TS e[V];
            __builtin_memcpy(e, tv[it], sizeof(e));
            *reinterpret_cast<float2 *>(t0 + i * L + w.r) = make_float2(raw_t(e[0]), raw_t(e[1]));
        }
    }
    __syncthreads();
    auto d0_row = [&](int p, int c) { return d0 + (p * CH + c) * L + w.r; };
    auto t0_row = [&](int p, int d) { return t0 + (p * 2 + d) * L + w.r; };
    auto t1_row = [&](int i, int d) { return t1 + (i * 3 + d) * L + w.r; };
    auto d1_row = [&](int i, int u, int c) { return d1 + ((i * 2 + u) * CH + c) * L + w.r; };
    // T_{n+1}'s transmittances at the columns x0/2 - 2 .. x0/2 + 1 (positions 2, 4,
    // 6, 8 from x0 - 6), as the merge up builds them
    for (int i = wave; i < F::t1_cols; i += NW) {
        const int p = 2 + 2 * i, y = w.y(p) + sb;
        float n0[V], n1[V], f00[V], f02[V], f10[V], f12[V];
        ld_f<V>(t0_row(p, 0), n0);
        ld_f<V>(t0_row(p, 1), n1);
        ld_f<V>(t0_row(p + 1, 0), f00);
        ld_f<V>(t0_row(p + 1, 0) + 2, f02);
        ld_f<V>(t0_row(p + 1, 1), f10);
        ld_f<V>(t0_row(p + 1, 1) + 2, f12);
        const bool in0 = w.in(y), in1 = w.in(y + 2);
        float e0[V], e1[V], e2[V];
#pragma unroll
        for (int j = 0; j < V; ++j) {
            e0[j] = stored_t(n0[j] * (in0 ? f00[j] : 1.f), none);
            e1[j] = stored_t(0.5f * (n1[j] * (in1 ? f02[j] : 1.f) + n0[j] * (in0 ? f10[j] : 1.f)), none);
            e2[j] = stored_t(n1[j] * (in1 ? f12[j] : 1.f), none);
        }
        st_f<V>(t1_row(i, 0), e0);
        st_f<V>(t1_row(i, 1), e1);
        st_f<V>(t1_row(i, 2), e2);
    }
    // dR_{n+1} at the columns x0/2 - 2 .. x0/2 + CC/2 - 1
    for (int i = wave; i < F::d1_cols * 2; i += NW) {
        const int ci = i >> 1, up = i & 1, c = (x0 >> 1) - 2 + ci, p = 2 * ci + 2;  // column 2c
        if (c < 0) continue;
        const int y = w.y(p);
        const int sh = 2 * up, yg = y - sb - sh, yg2 = y - 2 * (sb + sh);
        const bool in = c >= 1 && w.in(yg), in2 = c > 1 && w.in(yg2);
        float t[V], tn[V], t2[V];
        ld_f<V>(t0_row(p - 1, up) - sh, t);
        ld_f<V>(t0_row(p - 2, up) - 2 * sh, tn);
#pragma unroll
        for (int j = 0; j < V; ++j) t2[j] = stored_t(tn[j] * (w.in(yg) ? t[j] : 1.f), none);
#pragma unroll
        for (int c2 = 0; c2 < CH; ++c2) {
            float f0[V], g[V], g2[V], o[V];
            ld_f<V>(d0_row(p, c2), f0);
            ld_f<V>(d0_row(p - 1, c2) - sh, g);
            ld_f<V>(d0_row(p - 2, c2) - 2 * sh, g2);
            fused_dr<V>(f0, g, t, in, g2, t2, in2, o);
            st_f<V>(d1_row(ci, up, c2), o);
            if (ci >= 2 && w.r >= F::skip && w.r < own)
                st_f<V>(a.R[1] + c2 * plane + (q0 + ((unsigned)((c << (n + 1)) | (2 * ii + up)) << N) + (unsigned)y), o);
        }
    }
    __syncthreads();
    // dR_{n+2} at the columns x0/4 .. x0/4 + CC/4 - 1
    for (int i = wave; i < CC; i += NW) {
        const int Ci = i >> 2, k = i & 3, C = (x0 >> 2) + Ci, ci = 2 * Ci + 2;  // column 2C of level n+1
        const int e = (k >> 1) + (k & 1), sh = 2 * e;
        const int y = w.y(4 * Ci + 6), yg = y - 2 * sb - sh, yg2 = y - 2 * (2 * sb + sh);
        const bool in = C >= 1 && w.in(yg), in2 = C > 1 && w.in(yg2);
        float t[V], tn[V], t2[V];
        ld_f<V>(t1_row(ci - 1, e) - sh, t);
        ld_f<V>(t1_row(ci - 2, e) - 2 * sh, tn);
#pragma unroll
        for (int j = 0; j < V; ++j) t2[j] = stored_t(tn[j] * (w.in(yg) ? t[j] : 1.f), none);
#pragma unroll
        for (int c2 = 0; c2 < CH; ++c2) {
            float f0[V], g[V], g2[V], o[V];
            ld_f<V>(d1_row(ci, k >> 1, c2), f0);
            ld_f<V>(d1_row(ci - 1, k >> 1, c2) - sh, g);
            ld_f<V>(d1_row(ci - 2, k >> 1, c2) - 2 * sh, g2);
            fused_dr<V>(f0, g, t, in, g2, t2, in2, o);
            if (w.r >= F::skip && w.r < own)
                st_f<V>(a.R[2] + c2 * plane + (q0 + ((unsigned)((C << (n + 2)) | (4 * ii + k)) << N) + (unsigned)y), o);
        }
    }
}
