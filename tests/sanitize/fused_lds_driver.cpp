// Sanitizer driver for the LDS and buffer accesses of the kernels that run
// several merge levels at once (test infrastructure).  It includes the device
// header itself as host C++ (the few helpers the kernel file gives it are
// restated below; no address depends on a value) and runs blocks on the CPU.
//
//   bounds (AddressSanitizer): the threads of a block one after the other, every
//   tile, with the LDS array and every global buffer allocated at its exact size:
//   any access past one of them is reported.
//   races (ThreadSanitizer): every thread of a block as a thread of its own, the
//   block's barriers as barriers: any two accesses of the same bytes between two
//   barriers, one of them a write, are reported, also where the value read is used
//   by nothing.
#include <pthread.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <type_traits>
#include <vector>

#include "../../paper_2505_02041_amd/csrc/hrc_internal.h"

#ifndef __device__
#define __device__
#endif
#ifndef __forceinline__
#define __forceinline__ inline
#endif
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __all(x) (x)
#define __clz(x) __builtin_clz((unsigned)(x))

static thread_local struct { unsigned x; } blockIdx;
static pthread_barrier_t *barrier = nullptr;  // NULL: threads run one after the other
static void __syncthreads() {
    if (barrier) pthread_barrier_wait(barrier);
}

namespace hrc {

static float c_cone[kConeTable];

typedef _Float16 half2_t __attribute__((ext_vector_type(2)));
typedef _Float16 half4_t __attribute__((ext_vector_type(4)));
typedef _Float16 half8_t __attribute__((ext_vector_type(8)));

static float2 merge(float2 n, float2 f) { return make_float2(fmaf(n.y, f.x, n.x), n.y * f.y); }
static float4 merge(float4 n, float4 f) {
    return make_float4(fmaf(n.w, f.x, n.x), fmaf(n.w, f.y, n.y), fmaf(n.w, f.z, n.z), n.w * f.w);
}
template <typename I> I empty_interval();
template <> float2 empty_interval<float2>() { return make_float2(0.f, 1.f); }
template <> float4 empty_interval<float4>() { return make_float4(0.f, 0.f, 0.f, 1.f); }
static float2 lo(float4 v) { return make_float2(v.x, v.y); }
static float2 hi(float4 v) { return make_float2(v.z, v.w); }
static float4 pair(float2 a, float2 b) { return make_float4(a.x, a.y, b.x, b.y); }
static _Float16 to_half(float v) { return (_Float16)v; }
static void pin(float &) {}
static void pin(float2 &) {}
static void pin(float4 &) {}
template <typename Raw> void pin_raw(Raw &) {}
static float4 ld_pair(const half2_t *p) {
    const half4_t v = *reinterpret_cast<const half4_t *>(p);
    return make_float4((float)v.x, (float)v.y, (float)v.z, (float)v.w);
}
static void st_pair(float2 *p, float4 v) { *reinterpret_cast<float4 *>(p) = v; }
static void st_pair(half2_t *p, float4 v) {
    half4_t h = {to_half(v.x), to_half(v.y), to_half(v.z), to_half(v.w)};
    *reinterpret_cast<half4_t *>(p) = h;
}
static void st_iv(half2_t *p, float2 v) { *p = half2_t{to_half(v.x), to_half(v.y)}; }
static void st_iv(half4_t *p, float4 v) {
    *p = half4_t{to_half(v.x), to_half(v.y), to_half(v.z), to_half(v.w)};
}
static float4 ld4(const half4_t *p) {
    const half4_t v = *p;
    return make_float4((float)v.x, (float)v.y, (float)v.z, (float)v.w);
}
static void cvt_quad(half8_t v, float4 &a, float4 &b) {
    a = make_float4((float)v[0], (float)v[1], (float)v[2], (float)v[3]);
    b = make_float4((float)v[4], (float)v[5], (float)v[6], (float)v[7]);
}
static void st_quad(half2_t *p, float4 a, float4 b) {
    half8_t h = {to_half(a.x), to_half(a.y), to_half(a.z), to_half(a.w),
                 to_half(b.x), to_half(b.y), to_half(b.z), to_half(b.w)};
    *reinterpret_cast<half8_t *>(p) = h;
}
static void st_quad(float2 *, float4, float4) {}

#include "../../paper_2505_02041_amd/csrc/hrc_fused.h"

}  // namespace hrc

using namespace hrc;

enum class Kind { up, top, down, dr };
static const char *kind_name[] = {"up", "top", "down", "dr"};
static int blocks_run = 0;

// One block: `body` for each of its threads.
template <typename Body> static void run_block(unsigned tile, int threads, int lds_bytes, Body body) {
    // (16-byte aligned, its last byte the allocation's last)
    char *lds = static_cast<char *>(std::aligned_alloc(16, (size_t)lds_bytes));
    std::memset(lds, 0, (size_t)lds_bytes);
    ++blocks_run;
#ifdef RACES
    pthread_barrier_t b;
    pthread_barrier_init(&b, nullptr, (unsigned)threads);
    barrier = &b;
    struct Arg {
        unsigned tile;
        int tid;
        char *lds;
        Body *body;
    };
    std::vector<Arg> args((size_t)threads);
    std::vector<pthread_t> th((size_t)threads);
    pthread_attr_t at;
    pthread_attr_init(&at);
    pthread_attr_setstacksize(&at, 256 << 10);
    for (int t = 0; t < threads; ++t) {
        args[t] = Arg{tile, t, lds, &body};
        if (pthread_create(&th[t], &at, [](void *p) -> void * {
                Arg *a = static_cast<Arg *>(p);
                blockIdx.x = a->tile;
                (*a->body)(a->lds, a->tid);
                return nullptr;
            }, &args[t])) {
            std::fprintf(stderr, "FAIL pthread_create\n");
            std::exit(1);
        }
    }
    for (auto &t : th) pthread_join(t, nullptr);
    pthread_attr_destroy(&at);
    pthread_barrier_destroy(&b);
    barrier = nullptr;
#else
    blockIdx.x = tile;
    for (int t = 0; t < threads; ++t) {
        const int lane = t & 63;  // the wave's first and last lanes, and two between
        if (lane == 0 || lane == 1 || lane == 32 || lane == 63) body(lds, t);
    }
#endif
    std::free(lds);
}

// The tiles of one phase of level n of a 2^N grid, `store`: every level stored.
template <typename TS, typename F, typename Body>
static void run_kernel(Kind kind, int N, int n, int levels, bool store, int chunk_log2, Body body) {
    constexpr int ch = Store<TS>::ch;
    FuseArgs a{};
    const int S = 1 << N;
    a.N = N;
    a.n = n;
    a.levels = levels;
    a.nq = kind == Kind::dr ? 4 : 1;
    a.q0 = kind == Kind::dr ? 0 : 1;
    a.half = std::is_same<TS, half2_t>::value || std::is_same<TS, half4_t>::value;
    a.rgb = ch == 3;
    // the window and the chunks as the planner sets them
    a.nwin = (S + F::win - 1) / F::win;
    a.win = (S / 2 + a.nwin - 1) / a.nwin * 2;
    a.inv_nwin = a.nwin == 1 ? 0u : (unsigned)((0x100000000ull + a.nwin - 1) / (unsigned)a.nwin);
    a.lchunks = chunk_log2;
    for (int j = 0; j < 5; ++j) a.te[j] = n + j <= N ? (unsigned)t_level_entries(N, n + j) : 0;
    const unsigned tiles = (unsigned)a.nq * (((unsigned)a.nwin << n) << a.lchunks);
    a.eighth = tiles % 8 == 0 ? (int)(tiles / 8) : 0;
    std::vector<void *> held;
    auto buffer = [&](size_t bytes) {
        void *p = std::aligned_alloc(16, (bytes + 15) & ~size_t(15));
        std::memset(p, 0, bytes);
        held.push_back(p);
        return p;
    };
    auto t_level = [&](int j) { return buffer(a.nq * t_level_entries(N, n + j) * sizeof(TS)); };
    auto r_level = [&] { return static_cast<float *>(buffer((size_t)ch * a.nq * S * S * 4)); };
    std::vector<float> env((size_t)kQuadrants * kConeTable, 0.f);
    a.T[0] = t_level(0);
    if (kind == Kind::up) {
        for (int j = 1; j <= levels; ++j)
            if (store || j == levels) a.T[j] = t_level(j);
    } else if (kind == Kind::top) {
        for (int j = 1; store && j < levels; ++j) a.T[j] = t_level(j);
        for (int j = 0; j < levels; ++j)
            if (store || j == 0) a.R[j] = r_level();
        a.env = store ? env.data() : nullptr;
    } else if (kind == Kind::down) {
        a.R[0] = r_level();
        a.R[1] = store ? r_level() : nullptr;
        a.R[2] = r_level();
        a.env = store ? env.data() : nullptr;
    } else {
        for (int j = 0; j < 3; ++j) a.R[j] = r_level();
    }
    std::printf("%s interval %d bytes, N %d n %d levels %d store %d: %u tiles, LDS %d bytes\n",
                kind_name[(int)kind], (int)sizeof(TS) + (ch == 3 && sizeof(TS) == 8 ? 100 : 0), N, n,
                levels, (int)store, tiles, (int)F::lds);
    std::fflush(stdout);
    auto one = [&](unsigned t) {
        run_block(t, F::NT, F::lds, [&](char *lds, int tid) { body(a, lds, tid); });
    };
#ifdef RACES
    one(tiles / 2);
#else
    for (unsigned t = 0; t < tiles; ++t) one(t);
#endif
    for (void *p : held) std::free(p);
}

template <typename TS, int G> static void test_up(int N, int n, bool store) {
    run_kernel<TS, FuseUp<TS, G>>(Kind::up, N, n, G, store, N - n - G, [](const FuseArgs &a, char *l, int t) {
        fuse_up_block<TS, G>(a, l, t);
    });
}
template <typename TS, int M> static void test_top(int N, bool store) {
    run_kernel<TS, FuseTop<TS, M>>(Kind::top, N, N - M, M, store, 0, [](const FuseArgs &a, char *l, int t) {
        fuse_top_block<TS, M>(a, l, t);
    });
}
template <typename TS> static void test_down(int N, int n, bool store) {
    run_kernel<TS, FuseDown<TS>>(Kind::down, N, n, 2, store, N - n - (sizeof(TS) == 16 ? 2 : 3),
                                 [](const FuseArgs &a, char *l, int t) { fuse_down_block<TS>(a, l, t); });
}
template <typename TS> static void test_dr(int N, int n) {
    run_kernel<TS, FuseDr<TS>>(Kind::dr, N, n, 2, true, N - n - 3,
                               [](const FuseArgs &a, char *l, int t) { fuse_dr_block<TS>(a, l, t); });
}

template <typename TS> static void test_type() {
    constexpr bool one = Store<TS>::ch == 1;
#ifdef RACES
    const bool stores[] = {true};
#else
    const bool stores[] = {false, true};
#endif
    for (bool store : stores) {
        test_up<TS, 2>(8, 2, store);
        test_up<TS, 3>(8, 2, store);
        test_top<TS, 2>(4, store);
        test_top<TS, 3>(7, store);
        test_down<TS>(7, 2, store);
        if constexpr (one) {
            test_up<TS, 4>(8, 2, store);
            test_top<TS, 4>(8, store);
        }
#ifndef RACES
        test_top<TS, 3>(5, store);
        if constexpr (one) test_top<TS, 4>(6, store);
        test_up<TS, 2>(9, 5, store);
        test_down<TS>(6, 2, store);
        test_down<TS>(8, 3, store);
#endif
    }
    test_dr<TS>(7, 2);
#ifndef RACES
    test_dr<TS>(5, 2);
    test_dr<TS>(8, 4);
#endif
}

int main() {
    test_type<float2>();
    test_type<half2_t>();
    test_type<float4>();
    test_type<half4_t>();
    std::printf("fused kernels: %d blocks run\n", blocks_run);
    return 0;
}
