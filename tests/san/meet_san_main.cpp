// fs_colred_meet and fs_colred_left, fs_tile_put and fs_tile_meet of fs_device.h on the host: a thread for every lane, a barrier for
// every workgroup.  Under ThreadSanitizer an access to the workgroup's flag that no barrier orders is reported.  meet.inc is their text.
#include <pthread.h>

#include <cstdint>
#include <cstdio>
#include <thread>
#include <vector>

typedef uint32_t fs_u32;
#define FS_DEV inline
struct Lane {
  int x;
};
static thread_local Lane threadIdx;
static thread_local pthread_barrier_t* barrier;
static void __syncthreads() { pthread_barrier_wait(barrier); }
static unsigned long long ticks_now() {  // (a clock that every read moves on)
  static unsigned long long t = 0;
  return __atomic_fetch_add(&t, 1ull, __ATOMIC_RELAXED);
}
#define __builtin_amdgcn_s_memrealtime() ticks_now()
#define __builtin_amdgcn_s_sleep(n) std::this_thread::yield()
#define __builtin_amdgcn_s_waitcnt(n) ((void)0)
#define __builtin_amdgcn_readfirstlane(x) (x)
#define __hip_atomic_fetch_or(p, v, order, scope) __atomic_fetch_or(p, v, order)
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, order)
#define __hip_atomic_exchange(p, v, order, scope) __atomic_exchange_n(p, v, order)
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, order)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, order)
typedef float* __amdgpu_buffer_rsrc_t;
static float* fs_make_rsrc(float* p, fs_u32) { return p; }
template <int FV> static void fs_store_dev(const float (&src)[FV], float* p, fs_u32 bytes) {
  for (int f = 0; f < FV; ++f) __atomic_store(&p[bytes / 4 + f], const_cast<float*>(&src[f]), __ATOMIC_RELAXED);  // (two may put the same partial)
}
template <int K, int C, int WG, int FV> struct fs_colfold {
  static constexpr int CH = C / FV, NCH = K * CH, CPT = (NCH + WG - 1) / WG;
};
#include "meet.inc"

constexpr int WG = 16, N = 18;  // (lanes; two groups of counted workgroups)
static float part[N * 32];
static fs_u32 counters[32 * 3 + N];

struct Workgroup {
  pthread_barrier_t bar;
  fs_u32 flag[9] = {};
  int met[WG], folds[WG], ticks;
  std::vector<std::thread> lanes;
  void start(int idx, int t) {
    ticks = t;
    pthread_barrier_init(&bar, nullptr, WG);
    for (int k = 0; k < WG; ++k)
      lanes.emplace_back([this, idx, k] {
        threadIdx.x = k;
        barrier = &bar;
        float vals[2][1] = {{1.0f}, {2.0f}};
        met[k] = fs_colred_meet<1, 32, WG, 1>(vals, part, counters, flag, (fs_u32)idx, N, ticks);
        folds[k] = met[k] != 0;  // (its own slices; as the generated kernels do)
        if (met[k] == 2 && fs_colred_left(flag)) ++folds[k];
      });
  }
  // 0 left, 1 its slices, 2 those of workgroups that have left as well; -1 where its lanes disagree
  int end(int* saw) {
    for (std::thread& t : lanes) t.join();
    pthread_barrier_destroy(&bar);
    for (int k = 1; k < WG; ++k)
      if (met[k] != met[0] || folds[k] != folds[0]) return -1;
    *saw = met[0];
    return folds[0];
  }
};

// the first `gone` workgroups leave at once, the others wait
static int scenario(int gone) {
  int wrong = 0, lasts = 0, saw = 0;
  for (int w = 0; w < gone; ++w) {
    Workgroup g;
    g.start(w, 0);
    wrong += g.end(&saw) != 0 || saw != 0;
  }
  std::vector<Workgroup> rest(N - gone);
  for (int w = gone; w < N; ++w) rest[(size_t)(w - gone)].start(w, 1 << 30);
  for (Workgroup& g : rest) {
    const int folds = g.end(&saw);
    lasts += saw == 2;
    if (saw == 2 && gone > 0)
      for (int w = 0; w < N; ++w) wrong += (g.flag[1 + w / 32] >> (w & 31) & 1) != (w < gone);
    wrong += folds != (saw == 2 && gone > 0 ? 2 : 1);
  }
  for (fs_u32 c : counters) wrong += c != 0;
  return wrong + (lasts != 1);
}

// M workgroups of a tile in two stages: the first `early` of them start, the others when those are done.  Every partial comes from its
// own workgroup or one that waits, and all are there when a workgroup goes on.
template <int M> struct Tile {
  static constexpr int LANES = 4, W = (M + 31) / 32;
  fs_u32 counters[2] = {0, 0}, bits[4 * W] = {};
  float part[2][M * LANES];
  long taken[2] = {0, 0};
  int wrong = 0, wrong_sums = 0;
  struct Group {
    pthread_barrier_t bar;
    fs_u32 flag = 0;
    std::vector<std::thread> lanes;
  };
  std::vector<Group> groups{M};
  void start(int idx, int ticks) {
    Group& g = groups[(size_t)idx];
    pthread_barrier_init(&g.bar, nullptr, LANES);
    for (int k = 0; k < LANES; ++k)
      g.lanes.emplace_back([this, &g, idx, k, ticks] {
        threadIdx.x = k;
        barrier = &g.bar;
        int wait = ticks;
        for (int st = 0; st < 2; ++st) {
          auto put = [&](int b) {
            const float vals[1][1] = {{(float)(1 + st * 1000 + b * LANES + k)}};
            fs_tile_put<1, LANES, LANES, 1>(vals, part[st], b);
          };
          put(idx);
          int next = fs_tile_meet<M>(counters + st, bits + st * 2 * W, &g.flag, idx, wait);
          while (next >= 0) {
            if (k == 0) __atomic_fetch_add(&taken[st], 1l, __ATOMIC_RELAXED);
            wait = 0;
            put(next);
            next = fs_tile_next<M>(counters + st, bits + st * 2 * W, &g.flag, next);
          }
          for (int i = 0; i < M * LANES; ++i) {
            float x;
            __atomic_load(&part[st][i], &x, __ATOMIC_RELAXED);
            if (x != (float)(1 + st * 1000 + i)) __atomic_fetch_add(&wrong, 1, __ATOMIC_RELAXED), __atomic_fetch_add(&wrong_sums, 1, __ATOMIC_RELAXED);
          }
        }
      });
  }
  // the words hold what they like (a workspace that was never cleared): no more than an end of every wait is asked for
  int run_on(fs_u32 rubbish) {
    for (fs_u32* p : {counters, bits})
      for (int i = 0; i < (p == counters ? 2 : 4 * W); ++i) p[i] = rubbish;
    for (int w = 0; w < M; ++w) start(w, 50);
    for (Group& g : groups)
      for (std::thread& t : g.lanes) t.join();
    return 0;
  }
  int run(int early, int ticks) {
    for (float* p : {part[0], part[1]})
      for (int i = 0; i < M * LANES; ++i) p[i] = 0.0f;
    for (int w = 0; w < early; ++w) start(w, ticks);
    if (early < M)
      for (int w = 0; w < early; ++w)
        for (std::thread& t : groups[(size_t)w].lanes) t.join();
    for (int w = early; w < M; ++w) start(w, ticks);
    for (int w = early < M ? early : 0; w < M; ++w)
      for (std::thread& t : groups[(size_t)w].lanes) t.join();
    for (int st = 0; st < 2; ++st) {  // all have counted themselves; a partial that was claimed (those of late workgroups at least) was claimed once
      long claimed = 0;
      for (int w = 0; w < W; ++w) claimed += __builtin_popcount(bits[(st * 2 + 1) * W + w]);
      wrong += (counters[st] & ~kTileLate) != M || taken[st] != claimed || taken[st] < M - early || (early == M && ticks > 1000 && (taken[st] != 0 || counters[st] != M));
    }
    return wrong;
  }
};
template <int M> static int tile(int early, int ticks) { return Tile<M>().run(early, ticks); }
template <int M> static int claimed_by_nobody(int early) {  // the late ones' partials are marked as claimed: the early ones do them in the end
  Tile<M> t;
  for (int st = 0; st < 2; ++st)
    for (int w = 0; w < t.W; ++w) t.bits[(st * 2 + 1) * t.W + w] = ~0u;
  t.run(early, 50);
  return t.wrong_sums;
}

int main() {
  int wrong = scenario(0) + scenario(3) + scenario(N - 1) + scenario(16);
  wrong += tile<2>(2, 1 << 30) + tile<2>(1, 50) + tile<8>(8, 1 << 30) + tile<8>(3, 50) + tile<8>(1, 0) + tile<8>(8, 0) + tile<64>(64, 1 << 30) + tile<64>(40, 50) + tile<70>(70, 1 << 30) +
           tile<70>(20, 0) + tile<70>(66, 50) + claimed_by_nobody<8>(5) + claimed_by_nobody<40>(30) + Tile<8>().run_on(3) + Tile<8>().run_on(8) + Tile<40>().run_on(0x7f7f7f7fu) +
           Tile<40>().run_on(~0u);
  return printf("%d wrong\n", wrong), wrong != 0;
}
