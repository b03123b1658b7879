// fs_colred_meet and fs_colred_left of fs_device.h on the host: a thread for every lane, a barrier for every workgroup.  Under
// ThreadSanitizer an access to the workgroup's flag that no barrier orders is reported.  `meet.inc` is their text.
#include <pthread.h>

#include <cstdint>
#include <cstdio>
#include <thread>
#include <vector>

typedef uint32_t fs_u32;
#define FS_DEV static inline
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
#define __HIP_MEMORY_SCOPE_AGENT 0
#define __HIP_MEMORY_SCOPE_WORKGROUP 0
#define __hip_atomic_fetch_add(p, v, order, scope) __atomic_fetch_add(p, v, order)
#define __hip_atomic_exchange(p, v, order, scope) __atomic_exchange_n(p, v, order)
#define __hip_atomic_load(p, order, scope) __atomic_load_n(p, order)
#define __hip_atomic_store(p, v, order, scope) __atomic_store_n(p, v, order)
typedef float* __amdgpu_buffer_rsrc_t;
static float* fs_make_rsrc(float* p, fs_u32) { return p; }
template <int FV> static void fs_store_dev(const float (&src)[FV], float* p, fs_u32 bytes) {
  for (int f = 0; f < FV; ++f) p[bytes / 4 + f] = src[f];
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
  fs_u32 flag = 0;
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
        met[k] = fs_colred_meet<1, 32, WG, 1>(vals, part, counters, &flag, (fs_u32)idx, N, ticks);
        folds[k] = 0;
        for (int all = 0; all < met[k] && (all == 0 || fs_colred_left(&flag)); ++all) ++folds[k];  // as the generated kernels do
      });
  }
  // 0 left, 1 its slices, 2 all slices as well; -1 where its lanes disagree
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
    wrong += folds != (saw == 2 && gone > 0 ? 2 : 1);
  }
  for (fs_u32 c : counters) wrong += c != 0;
  return wrong + (lasts != 1);
}

int main() {
  const int wrong = scenario(0) + scenario(3) + scenario(N - 1) + scenario(16);
  return printf("%d wrong\n", wrong), wrong != 0;
}
