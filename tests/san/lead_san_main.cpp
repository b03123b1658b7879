// The pieces of whole cache lines of fs_device.h (fs_lead_...) on the host, lane after lane, on tensors of exact size: what a row's lanes load,
// reduce and store against the row itself, with as many vectors a lane as the schedule gives it (lead_vectors).  lead.inc is their text.
#include <cstdint>
#include <cstdio>
#include <cstring>
#include <vector>

#define FS_DEV inline
typedef uint16_t fs_u16;
typedef uint8_t fs_u8;
template <int DT> struct fs_elem;
template <> struct fs_elem<0> { typedef float type; };
template <> struct fs_elem<1> { typedef fs_u16 type; };
template <> struct fs_elem<2> { typedef fs_u8 type; };
template <typename T, int N> struct fs_vec {
  struct type {
    T x[N];
    T& operator[](int k) { return x[k]; }
    const T& operator[](int k) const { return x[k]; }
  };
};
template <int DT> float fs_to_f32(typename fs_elem<DT>::type v) { return (float)v; }
template <int DT> typename fs_elem<DT>::type fs_from_f32(float v) { return (typename fs_elem<DT>::type)v; }
static const char* wrong = nullptr;
template <int DT, int V, bool NT, bool UA = false> typename fs_vec<typename fs_elem<DT>::type, V>::type fs_load_raw(const void* base, long i) {
  typename fs_vec<typename fs_elem<DT>::type, V>::type v;
  for (int k = 0; k < V; ++k) v[k] = static_cast<const typename fs_elem<DT>::type*>(base)[i + k];
  return v;
}
template <int DT, int V, bool NT> void fs_store_vec(const float* src, void* base, long i) {
  if (i % V) wrong = "a store that is not aligned";
  for (int k = 0; k < V; ++k) static_cast<typename fs_elem<DT>::type*>(base)[i + k] = fs_from_f32<DT>(src[k]);
}
template <int KIND> float fs_red_identity() { return KIND == 0 ? 0.0f : -1e30f; }
template <int KIND> float fs_red_op(float a, float b) { return KIND == 0 ? a + b : a > b ? a : b; }
#include "lead.inc"

static int cases = 0;
template <int DT, int DT_OUT, int V, int L, int C, int LEAD> void one(int R) {
  typedef typename fs_elem<DT>::type T;
  typedef typename fs_elem<DT_OUT>::type TO;
  constexpr int NVL = (lead_vectors(C, V, LEAD) + L - 1) / L;
  std::vector<T> x((size_t)R * C);
  std::vector<TO> y((size_t)R * C), seen((size_t)R * C, 0);
  for (size_t i = 0; i < x.size(); ++i) x[i] = (T)(1 + i * 7 % 97);
  for (int row = 0; row < R; ++row) {
    const long row0 = (long)row * C;
    const int lead = (int)(row0 & (LEAD - 1));
    float sum = 0.0f, most = -1e30f, want = 0.0f, want_most = 0.0f;
    for (int c = 0; c < C; ++c) want += (float)x[row0 + c], want_most = want_most > (float)x[row0 + c] ? want_most : (float)x[row0 + c];
    for (int lir = 0; lir < L; ++lir) {
      for (int j = 0; j < NVL; ++j) {  // (those that are asked for ahead: whole vectors at aligned places)
        if ((j + 1) * L * V > C) continue;
        if ((row0 - lead + (j * L + lir) * V) % V || fs_lead_at<V, L, C>(lead, lir, row == R - 1, j) != (j * L + lir) * V) wrong = "a vector inside the row is moved";
      }
      float v[NVL * V];
      fs_lead_load_row<DT, V, NVL, L, C, false>(v, x.data(), row0, lead, lir, row == R - 1);
      sum += fs_lead_lane_reduce<0, V, NVL, L, C, LEAD>(v, lead, lir);
      const float m = fs_lead_lane_reduce<1, V, NVL, L, C, LEAD>(v, lead, lir);
      most = most > m ? most : m;
      fs_lead_store_row<DT_OUT, V, NVL, L, C, LEAD, false>(v, y.data(), row0, lead, lir, true);
      fs_lead_store_row<DT_OUT, V, NVL, L, C, LEAD, false>(v, seen.data(), row0, lead, lir, false);
    }
    if (sum != want || most != want_most) wrong = "a reduction";
  }
  for (size_t i = 0; i < x.size(); ++i)
    if ((float)y[i] != (float)x[i] || seen[i]) wrong = "a stored element";
  ++cases;
  if (wrong) std::printf("C %d R %d V %d L %d: %s\n", C, R, V, L, wrong), wrong = nullptr;
}
template <int C> void widths() {
  for (int R : {1, 2, 3, 33}) {
    one<0, 0, 4, 8, C, 32>(R);
    one<0, 0, 4, 64, C, 32>(R);
    one<0, 0, 2, 16, C, 32>(R);
    one<1, 1, 8, 16, C, 64>(R);
    one<1, 1, 2, 64, C, 64>(R);
    one<1, 0, 4, 32, C, 64>(R);
    one<2, 0, 4, 16, C, 128>(R);
  }
}

int main() {
  widths<256>(), widths<257>(), widths<258>(), widths<259>(), widths<260>(), widths<264>(), widths<287>(), widths<288>(), widths<289>(), widths<320>(), widths<321>();
  widths<385>(), widths<511>(), widths<513>(), widths<577>(), widths<600>(), widths<639>(), widths<1001>(), widths<1023>(), widths<1025>();
  std::printf("%d cases\n", cases);
}
