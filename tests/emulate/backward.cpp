// Runs the backward kernels on the CPU, workgroup by workgroup, with every tensor between pages that
// may not be touched: a read or write out of range ends the program and is named.  Transfers into
// LDS land at once, so this shows wrong addresses, wrong indexes and wrong results, not missing waits.
//
//   backward <f16|bf16> <threshold of dropped bytes> <heads> <grid> <slab rows> <edge: 0|1> <values> <lengths> [<keys attended>]
//
// (edge 1: tensors end at a forbidden page, 0: they begin behind one; lengths and key counts separated by
// commas; values "normal", or "last": every row attends to its sequence's last key alone, with scores' gradients of
// the size that values of 64 give).  Prints the largest relative errors of the one pass against the two
// passes (dq dk dv), its errors against sums in double (without dropout), and what is not finite.
#include <hip/hip_runtime.h>

#include "translated/bwd_fused_kernel.h"

#include <signal.h>
#include <stdio.h>
#include <stdlib.h>
#include <sys/mman.h>
#include <unistd.h>

#include <functional>
#include <map>
#include <random>
#include <string>
#include <vector>

using namespace fmha;

namespace emu {

constexpr int kLanes = 64, kMaxThreads = 512;
constexpr size_t kStack = 512 << 10, kLds = 160 << 10;

struct Fiber {
  void* sp;
  char* stack;
  Index tid;
  enum { kReady, kMeeting, kDone } state;
  Meeting what;
  int imm;
  void* site;
  unsigned char in[64], out[64];
};
Fiber fibers[kMaxThreads], *current;
void* scheduler;
std::function<void()> kernel;
Index block, grid;
unsigned char* lds;
const void* kernarg;

extern "C" void emu_switch(void** save, void* to);
asm(".text\n.globl emu_switch\nemu_switch:\n"
    "push %rbp\npush %rbx\npush %r12\npush %r13\npush %r14\npush %r15\nmov %rsp,(%rdi)\n"
    "mov %rsi,%rsp\npop %r15\npop %r14\npop %r13\npop %r12\npop %rbx\npop %rbp\nret\n");

Index& thread() { return current->tid; }
unsigned char* in() { return current->in; }
unsigned char* out() { return current->out; }

__attribute__((noinline)) void meet(Meeting what, int imm) {
  current->what = what;
  current->imm = imm;
  current->site = __builtin_return_address(0);
  current->state = Fiber::kMeeting;
  emu_switch(&current->sp, scheduler);
}
void start() {
  kernel();
  current->state = Fiber::kDone;
  emu_switch(&current->sp, scheduler);
}

struct Tensor {
  char *begin, *end;
  const char* name;
};
std::vector<Tensor> tensors;

void out_of_range(const char* what, const void* at) {
  fprintf(stderr, "out of range: %s %p, workgroup %u, thread %u\n", what, at, block.x, current ? current->tid.x : 0u);
  for (auto& t : tensors) fprintf(stderr, "  %-6s %p .. %p\n", t.name, (void*)t.begin, (void*)t.end);
  _exit(3);
}
void dma(const void* from, uint32_t to, int bytes) {
  bool inside = false;
  for (auto& t : tensors) inside |= (char*)from >= t.begin && (char*)from + bytes <= t.end;
  if (!inside) out_of_range("source of a transfer", from);
  const uint32_t at = to + bytes * (current->tid.x % kLanes) - (uint32_t)(uintptr_t)lds;
  if (at + bytes > kLds) out_of_range("LDS transfer", (void*)(uintptr_t)at);
  memcpy(lds + at, from, bytes);
}

template <typename V>
float element(const unsigned char* p, int i) {
  V v;
  memcpy(&v, p + 2 * i, 2);
  return (float)v;
}
// N x N x K product: a lane holds 8 contraction slots of a row of A and of a column of B, and N * N / 64 results
template <typename V, int N, int K>
void product(Fiber* w) {
  static float a[N][K], b[K][N];
  for (int l = 0; l < kLanes; l++)
    for (int e = 0; e < 8; e++) {
      a[l % N][8 * (l / N) + e] = element<V>(w[l].in, e);
      b[8 * (l / N) + e][l % N] = element<V>(w[l].in + 16, e);
    }
  for (int l = 0; l < kLanes; l++) {
    constexpr int n = N * N / kLanes;
    float d[n];
    for (int r = 0; r < n; r++) {
      const int row = N == 32 ? 8 * (r / 4) + 4 * (l / N) + r % 4 : 4 * (l / N) + r;
      d[r] = 0.f;
      for (int k = 0; k < K; k++) d[r] += a[row][k] * b[k][l % N];
    }
    memcpy(w[l].out, d, sizeof d);
  }
}
void perform(const std::vector<Fiber*>& g) {
  Fiber* w = g[0];
  for (Fiber* f : g)
    if (w->what != kFirstLane && (g.size() != kLanes || f->what != w->what || f->imm != w->imm)) {
      fprintf(stderr, "%zu lanes at a meeting of all (%d, %d)\n", g.size(), w->what, f->what);
      _exit(3);
    }
  switch (w->what) {
    case kFirstLane:
      for (Fiber* f : g) memcpy(f->out, w->in, 4);
      break;
    case kDpp:  // permutations within four, mirrored in eight, mirrored in sixteen
      for (int i = 0; i < kLanes; i++) {
        const int c = w->imm, from = c < 0x100 ? (i & ~3) | ((c >> (2 * (i & 3))) & 3) : c == 0x141 ? i ^ 7 : i ^ 15;
        memcpy(w[i].out, w[from].in, 4);
      }
      break;
    case kSwapHalves:
      for (int i = 0; i < kLanes; i++) {
        memcpy(w[i].out, w[i & 31].in, 4);
        memcpy(w[i].out + 4, w[i | 32].in, 4);
      }
      break;
    case kReadTr16:
      for (int i = 0; i < kLanes; i++)
        for (int e = 0; e < 4; e++) {
          uint64_t p;
          memcpy(&p, w[(i & ~15) + 4 * e + (i & 15) / 4].in, 8);
          memcpy(w[i].out + 2 * e, (char*)p + 2 * (i & 3), 2);
        }
      break;
    case kMfma32F16: product<_Float16, 32, 16>(w); break;
    case kMfma32Bf16: product<__bf16, 32, 16>(w); break;
    case kMfma16F16: product<_Float16, 16, 32>(w); break;
    case kMfma16Bf16: product<__bf16, 16, 32>(w); break;
    default: break;
  }
  for (Fiber* f : g) f->state = Fiber::kReady;
}
void run_workgroup(int threads) {
  for (int t = 0; t < threads; t++) {
    Fiber& f = fibers[t];
    if (!f.stack) f.stack = (char*)mmap(nullptr, kStack, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
    void** sp = (void**)(f.stack + kStack - 64);
    *--sp = nullptr;
    *--sp = (void*)start;
    for (int i = 0; i < 6; i++) *--sp = nullptr;
    f.sp = sp;
    f.tid.x = t;
    f.state = Fiber::kReady;
  }
  while (true) {
    for (int w = 0; w < threads; w += kLanes)
      while (true) {
        for (int i = w; i < w + kLanes; i++)
          if (fibers[i].state == Fiber::kReady) {
            current = &fibers[i];
            emu_switch(&scheduler, current->sp);
          }
        // The fewest lanes of one place at a time, and reads of a first lane ahead of what all lanes meet for: that
        // is a branch of their own, or a copy that the compiler made of code behind a branch.
        std::map<void*, std::vector<Fiber*>> places;
        std::vector<Fiber*> all;
        for (int i = w; i < w + kLanes; i++)
          if (fibers[i].state == Fiber::kMeeting && fibers[i].what != kWorkgroup) {
            if (fibers[i].what == kFirstLane) places[fibers[i].site].push_back(&fibers[i]);
            all.push_back(&fibers[i]);
          }
        if (all.empty()) break;
        for (auto& p : places)
          if (p.second.size() < all.size() || all[0]->what != kFirstLane) all = p.second;
        perform(all);
      }
    int waiting = 0;
    for (int t = 0; t < threads; t++) waiting += fibers[t].state == Fiber::kMeeting;
    if (waiting == 0) return;
    if (waiting != threads) {
      fprintf(stderr, "a barrier of %d threads out of %d\n", waiting, threads);
      _exit(3);
    }
    for (int t = 0; t < threads; t++) fibers[t].state = Fiber::kReady;
  }
}

int edge;
template <typename T>
T* tensor(size_t n, const char* name) {
  const size_t bytes = n * sizeof(T), pages = (bytes + 4095) / 4096 * 4096;
  char* p = (char*)mmap(nullptr, pages + 8192, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS, -1, 0);
  mprotect(p + 4096, pages, PROT_READ | PROT_WRITE);
  char* begin = p + 4096 + (edge ? pages - bytes : 0);
  tensors.push_back({begin, begin + bytes, name});
  return (T*)begin;
}
void fault(int, siginfo_t* info, void*) { out_of_range("access", info->si_addr); }

}  // namespace emu

static std::vector<int> numbers(const char* s) {
  std::vector<int> r;
  for (char* end; *s; s = *end ? end + 1 : end) r.push_back((int)strtol(s, &end, 10));
  return r;
}

template <typename T>
static void run(uint32_t thr, int heads, int grid, int slab_rows, bool last, const std::vector<int>& lens, const std::vector<int>& used) {
  using emu::tensor;
  const int batch = (int)lens.size();
  std::vector<int> first(1, 0), keys;
  for (int i = 0; i < batch; i++) {
    first.push_back(first[i] + lens[i]);
    keys.push_back(used.empty() ? lens[i] : std::min(std::max(used[i], 0), lens[i]));
  }
  const int total = first[batch];
  const size_t n = (size_t)total * heads * kHeadDim, rows = (size_t)total * heads;
  T *q = tensor<T>(n, "q"), *k = tensor<T>(n, "k"), *v = tensor<T>(n, "v"), *o = tensor<T>(n, "o"), *g = tensor<T>(n, "d_o");
  T* grad[3] = {tensor<T>(n, "dq"), tensor<T>(n, "dk"), tensor<T>(n, "dv")};
  float *lse = tensor<float>(rows, "lse"), *dsum = tensor<float>(rows + 1, "dsum"), *lse2 = tensor<float>(rows + 1, "lse2");
  int32_t* count = tensor<int32_t>(64, "count");
  uint32_t* feed = tensor<uint32_t>(kFeedWords, "feed");
  memset(feed, 0, sizeof(uint32_t) * kFeedWords);

  std::mt19937 rng(lens[0] + 7 * batch);
  std::normal_distribution<float> normal;
  for (int i = 0; i < batch; i++)
    for (int t = first[i]; t < first[i + 1]; t++)
      for (int x = 0; x < heads * kHeadDim; x++) {
        const size_t at = (size_t)t * heads * kHeadDim + x;
        const bool is_last = t - first[i] == keys[i] - 1;
        q[at] = (T)(last ? 2.f : normal(rng));
        k[at] = (T)(last ? (is_last ? 4.f : 0.f) : normal(rng));
        v[at] = (T)(last ? 64.f : normal(rng));
        g[at] = (T)(last ? 64.f : normal(rng));
      }

  BwdArgs a;
  memset(&a, 0, sizeof a);
  a.pb.n_tiles = count;
  a.pb.heads = heads;
  a.pb.total_tokens = total;
  a.pb.scale = 0.125f;
  a.drop = DropArgs{thr, 7u, 1u, 256.f / (256 - thr)};
  a.feed = FeedArgs{feed, 1};

  // O and the log-sum-exp (the mask is the kernels' own, drawn for 32 x 32 scores at a time as they draw it),
  // and the gradients in double
  std::vector<double> ref[3];
  for (auto& r : ref) r.assign(n, 0.);
  for (int i = 0; i < batch; i++)
    for (int h = 0; h < heads; h++) {
      auto at = [&](int t) { return ((size_t)(first[i] + t) * heads + h) * kHeadDim; };
      std::vector<double> p(keys[i]);
      for (int x = 0; x < lens[i]; x++) {
        double top = -1e300, sum = 0, d = 0, out[kHeadDim] = {};
        for (int y = 0; y < keys[i]; y++) {
          p[y] = 0;
          for (int c = 0; c < kHeadDim; c++) p[y] += (double)q[at(x) + c] * (double)k[at(y) + c];
          top = std::max(top, p[y] *= 0.125);
        }
        for (int y = 0; y < keys[i]; y++) sum += p[y] = exp(p[y] - top);
        lse[(size_t)h * total + first[i] + x] = keys[i] ? (float)(top + log(sum)) : -INFINITY;
        for (int y = 0; y < keys[i]; y++) {
          p[y] /= sum;
          bool kept = true;
          if (thr) {
            const u32x4 w = philox4x32_10(y >> 2, x >> 2, first[i], h, a.drop.k0, a.drop.k1);
            const int word = ((x & 3) - (y >> 3)) & 3, byte = ((y & 3) - (x >> 3)) & 3;
            kept = ((w[word] >> (8 * byte)) & 255) >= thr;
          }
          for (int c = 0; c < kHeadDim; c++) out[c] += kept ? p[y] * a.drop.rp * (double)v[at(y) + c] : 0.;
        }
        for (int c = 0; c < kHeadDim; c++) {
          o[at(x) + c] = (T)(float)out[c];
          d += out[c] * (double)g[at(x) + c];
        }
        for (int y = 0; y < keys[i] && !thr; y++) {
          double dp = 0;
          for (int c = 0; c < kHeadDim; c++) dp += (double)g[at(x) + c] * (double)v[at(y) + c];
          const double ds = 0.125 * p[y] * (dp - d);
          for (int c = 0; c < kHeadDim; c++) {
            ref[0][at(x) + c] += ds * (double)k[at(y) + c];
            ref[1][at(y) + c] += ds * (double)q[at(x) + c];
            ref[2][at(y) + c] += p[y] * (double)g[at(x) + c];
          }
        }
      }
    }

  // the lists, as schedule.h leaves them
  std::vector<TileItem> seqs, tiles;
  for (int i = 0; i < batch; i++)
    if (lens[i] > 0) seqs.push_back(TileItem{first[i], lens[i], keys[i], 0});
  auto bucket = [](const TileItem& s) { return std::max(127 - (s.nk + 7) / 8, 0); };
  std::stable_sort(seqs.begin(), seqs.end(), [&](const TileItem& x, const TileItem& y) { return bucket(x) < bucket(y); });
  for (const TileItem& s : seqs) {
    count[used.empty() ? (bucket(s) < 127 - 16 ? 1 : bucket(s) < 127 - 8 ? 2 : 3) : 1]++;
    for (int r = 0; r < s.len; r += kTileRows) tiles.push_back(TileItem{s.r0, s.len, s.nk, r});
  }
  count[0] = (int)tiles.size();
  TileItem *list = tensor<TileItem>(tiles.size(), "tiles"), *whole = tensor<TileItem>(seqs.size(), "seqs");
  std::copy(tiles.begin(), tiles.end(), list);
  std::copy(seqs.begin(), seqs.end(), whole);
  auto bits = [](T* p) { return reinterpret_cast<uint16_t*>(p); };
  a.pb.tiles = list;
  a.seqs = whole;
  a.slab = tensor<float>((size_t)grid * slab_rows * kHeadDim, "slab");
  a.slab_rows = slab_rows;
  a.q = bits(q), a.k = bits(k), a.v = bits(v), a.o = bits(o), a.d_o = bits(g);
  a.dq = bits(grad[0]), a.dk = bits(grad[1]), a.dv = bits(grad[2]);
  a.lse = lse, a.dsum = dsum, a.lse2 = lse2;
  a.q_stride = a.k_stride = a.v_stride = a.o_stride = a.do_stride = a.dq_stride = a.dk_stride = a.dv_stride = heads * kHeadDim;
  emu::kernarg = &a;
  emu::grid.x = grid;
  auto launch = [&](int threads, std::function<void()> f) {
    emu::kernel = f;
    for (int b = 0; b < grid; b++) {
      emu::block.x = b;
      memset(emu::lds, 0xff, emu::kLds);  // (NaN)
      emu::run_workgroup(threads);
    }
  };
  auto results = [&]() {
    std::vector<float> r[3];
    for (int x = 0; x < 3; x++)
      for (size_t i = 0; i < n; i++) {
        r[x].push_back((float)grad[x][i]);
        grad[x][i] = (T)NAN;
      }
    return std::vector<std::vector<float>>(r, r + 3);
  };
  results();
  launch(kFusedThreads, [&] { thr ? bwd_fused_kernel<T, true>(a) : bwd_fused_kernel<T, false>(a); });
  const auto one = results();
  for (size_t i = 0; i < rows + 1; i++) dsum[i] = lse2[i] = NAN;
  launch(kThreads, [&] { thr ? bwd_dq_kernel<T, true>(a) : bwd_dq_kernel<T, false>(a); });
  launch(kThreads, [&] { thr ? bwd_dkv_kernel<T, true>(a) : bwd_dkv_kernel<T, false>(a); });
  const auto two = results();

  double claimed = 0;
  for (int i = 0; i < kFeedWords; i++) claimed += feed[i];
  printf("counters %g\n", claimed);
  for (int x = 0; x < 3; x++) {
    double diff = 0, off = 0, norm = 0, norm_ref = 0, largest = 0;
    size_t bad_one = 0, bad_two = 0;
    for (size_t i = 0; i < n; i++) {
      bad_one += !isfinite(one[x][i]);
      bad_two += !isfinite(two[x][i]);
      diff += pow((double)one[x][i] - two[x][i], 2);
      off += pow(one[x][i] - ref[x][i], 2);
      norm += pow((double)two[x][i], 2);
      norm_ref += pow(ref[x][i], 2);
      largest = std::max(largest, fabs((double)one[x][i]));
    }
    printf("%s two_passes %g double %g not_finite %zu %zu largest %g\n", x == 0 ? "dq" : x == 1 ? "dk" : "dv",
           sqrt(diff / std::max(norm, 1e-30)), thr ? 0. : sqrt(off / std::max(norm_ref, 1e-30)), bad_one, bad_two, largest);
  }
}

int main(int argc, char** argv) {
  if (argc < 9) return 2;
  char* low = (char*)mmap(nullptr, emu::kLds + 1024, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_32BIT, -1, 0);
  emu::lds = (unsigned char*)(((uintptr_t)low + 1023) & ~(uintptr_t)1023);
  static char other_stack[65536];
  stack_t ss = {other_stack, 0, sizeof other_stack};
  sigaltstack(&ss, nullptr);
  struct sigaction sa = {};
  sa.sa_sigaction = emu::fault;
  sa.sa_flags = SA_SIGINFO | SA_ONSTACK;
  sigaction(SIGSEGV, &sa, nullptr);
  emu::edge = atoi(argv[6]);
  const uint32_t thr = (uint32_t)atoi(argv[2]);
  const std::vector<int> lens = numbers(argv[8]), used = argc > 9 ? numbers(argv[9]) : std::vector<int>();
  auto go = std::string(argv[1]) == "f16" ? run<_Float16> : run<__bf16>;
  go(thr, atoi(argv[3]), atoi(argv[4]), atoi(argv[5]), std::string(argv[7]) == "last", lens, used);
  return 0;
}
