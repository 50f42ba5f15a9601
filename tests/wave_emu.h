// Runs a generated kernel on the CPU, for tests: every thread of a block is a fibre, and what crosses lanes (shuffles, ballots,
// lane permutes, matrix instructions, wave barriers, __syncthreads) is a point where the fibres of a wave or of a block
// meet.  Between two such points the lanes run one after the other, so an exchange through LDS without one shows up as a
// wrong result.  Buffers come from emu_alloc(): they end at a page that cannot be accessed (emu_reserve(): address space
// only), so an access behind their end is reported by emu_run() instead of going unseen.
//
// Where lanes of a wave wait at different places, those at the lowest source line go first (a loop's lanes before the code
// behind it).  Blocks run one after the other.
#include <csetjmp>
#include <csignal>
#include <cmath>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <sys/mman.h>
#include <ucontext.h>
#include <vector>

#define __global__
#define __device__
#define __forceinline__ inline
#define __restrict__ __restrict
#define __shared__ static
#define __launch_bounds__(...)
#define __noinline__ __attribute__((noinline))

struct emu_dim3 { unsigned x, y, z; };

namespace emu {
constexpr size_t STACK = 256 * 1024;
union Word {                                          // what a lane hands over
    uint64_t u[4];
    double d[4];
};
struct Lane {
    jmp_buf here;
    ucontext_t ctx;
    char *stack;
    int state;                                        // 0 not started, 1 ready, 2 at a meeting of the wave, 3 at a block barrier, 4 done
    int line;
    emu_dim3 tid;
    Word in;
};
struct Wave {
    std::vector<Lane> lane;
    Word got[64];                                     // handed over by the lanes that met last
    unsigned long long met;
};
static std::vector<Wave> *block;
static Lane *cur;
static Wave *cur_wave;
static jmp_buf sched;
static emu_dim3 block_idx, grid_dim, block_dim;
static void (*kernel)(const void *);
static const void *kernel_args;
static bool last_first;
static sigjmp_buf fault;
static void *fault_at;
static char fault_text[256];

inline void yield()
{
    if (!_setjmp(cur->here))
        _longjmp(sched, 1);
}
inline void fail(const char *what, int line)
{
    std::snprintf(fault_text, sizeof fault_text, "%s (line %d)", what, line);
    siglongjmp(fault, 2);
}
inline const Wave &meet(int line, Word w)
{
    cur->in = w;
    cur->line = line;
    cur->state = 2;
    yield();
    return *cur_wave;
}
inline int lane_id() { return (int)(cur->tid.x & 63); }
inline Word word(uint64_t a, uint64_t b = 0, uint64_t c = 0)
{
    Word w = {};
    w.u[0] = a, w.u[1] = b, w.u[2] = c;
    return w;
}
inline void entry()
{
    kernel(kernel_args);
    cur->state = 4;
    _longjmp(sched, 1);
}
inline void resume(Wave &w, Lane &l)
{
    cur = &l;
    cur_wave = &w;
    if (_setjmp(sched))
        return;
    if (l.state == 0) {
        l.state = 1;
        setcontext(&l.ctx);
    }
    l.state = 1;
    _longjmp(l.here, 1);
}
inline void on_segv(int, siginfo_t *si, void *)
{
    fault_at = si->si_addr;
    siglongjmp(fault, 1);
}
inline void run_block()
{
    for (;;) {
        bool any = false, moved = false;
        for (Wave &w : *block) {
            unsigned long long go = 0;
            int line = INT32_MAX;
            for (int l = 0; l < 64; ++l) {            // those that can run at once, or else those at the first meeting
                Lane &x = w.lane[l];
                any |= x.state != 4;
                if (x.state <= 1)
                    line = -1;
                else if (x.state == 2 && x.line < line)
                    line = x.line;
            }
            if (line == INT32_MAX)
                continue;
            for (int l = 0; l < 64; ++l)
                if (line == -1 ? w.lane[l].state <= 1 : (w.lane[l].state == 2 && w.lane[l].line == line))
                    go |= 1ull << l;
            if (line != -1) {
                w.met = go;
                for (int l = 0; l < 64; ++l)
                    w.got[l] = (go >> l & 1) ? w.lane[l].in : Word{};
            }
            moved = true;
            for (int l = 0; l < 64; ++l) {
                const int i = last_first ? 63 - l : l;
                if (go >> i & 1)
                    resume(w, w.lane[i]);
            }
        }
        if (!any)
            return;
        if (moved)
            continue;
        for (Wave &w : *block)                        // everybody waits at the block barrier
            for (Lane &l : w.lane)
                if (l.state == 3)
                    l.state = 1;
    }
}
}  // namespace emu

#define threadIdx (emu::cur->tid)
#define blockIdx (emu::block_idx)
#define gridDim (emu::grid_dim)
#define blockDim (emu::block_dim)

template <typename T>
inline T emu_from(int line, T v, int src)             // v of lane src of the wave
{
    emu::Word w = {};
    std::memcpy(&w, &v, sizeof v);
    const emu::Word got = emu::meet(line, w).got[src & 63];
    std::memcpy(&v, &got, sizeof v);
    return v;
}
template <typename T>
inline T emu_shfl_up(int line, T v, int d, int width)
{
    const int l = emu::lane_id(), src = (l & (width - 1)) < d ? l : l - d;
    return emu_from(line, v, src);
}
inline int emu_first(int line, int v)
{
    const emu::Wave &w = emu::meet(line, emu::word((unsigned)v));
    return (int)w.got[__builtin_ctzll(w.met)].u[0];
}
inline unsigned long long emu_ballot(int line, bool p)
{
    const emu::Wave &w = emu::meet(line, emu::word(p));
    unsigned long long r = 0;
    for (int l = 0; l < 64; ++l)
        r |= (unsigned long long)w.got[l].u[0] << l;
    return r;
}
inline int emu_dpp(int line, int old, int src, int ctrl, int rowmask, bool bound0)
{
    const emu::Wave &w = emu::meet(line, emu::word((unsigned)src));
    const int l = emu::lane_id(), row = l & ~15, k = l & 15;
    int from = -1;
    if (ctrl < 0x100)
        from = (l & ~3) | (ctrl >> (2 * (l & 3)) & 3);
    else if (ctrl > 0x110 && ctrl < 0x120)
        from = k - (ctrl & 15) >= 0 ? l - (ctrl & 15) : -1;
    else if (ctrl > 0x120 && ctrl < 0x130)
        from = row + ((k - (ctrl & 15)) & 15);
    else if (ctrl == 0x140)
        from = row + 15 - k;
    else if (ctrl == 0x141)
        from = (l & ~7) + 7 - (l & 7);
    else if (ctrl == 0x142)
        from = row >= 16 ? row - 1 : -1;
    else if (ctrl == 0x143)
        from = l >= 32 ? 31 : -1;
    else
        emu::fail("lane permute that is not modelled", line);
    if (!(rowmask >> (l >> 4) & 1))
        return old;
    return from < 0 ? (bound0 ? 0 : old) : (int)w.got[from].u[0];
}
struct emu_pair {
    unsigned v[2];
    unsigned operator[](int i) const { return v[i]; }
};
inline emu_pair emu_swap(int line, unsigned a, unsigned b, int rowlen)      // odd rows of a with even rows of b
{
    const emu::Wave &w = emu::meet(line, emu::word(a, b));
    const int l = emu::lane_id();
    const bool odd = l / rowlen & 1;
    return odd ? emu_pair{{(unsigned)w.got[l - rowlen].u[1], b}} : emu_pair{{a, (unsigned)w.got[l + rowlen].u[0]}};
}
inline double emu_mfma4(int line, double a, double b, double c)
{
    emu::Word x = {};
    x.d[0] = a, x.d[1] = b;
    const emu::Wave &w = emu::meet(line, x);
    const int l = emu::lane_id(), j = l & 3, blk = l >> 2 & 3, i = l >> 4;
    for (int k = 0; k < 4; ++k)
        c = std::fma(w.got[i + 4 * blk + 16 * k].d[0], w.got[j + 4 * blk + 16 * k].d[1], c);
    return c;
}
typedef double emu_d4 __attribute__((ext_vector_type(4)));
inline emu_d4 emu_mfma16(int line, double a, double b, emu_d4 c)
{
    emu::Word x = {};
    x.d[0] = a, x.d[1] = b;
    const emu::Wave &w = emu::meet(line, x);
    const int l = emu::lane_id(), j = l & 15;
    for (int r = 0; r < 4; ++r)
        for (int k = 0; k < 4; ++k)
            c[r] = std::fma(w.got[(l >> 4) + 4 * r + 16 * k].d[0], w.got[j + 16 * k].d[1], c[r]);
    return c;
}
struct emu_rsrc {
    const char *p;
    unsigned n;
};
typedef unsigned emu_u4 __attribute__((ext_vector_type(4)));
typedef unsigned emu_u2 __attribute__((ext_vector_type(2)));
template <typename T>
inline T emu_buffer_load(emu_rsrc r, unsigned vo, unsigned so)          // words past the end read 0
{
    unsigned t[sizeof(T) / 4];
    for (unsigned i = 0; i < sizeof(T) / 4; ++i) {
        t[i] = 0;
        if ((uint64_t)vo + so + 4 * i + 4 <= r.n)
            std::memcpy(&t[i], r.p + so + vo + 4 * i, 4);
    }
    T v;
    std::memcpy(&v, t, sizeof v);
    return v;
}
inline int __double2loint(double x) { uint64_t u; std::memcpy(&u, &x, 8); return (int)(u & 0xffffffffu); }
inline int __double2hiint(double x) { uint64_t u; std::memcpy(&u, &x, 8); return (int)(u >> 32); }
inline double __hiloint2double(int hi, int lo)
{
    const uint64_t u = (uint64_t)(unsigned)hi << 32 | (unsigned)lo;
    double x;
    std::memcpy(&x, &u, 8);
    return x;
}
inline int __popcll(unsigned long long x) { return __builtin_popcountll(x); }
inline unsigned __umul24(unsigned a, unsigned b) { return (a & 0xffffffu) * (b & 0xffffffu); }
template <typename T> inline T min(T a, T b) { return b < a ? b : a; }
template <typename T> inline T max(T a, T b) { return a < b ? b : a; }
template <typename T> inline void unsafeAtomicAdd(T *p, T v) { *p += v; }
template <typename T> inline T atomicAdd(T *p, T v) { const T o = *p; *p = o + v; return o; }
using std::fma;

#define __syncthreads() (emu::cur->state = 3, emu::yield())
#define __shfl(v, src, ...) emu_from(__LINE__, v, (src) + (emu_width(__VA_ARGS__) < 64 ? (emu::lane_id() & ~(emu_width(__VA_ARGS__) - 1)) : 0))
#define __shfl_up(v, d, ...) emu_shfl_up(__LINE__, v, d, emu_width(__VA_ARGS__))
#define __shfl_xor(v, m, ...) emu_from(__LINE__, v, emu::lane_id() ^ (m))
#define __ballot(p) emu_ballot(__LINE__, p)
#define __builtin_amdgcn_readlane(v, l) emu_from(__LINE__, (int)(v), l)
#define __builtin_amdgcn_readfirstlane(v) emu_first(__LINE__, (int)(v))
#define __builtin_amdgcn_update_dpp(old, src, ctrl, rm, bm, bc) emu_dpp(__LINE__, old, src, ctrl, rm, bc)
#define __builtin_amdgcn_permlane32_swap(a, b, x, y) emu_swap(__LINE__, a, b, 32)
#define __builtin_amdgcn_permlane16_swap(a, b, x, y) emu_swap(__LINE__, a, b, 16)
#define __builtin_amdgcn_mfma_f64_4x4x4f64(a, b, c, x, y, z) emu_mfma4(__LINE__, a, b, c)
#define __builtin_amdgcn_mfma_f64_16x16x4f64(a, b, c, x, y, z) emu_mfma16(__LINE__, a, b, c)
#define __builtin_amdgcn_wave_barrier() (void)emu::meet(__LINE__, emu::word(0))
#define __builtin_amdgcn_s_waitcnt(x) (void)0
#define __builtin_amdgcn_s_setprio(x) (void)0
#define __builtin_amdgcn_fence(...) (void)0
#define __builtin_amdgcn_make_buffer_rsrc(p, stride, n, flags) emu_rsrc{(const char *)(p), (unsigned)(n)}
#define __builtin_amdgcn_raw_buffer_load_b128(r, vo, so, aux) emu_buffer_load<emu_u4>(r, (unsigned)(vo), (unsigned)(so))
#define __builtin_amdgcn_raw_buffer_load_b64(r, vo, so, aux) emu_buffer_load<emu_u2>(r, (unsigned)(vo), (unsigned)(so))
#undef __hip_atomic_store
#undef __hip_atomic_load
#undef __hip_atomic_fetch_add
#define __hip_atomic_store(p, v, o, s) (void)(*(p) = (v))
#define __hip_atomic_load(p, o, s) (*(p))
#define __hip_atomic_fetch_add(p, v, o, s) ((*(p) += (v)) - (v))
inline int emu_width(int w = 64) { return w; }

extern "C" {
// `bytes` of zeros that end at an inaccessible page (to 16 bytes)
void *emu_alloc(size_t bytes)
{
    const size_t page = 4096, body = (bytes + page - 1) / page * page, used = (bytes + 15) / 16 * 16;
    char *p = (char *)mmap(nullptr, body + 2 * page, PROT_NONE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0);
    if (p == MAP_FAILED || (body && mprotect(p + page, body, PROT_READ | PROT_WRITE)))
        return nullptr;
    return p + page + body - used;
}
// one block of `threads` after the other, the lanes of a wave from the first or from the last one on; 0, or -1 with the
// reason in emu_error()
int emu_run(void (*kernel)(const void *), const void *args, unsigned blocks, unsigned threads, int lanes_last_first)
{
    using namespace emu;
    last_first = lanes_last_first != 0;
    std::vector<Wave> waves(threads / 64);
    static std::vector<char *> stacks;
    while (stacks.size() < threads)
        stacks.push_back((char *)mmap(nullptr, STACK, PROT_READ | PROT_WRITE, MAP_PRIVATE | MAP_ANONYMOUS | MAP_NORESERVE, -1, 0));
    for (unsigned t = 0; t < threads; ++t) {
        if (t % 64 == 0)
            waves[t / 64].lane.resize(64);
        waves[t / 64].lane[t % 64].tid = emu_dim3{t, 0, 0};
        waves[t / 64].lane[t % 64].stack = stacks[t];
    }
    static char sigstack[64 * 1024];
    stack_t ss = {}, oss = {};
    ss.ss_sp = sigstack;
    ss.ss_size = sizeof sigstack;
    sigaltstack(&ss, &oss);
    struct sigaction sa = {}, old = {};
    sa.sa_sigaction = on_segv;
    sa.sa_flags = SA_SIGINFO | SA_ONSTACK;
    sigaction(SIGSEGV, &sa, &old);
    block = &waves;
    emu::kernel = kernel;
    kernel_args = args;
    grid_dim = emu_dim3{blocks, 1, 1};
    block_dim = emu_dim3{threads, 1, 1};
    fault_text[0] = 0;
    int rc = sigsetjmp(fault, 1);
    if (rc == 0) {
        for (unsigned b = 0; b < blocks; ++b) {
            block_idx = emu_dim3{b, 0, 0};
            for (Wave &w : waves)
                for (Lane &l : w.lane) {
                    l.state = 0;
                    getcontext(&l.ctx);
                    l.ctx.uc_stack.ss_sp = l.stack;
                    l.ctx.uc_stack.ss_size = STACK;
                    l.ctx.uc_link = nullptr;
                    makecontext(&l.ctx, entry, 0);
                }
            run_block();
        }
    } else if (rc == 1) {
        std::snprintf(fault_text, sizeof fault_text, "block %u, thread %u: access outside its buffers (%p)", block_idx.x, cur->tid.x, fault_at);
    }
    sigaction(SIGSEGV, &old, nullptr);
    sigaltstack(&oss, nullptr);
    return rc ? -1 : 0;
}
const char *emu_error() { return emu::fault_text; }
}
