// Host side of the ternary-linear library: geometry, packers and the host decoders.
// Pure C++ (no HIP calls); compiled into libtl.so together with the kernels.
#include "tl.h"

#include <pthread.h>
#include <sched.h>
#include <signal.h>
#include <unistd.h>

#include <atomic>
#include <cmath>
#include <condition_variable>
#include <cstdio>
#include <cstring>
#include <memory>
#include <mutex>
#include <new>
#include <thread>

namespace {

constexpr int kTritsPerByte = 5;

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }

inline bool shape_ok(int64_t N, int64_t K) {
    return N >= 1 && K >= 1 && N < (int64_t(1) << 40) && K < (int64_t(1) << 40);
}

// digit = w + 1 for w in {-1,0,1}; anything else maps to a value > 2.
inline unsigned digit_of(int8_t w) { return static_cast<unsigned>(static_cast<uint8_t>(w + 1)); }

// The packers read weights eight at a time.  They are bound by instructions, not by memory (one weight at a time:
// 4096 x 4096 to 2-bit words 7.05 ms, 2.4 GB/s of weights).  Bytes -1, 0, 1 become digits 0, 1, 2, byte by byte
// without carries between them; anything else becomes a byte that is_digits tells apart.
inline uint64_t load8(const int8_t* p) {
    uint64_t v;
    std::memcpy(&v, p, 8);                          // little-endian: weight i in byte i
    return v;
}
constexpr uint64_t kOnes = 0x0101010101010101ull;
inline uint64_t digits8(uint64_t w) { return ((w & (kOnes * 0x7F)) + kOnes) ^ (w & (kOnes * 0x80)); }
// nonzero if some byte of d is not 0, 1 or 2
inline uint64_t not_digits(uint64_t d) { return (d & (kOnes * 0xFC)) | (d & (d >> 1) & kOnes); }

// `whole` packed words of 16 weights; returns nonzero if a value was no weight.  The 2-bit fields of eight bytes are drawn
// together in three steps.  A copy for AVX2, four loads to an instruction, is taken where the CPU has it (4096 x 4096
// on one core of a server: one weight at a time 12.6 ms, eight 3.0 ms, with AVX2 1.6 ms).
inline __attribute__((always_inline)) uint64_t pack_words(const int8_t* row, uint32_t* dst, int64_t whole) {
    uint64_t off = 0;
    for (int64_t i = 0; i < whole; ++i) {
        const uint64_t a = digits8(load8(row + 16 * i)), b = digits8(load8(row + 16 * i + 8));
        off |= not_digits(a) | not_digits(b);
        uint64_t p = (a | (a >> 6)) & 0x000F000F000F000Full, q = (b | (b >> 6)) & 0x000F000F000F000Full;
        p = (p | (p >> 12)) & 0x000000FF000000FFull;
        q = (q | (q >> 12)) & 0x000000FF000000FFull;
        dst[i] = static_cast<uint32_t>((p | (p >> 24)) & 0xFFFFu) | static_cast<uint32_t>(q | (q >> 24)) << 16;
    }
    return off;
}
uint64_t pack_words_any(const int8_t* row, uint32_t* dst, int64_t whole) { return pack_words(row, dst, whole); }
#if defined(__x86_64__) && !defined(__HIP_DEVICE_COMPILE__)
__attribute__((target("avx2"))) uint64_t pack_words_avx2(const int8_t* row, uint32_t* dst, int64_t whole) { return pack_words(row, dst, whole); }
inline bool has_avx2() { return __builtin_cpu_supports("avx2"); }
#else
uint64_t pack_words_avx2(const int8_t* row, uint32_t* dst, int64_t whole) { return pack_words(row, dst, whole); }
inline bool has_avx2() { return false; }
#endif

// CPUs this thread may run on
struct Cpus {
    unsigned long mask[16384 / (8 * sizeof(unsigned long))] = {};
    Cpus() { if (sched_getaffinity(0, sizeof mask, reinterpret_cast<cpu_set_t*>(mask)) != 0) mask[0] = 1; }
    int count() const { return CPU_COUNT_S(sizeof mask, reinterpret_cast<const cpu_set_t*>(mask)); }
    bool operator==(const Cpus& o) const { return std::memcmp(mask, o.mask, sizeof mask) == 0; }
};

// CPUs that the process's control group is given time for (cgroup v2 "quota period" or v1's two files), or a large number
int cpu_quota() {
    long long quota = -1, period = 0;
    if (FILE* f = std::fopen("/sys/fs/cgroup/cpu.max", "re")) {
        if (std::fscanf(f, "%lld %lld", &quota, &period) != 2) quota = -1;       // "max 100000": no quota
        std::fclose(f);
    } else if (FILE* q = std::fopen("/sys/fs/cgroup/cpu/cpu.cfs_quota_us", "re")) {
        if (std::fscanf(q, "%lld", &quota) != 1) quota = -1;
        std::fclose(q);
        if (FILE* p = std::fopen("/sys/fs/cgroup/cpu/cpu.cfs_period_us", "re")) {
            if (std::fscanf(p, "%lld", &period) != 1) period = 0;
            std::fclose(p);
        }
    }
    if (quota <= 0 || period <= 0) return 1 << 20;
    return quota < period ? 1 : static_cast<int>(quota / period < (1 << 20) ? quota / period : 1 << 20);
}

// The work of one call of a packer: rows 0 .. N - 1 in pieces, which the caller and helpers take as they come.
struct Pieces {
    int64_t N, rows_each, count;
    unsigned (*pack)(const void* rows, int64_t n0, int64_t n1);
    const void* rows;                                      // the caller's: read for a piece that was taken, and the caller waits for those
    int helpers;                                           // that may still join (under Helpers::m)
    std::atomic<int64_t> next{0}, done{0};
    std::atomic<unsigned> bad{0};
    void work() {
        for (int64_t p = next.fetch_add(1); p < count; p = next.fetch_add(1)) {
            const int64_t n0 = p * rows_each;
            if (pack(rows, n0, n0 + rows_each < N ? n0 + rows_each : N)) bad.store(1);
            done.fetch_add(1);
        }
    }
};

// Up to 7 threads that wait for calls of the packers: started by the first call that wants them, one call's at a time (another one meanwhile works
// alone), ended with the library.  Nothing waits for a helper that has not begun: a call ends when the pieces that were taken are done.  Threads
// started and joined in every call waited for cores on which a program's own workers still spun.  us on 8 cores, 2-bit words, right after the tensor operation
// that made the weights / repeated, one thread -> such threads -> these: 2048 x 1024 354 / 209 -> 1296 / 175 -> 348 / 155, 2048 x 2048 586 / 426 -> 2357 / 201 ->
// 395 / 226, 4096 x 4096 2423 / 2107 -> 2969 / 528 -> 1381 / 347; 1.6-bit codes, 1024 x 1024 400 / 351 -> 3191 / 225 -> 235 / 129, 4096 x 4096 5469 /
// 5439 -> 3133 / 1051 -> 2587 / 932.  A forked child has none of its parent's threads and starts its own.
class Helpers {
public:
    static constexpr int kMost = 7;
    const pid_t pid = getpid();
    const Cpus cpus;
    const int quota = cpu_quota();

    void run(const std::shared_ptr<Pieces>& p) {
        if (!busy.exchange(true)) {
            {
                std::lock_guard<std::mutex> hold(m);
                if (!stop && started < p->helpers) start(p->helpers);
                current = p;
            }
            wake.notify_one();
            p->work();
            {
                std::lock_guard<std::mutex> hold(m);
                current.reset();
            }
            busy.store(false);
        } else {
            p->work();
        }
        for (int spins = 0; p->done.load() < p->count; ++spins) {
            if (spins >= 200) sched_yield();
        }
    }
    void end() {
        {
            std::lock_guard<std::mutex> hold(m);
            stop = true;
        }
        wake.notify_all();
        for (int i = 0; i < started; ++i) threads[i].join();
    }

private:
    // under m; the program's signals stay with its own threads
    void start(int count) {
        sigset_t all, before;
        sigfillset(&all);
        pthread_sigmask(SIG_SETMASK, &all, &before);
        try {
            for (; started < count && started < kMost; ++started) threads[started] = std::thread([this] { serve(); });
        } catch (...) {                                    // no thread to be had: those there are
        }
        pthread_sigmask(SIG_SETMASK, &before, nullptr);
    }
    void serve() {
        std::shared_ptr<Pieces> last;
        for (;;) {
            {
                std::unique_lock<std::mutex> hold(m);
                wake.wait(hold, [&] { return stop || (current && current != last && current->helpers > 0); });
                if (stop) return;
                last = current;
                if (--last->helpers > 0) wake.notify_one();
            }
            last->work();
        }
    }
    std::mutex m;
    std::condition_variable wake;
    std::shared_ptr<Pieces> current;
    std::thread threads[kMost];
    int started = 0;
    bool stop = false;
    std::atomic<bool> busy{false};
};

// This process's helpers.  The object itself is never freed: a thread may still be in a call when the library ends.
std::atomic<Helpers*> g_helpers{nullptr};
Helpers* helpers() {
    Helpers* h = g_helpers.load();
    if (h && h->pid == getpid()) return h;
    Helpers* mine = new (std::nothrow) Helpers;
    if (mine == nullptr) return nullptr;
    if (g_helpers.compare_exchange_strong(h, mine)) return mine;
    delete mine;
    return h;
}
struct EndHelpers {
    ~EndHelpers() {
        Helpers* h = g_helpers.load();
        if (h && h->pid == getpid()) h->end();
    }
} g_end_helpers;

// The packers' rows 0 .. N - 1: rows(n0, n1) packs some and returns nonzero for a value that is no weight.  A thread for every `share` weights, which one
// packs in 45 us (2-bit words), 25 and 40 us (the two 1.6-bit codes) on a server, at most 8.
template <class Rows>
unsigned over_rows(int64_t N, int64_t K, double share, const Rows& rows) {
    const double want = static_cast<double>(N) * static_cast<double>(K) / share;
    if (want < 2.0 || N < 2) return rows(int64_t(0), N);
    const Cpus here;
    int threads = want < Helpers::kMost + 1 ? static_cast<int>(want) : Helpers::kMost + 1;
    if (threads > here.count()) threads = here.count();
    Helpers* const h = threads > 1 ? helpers() : nullptr;
    if (h != nullptr && threads > h->quota) threads = h->quota;
    if (h == nullptr || threads < 2 || !(h->cpus == here)) return rows(int64_t(0), N);
    std::shared_ptr<Pieces> p;
    try {
        p = std::make_shared<Pieces>();
    } catch (...) {
        return rows(int64_t(0), N);
    }
    p->N = N;
    p->rows_each = ceil_div(N, int64_t(8) * threads);
    p->count = ceil_div(N, p->rows_each);
    p->pack = [](const void* r, int64_t n0, int64_t n1) -> unsigned { return (*static_cast<const Rows*>(r))(n0, n1); };
    p->rows = &rows;
    p->helpers = threads - 1;
    h->run(p);
    return p->bad.load();
}
constexpr double kShare2Bit = 1e6, kShare1p6 = 1.5e5;

// Base-3 byte -> its five digits, least significant first (digits of v mod 243 for v > 242).
struct Base3Table {
    uint8_t d[256][kTritsPerByte];
    Base3Table() {
        for (int v = 0; v < 256; ++v) {
            int r = v % 243;
            for (int i = 0; i < kTritsPerByte; ++i) { d[v][i] = static_cast<uint8_t>(r % 3); r /= 3; }
        }
    }
};

const Base3Table& base3_table() {
    static const Base3Table t;
    return t;
}

}  // namespace

extern "C" {

const char* tl_status_str(tl_status s) {
    switch (s) {
        case TL_OK: return "ok";
        case TL_ERR_NULL: return "null pointer";
        case TL_ERR_SHAPE: return "bad shape";
        case TL_ERR_VALUE: return "value outside the ternary code";
        case TL_ERR_ALIGN: return "pointer not 16-byte aligned";
        case TL_ERR_UNSUPPORTED: return "unsupported format, path or shape";
        case TL_ERR_HIP: return "HIP runtime error";
    }
    return "unknown status";
}

size_t tl_row_stride_bytes(tl_format fmt, int64_t K) {
    if (K < 1 || K >= (int64_t(1) << 40)) return 0;
    switch (fmt) {
        case TL_FMT_2BIT: return static_cast<size_t>(4 * ceil_div(K, 16));
        case TL_FMT_1P6BIT:
        case TL_FMT_1P6BIT_FX: return static_cast<size_t>(16 * ceil_div(ceil_div(K, kTritsPerByte), 16));
        default: return 0;                       // an unknown format
    }
}

size_t tl_packed_bytes(tl_format fmt, int64_t N, int64_t K) {
    if (!shape_ok(N, K)) return 0;
    return static_cast<size_t>(N) * tl_row_stride_bytes(fmt, K);
}

namespace {

// fp64 -> fp16 bits, round to nearest even; subnormals kept, overflow to infinity.
uint16_t double_to_half_bits(double v) {
    const uint16_t sign = std::signbit(v) ? 0x8000u : 0u;
    const double a = std::fabs(v);
    if (std::isnan(a)) return static_cast<uint16_t>(sign | 0x7E00u);
    if (a >= 65520.0) return static_cast<uint16_t>(sign | 0x7C00u);
    int e = 0;
    (void)std::frexp(a, &e);                        // a = f * 2^e, f in [0.5, 1)
    e -= 1;                                         // a in [2^e, 2^(e+1))
    if (a == 0.0 || e < -14) {                      // subnormal range: units of 2^-24
        const double q = std::nearbyint(std::ldexp(a, 24));
        return static_cast<uint16_t>(sign | static_cast<uint16_t>(q));   // q = 1024 is the least normal
    }
    double m = std::nearbyint(std::ldexp(a, 10 - e));                    // in [1024, 2048]
    if (m >= 2048.0) { m = 1024.0; e += 1; }
    if (e > 15) return static_cast<uint16_t>(sign | 0x7C00u);
    return static_cast<uint16_t>(sign | ((e + 15) << 10) | (static_cast<int>(m) - 1024));
}

}  // namespace

// App. B "Forward Pass": gamma = eps + mean |W|, What = round(clip(W / gamma, -1, 1)).
tl_status tl_quantize(const float* W, int64_t N, int64_t K, double eps, int8_t* What,
                      double* gamma, uint16_t* gamma_fp16_bits) {
    if (!W || !What) return TL_ERR_NULL;
    if (!shape_ok(N, K)) return TL_ERR_SHAPE;
    if (!(eps >= 0.0) || !std::isfinite(eps)) return TL_ERR_VALUE;
    const int64_t count = N * K;
    // sum of |W| in fp64 with a running compensation (Neumaier), so that the result does not
    // depend on the order more than in its last bit
    double sum = 0.0, comp = 0.0;
    bool bad = false;
    for (int64_t i = 0; i < count; ++i) {
        const double a = std::fabs(static_cast<double>(W[i]));
        bad |= !std::isfinite(a);
        const double t = sum + a;
        comp += (sum >= a) ? (sum - t) + a : (a - t) + sum;
        sum = t;
    }
    if (bad) return TL_ERR_VALUE;
    const double g = eps + (sum + comp) / static_cast<double>(count);
    if (gamma) *gamma = g;
    if (gamma_fp16_bits) *gamma_fp16_bits = double_to_half_bits(g);
    for (int64_t i = 0; i < count; ++i) {
        double q = (g > 0.0) ? static_cast<double>(W[i]) / g : 0.0;
        q = q < -1.0 ? -1.0 : (q > 1.0 ? 1.0 : q);
        What[i] = static_cast<int8_t>(std::nearbyint(q));              // half to even
    }
    return TL_OK;
}

// Sec. 3.1 with k = 16: weight 16i+j in bits [2j+1:2j].  A short last word is built from its top digit down
// (Horner in base 4).
tl_status tl_pack_2bit(const int8_t* W, int64_t N, int64_t K, uint32_t* out) {
    if (!W || !out) return TL_ERR_NULL;
    if (!shape_ok(N, K)) return TL_ERR_SHAPE;
    const int64_t words = ceil_div(K, 16);
    const bool avx2 = has_avx2();
    const unsigned any_bad = over_rows(N, K, kShare2Bit, [=](int64_t n0, int64_t n1) {
        unsigned bad = 0;
        for (int64_t n = n0; n < n1; ++n) {
            const int8_t* row = W + n * K;
            uint32_t* dst = out + n * words;
            const int64_t whole = K / 16;
            bad |= ((avx2 ? pack_words_avx2(row, dst, whole) : pack_words_any(row, dst, whole)) != 0);
            for (int64_t i = whole; i < words; ++i) {
                const int64_t base = 16 * i;
                const int len = static_cast<int>(K - base < 16 ? K - base : 16);
                uint32_t word = 0;
                for (int j = 15; j >= 0; --j) {
                    const unsigned dgt = (j < len) ? digit_of(row[base + j]) : 1u;
                    bad |= (dgt > 2u);
                    word = (word << 2) | (dgt & 3u);
                }
                dst[i] = word;
            }
        }
        return bad;
    });
    return any_bad ? TL_ERR_VALUE : TL_OK;
}

// Plain base-3 byte, digit i of the byte = weight 5b+i (Horner from the top digit).
tl_status tl_pack_1p6bit(const int8_t* W, int64_t N, int64_t K, uint8_t* out) {
    if (!W || !out) return TL_ERR_NULL;
    if (!shape_ok(N, K)) return TL_ERR_SHAPE;
    const int64_t stride = static_cast<int64_t>(tl_row_stride_bytes(TL_FMT_1P6BIT, K));
    const int64_t nbytes = ceil_div(K, kTritsPerByte);
    const unsigned any_bad = over_rows(N, K, kShare1p6, [=](int64_t n0, int64_t n1) {
        unsigned bad = 0;
        for (int64_t n = n0; n < n1; ++n) {
            const int8_t* row = W + n * K;
            uint8_t* dst = out + n * stride;
            // bytes whose weights are followed by three more: five digits of an 8-byte load, gathered by one product
            // (each byte of it up to the fifth is a sum of digits times distinct powers of 3, below 256: no carries)
            constexpr uint64_t kGather = (1ull << 32) | (3ull << 24) | (9ull << 16) | (27ull << 8) | 81ull;
            uint64_t off = 0;
            const int64_t whole = K >= 8 ? (K - 8) / kTritsPerByte + 1 : 0;
            for (int64_t b = 0; b < whole; ++b) {
                const uint64_t d = digits8(load8(row + kTritsPerByte * b)) & 0xFFFFFFFFFFull;
                off |= not_digits(d);
                dst[b] = static_cast<uint8_t>((d * kGather) >> 32);
            }
            bad |= (off != 0);
            for (int64_t b = whole; b < nbytes; ++b) {
                const int64_t base = kTritsPerByte * b;
                unsigned v = 0;
                for (int i = kTritsPerByte - 1; i >= 0; --i) {
                    const unsigned dgt = (base + i < K) ? digit_of(row[base + i]) : 1u;
                    bad |= (dgt > 2u);
                    v = v * 3u + (dgt > 2u ? 0u : dgt);
                }
                dst[b] = static_cast<uint8_t>(v);
            }
            std::memset(dst + nbytes, 0, static_cast<size_t>(stride - nbytes));
        }
        return bad;
    });
    return any_bad ? TL_ERR_VALUE : TL_OK;
}

// Sec. 3.2 / App. E with k = 5, p = 8: digits big-endian, byte = floor((256 Nval + 242) / 243).
tl_status tl_pack_1p6bit_fx(const int8_t* W, int64_t N, int64_t K, uint8_t* out) {
    if (!W || !out) return TL_ERR_NULL;
    if (!shape_ok(N, K)) return TL_ERR_SHAPE;
    const int64_t stride = static_cast<int64_t>(tl_row_stride_bytes(TL_FMT_1P6BIT, K));
    const int64_t nbytes = ceil_div(K, kTritsPerByte);
    const unsigned any_bad = over_rows(N, K, kShare1p6, [=](int64_t n0, int64_t n1) {
        unsigned bad = 0;
        for (int64_t n = n0; n < n1; ++n) {
            const int8_t* row = W + n * K;
            uint8_t* dst = out + n * stride;
            // as in tl_pack_1p6bit, the powers of 3 the other way round
            constexpr uint64_t kGather = (81ull << 32) | (27ull << 24) | (9ull << 16) | (3ull << 8) | 1ull;
            uint64_t off = 0;
            const int64_t whole = K >= 8 ? (K - 8) / kTritsPerByte + 1 : 0;
            for (int64_t b = 0; b < whole; ++b) {
                const uint64_t d = digits8(load8(row + kTritsPerByte * b)) & 0xFFFFFFFFFFull;
                off |= not_digits(d);
                const uint32_t nval = static_cast<uint32_t>((d * kGather) >> 32) & 255u;
                dst[b] = static_cast<uint8_t>((nval * 256u + 242u) / 243u);
            }
            bad |= (off != 0);
            for (int64_t b = whole; b < nbytes; ++b) {
                const int64_t base = kTritsPerByte * b;
                unsigned nval = 0;
                for (int j = 0; j < kTritsPerByte; ++j) {
                    const unsigned dgt = (base + j < K) ? digit_of(row[base + j]) : 1u;
                    bad |= (dgt > 2u);
                    nval = nval * 3u + (dgt > 2u ? 0u : dgt);
                }
                dst[b] = static_cast<uint8_t>((nval * 256u + 242u) / 243u);
            }
            std::memset(dst + nbytes, 0, static_cast<size_t>(stride - nbytes));
        }
        return bad;
    });
    return any_bad ? TL_ERR_VALUE : TL_OK;
}

// Decode of the fixed-point code: b = ceil(256 V / 243) is inverted by V = floor(243 b / 256),
// and V's base-3 digits, most significant first, are the weights + 1.  (App. F, Alg. 1 peels the
// same digits off with multiplications by 3; the tests hold this decode against it.)
tl_status tl_unpack_1p6bit_fx(const uint8_t* packed, int64_t N, int64_t K, int8_t* W_out) {
    if (!packed || !W_out) return TL_ERR_NULL;
    if (!shape_ok(N, K)) return TL_ERR_SHAPE;
    const int64_t stride = static_cast<int64_t>(tl_row_stride_bytes(TL_FMT_1P6BIT, K));
    static const unsigned kPow3[kTritsPerByte] = {81u, 27u, 9u, 3u, 1u};
    for (int64_t n = 0; n < N; ++n) {
        const uint8_t* src = packed + n * stride;
        int8_t* row = W_out + n * K;
        for (int64_t base = 0; base < K; base += kTritsPerByte) {
            const unsigned value = (243u * src[base / kTritsPerByte]) >> 8;
            for (int i = 0; i < kTritsPerByte && base + i < K; ++i)
                row[base + i] = static_cast<int8_t>(static_cast<int>((value / kPow3[i]) % 3u) - 1);
        }
    }
    return TL_OK;
}

tl_status tl_unpack(tl_format fmt, const void* packed, int64_t N, int64_t K, int8_t* W_out) {
    if (!packed || !W_out) return TL_ERR_NULL;
    if (!shape_ok(N, K)) return TL_ERR_SHAPE;
    unsigned bad = 0;
    if (fmt == TL_FMT_2BIT) {
        const int64_t words = ceil_div(K, 16);
        const uint32_t* src = static_cast<const uint32_t*>(packed);
        for (int64_t n = 0; n < N; ++n) {
            int8_t* row = W_out + n * K;
            for (int64_t i = 0; i < words; ++i) {
                uint32_t word = src[n * words + i];
                const int64_t base = 16 * i;
                const int len = static_cast<int>(K - base < 16 ? K - base : 16);
                for (int j = 0; j < len; ++j, word >>= 2) {
                    const unsigned dgt = word & 3u;
                    bad |= (dgt == 3u);
                    row[base + j] = static_cast<int8_t>(static_cast<int>(dgt) - 1);
                }
            }
        }
        return bad ? TL_ERR_VALUE : TL_OK;
    }
    if (fmt == TL_FMT_1P6BIT) {
        const Base3Table& T = base3_table();
        const int64_t stride = static_cast<int64_t>(tl_row_stride_bytes(fmt, K));
        const uint8_t* src = static_cast<const uint8_t*>(packed);
        for (int64_t n = 0; n < N; ++n) {
            int8_t* row = W_out + n * K;
            for (int64_t base = 0; base < K; base += kTritsPerByte) {
                const uint8_t v = src[n * stride + base / kTritsPerByte];
                bad |= (v > 242u);
                for (int i = 0; i < kTritsPerByte && base + i < K; ++i)
                    row[base + i] = static_cast<int8_t>(static_cast<int>(T.d[v][i]) - 1);
            }
        }
        return bad ? TL_ERR_VALUE : TL_OK;
    }
    if (fmt == TL_FMT_1P6BIT_FX)
        return tl_unpack_1p6bit_fx(static_cast<const uint8_t*>(packed), N, K, W_out);
    return TL_ERR_UNSUPPORTED;
}

}  // extern "C"
