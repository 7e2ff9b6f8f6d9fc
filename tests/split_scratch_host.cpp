// The host side of products that the library cuts by itself, in their contraction or into two launches, on a stand-in for the HIP runtime:
// this program defines the runtime calls of that path, so that the library's calls come here and nothing reaches a GPU.  A stream and an
// event carry clocks (which operations of each stream lie before them); a part of the scratch space must only be taken up by a stream
// that comes after its last user.  The argument names the test; exit status 0: passed.
#include <hip/hip_runtime_api.h>

#include <cstdint>
#include <cstdio>
#include <cstring>
#include <exception>
#include <map>
#include <vector>

namespace tio {
namespace k {
void gemm(hipStream_t s, int dtype, bool a_km, bool b_km, int64_t M, int64_t N, int64_t K, const void *A, int64_t lda, const void *B, int64_t ldb,
          const void *bias, const void *resid, int64_t ldr, void *C, int64_t ldc, void *rowsum, void *workspace, int splits, bool accumulate);
}
}  // namespace tio

namespace {
constexpr int BF16 = 1, STREAMS = 8;
using Clock = std::map<hipStream_t, int>;            // stream -> number of its operations that lie before
std::map<hipStream_t, Clock> streams;
std::map<hipEvent_t, Clock> events;
std::map<hipStream_t, int> device_of;
int launches = 0, event_calls = 0, records_to_fail = 0;
void *last_first_arg = nullptr;
struct Launched { int64_t M, N; int streamed; uintptr_t A, B, bias, resid, C, rowsum; int64_t ldr, ldc; int rowsum_acc; };
bool keep_launches = false;                          // launches of the product kernels alone: their arguments are read by position
std::vector<Launched> launched;
struct Config { dim3 grid, block; size_t lds; hipStream_t stream; } config;
constexpr int64_t ARRAY_BYTES = (int64_t)4 * 72 << 20;
alignas(256) unsigned char image[64];                // stands for the array of the device image: never read or written

hipStream_t stream(int i) { return reinterpret_cast<hipStream_t>(static_cast<uintptr_t>(0x1000 * (i + 1))); }
void merge(Clock &into, const Clock &from) {
    for (auto &[s, n] : from)
        if (into[s] < n) into[s] = n;
}
}  // namespace

extern "C" {
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *status) { *status = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipGetDevice(int *dev) { *dev = 0; return hipSuccess; }
hipError_t hipStreamGetDevice(hipStream_t s, hipDevice_t *dev) { *dev = device_of[s]; return hipSuccess; }
hipError_t hipThreadExchangeStreamCaptureMode(hipStreamCaptureMode *) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { *p = image; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t *e, unsigned) {
    static uintptr_t next = 0x100000;
    *e = reinterpret_cast<hipEvent_t>(next += 16);
    events[*e];
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) {
    ++event_calls;
    if (records_to_fail) { --records_to_fail; return hipErrorUnknown; }
    events[e] = streams[s];
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { ++event_calls; merge(streams[s], events[e]); return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t s) { config = {grid, block, lds, s}; return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *s) {
    *grid = config.grid; *block = config.block; *lds = config.lds; *s = config.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *, dim3, dim3, void **args, size_t, hipStream_t s) {
    ++launches;
    ++streams[s][s];
    last_first_arg = *static_cast<void **>(args[0]);
    auto number = [&](int i) { return *static_cast<int64_t *>(args[i]); };
    auto address = [&](int i) { return *static_cast<uintptr_t *>(args[i]); };
    if (keep_launches)
        launched.push_back({number(9), number(10), *static_cast<int *>(args[19]), address(0), address(2), address(4), address(5), address(7), address(14),
                            number(6), number(8), *static_cast<int *>(args[17])});
    return hipSuccess;
}
}

namespace {
struct Use { hipStream_t stream; int operations; };
std::map<void *, Use> parts;                         // part of the scratch space -> its last user and that stream's operations so far

// a product of 200 x 300 x 15000, which the library cuts: two launches, of which the second reads the partials (its first argument)
bool product(hipStream_t s, bool accumulate = false, const void *resid = nullptr) {
    void *const operand = image;
    launches = 0;
    tio::k::gemm(s, BF16, false, false, 200, 300, 15000, operand, 15000, operand, 15000, nullptr, resid, 304, operand, 304, nullptr, nullptr, 1,
                 accumulate);
    if (launches != 2) return launches == 1;
    const auto last = parts.find(last_first_arg);
    if (last != parts.end() && streams[s][last->second.stream] < last->second.operations) {
        std::printf("a part of the scratch space is taken up while another stream may be using it\n");
        return false;
    }
    parts[last_first_arg] = {s, streams[s][s]};
    return true;
}

bool cuts_and_waits() {
    for (int i = 0; i < 40; ++i)
        if (!product(stream(i * 5 % STREAMS)) || launches != 2) return false;
    return parts.size() > 1;
}

// accumulate adds to C in place of a residual: both together are refused before anything is launched, whatever the size
bool refuses_accumulate_with_residual() {
    try {
        product(stream(0), true, image);
    } catch (const std::exception &) {
        return launches == 0;
    }
    std::printf("accepted, %d launches\n", launches);
    return false;
}
// A part whose last use has left no event behind is not handed out again
bool a_failed_record_ends_the_sharing() {
    if (!product(stream(0)) || !product(stream(1))) return false;
    records_to_fail = 1;
    if (!product(stream(2)) || records_to_fail) return false;
    for (int i = 0; i < 40; ++i)
        if (!product(stream(3 + i % (STREAMS - 3)))) return false;
    return true;
}
// The scratch space and its events are those of the current device: a stream of another one takes its products in one range
bool leaves_streams_of_other_devices_alone() {
    device_of[stream(1)] = 1;
    if (!product(stream(0)) || launches != 2) return false;
    const int before = event_calls;
    if (!product(stream(1)) || launches != 1) { std::printf("%d launches\n", launches); return false; }
    return event_calls == before && product(nullptr) && launches == 2;
}
// Products whose partials take a few MiB and up to 64: as many streams as there are parts do not wait for each other, whatever the sizes;
// with more streams, what one takes up has been left by every earlier user of any of its bytes
struct Shape { int64_t M, N, K, ranges; };
constexpr Shape SHAPES[] = {{200, 300, 15000, 8}, {8192, 768, 50257, 2}, {4096, 1024, 32000, 4}, {300, 300, 8000, 8}, {4096, 1792, 12940, 2}, {8192, 1024, 32000, 2}};
int64_t partial_bytes(const Shape &p) { return p.ranges * (p.M * ((p.N + 3) / 4 * 4) + p.M) * 4; }
bool shape_on(const Shape &p, hipStream_t s) {
    launches = 0;
    tio::k::gemm(s, BF16, false, true, p.M, p.N, p.K, image, (p.K + 7) / 8 * 8, image, p.N + 8, nullptr, nullptr, 0, image, p.N, nullptr, nullptr, 1, false);
    if (launches != 2) std::printf("%d launches of %d x %d x %d\n", launches, (int)p.M, (int)p.N, (int)p.K);
    return launches == 2;
}
bool large_products_of_four_streams_do_not_wait() {
    for (int i = 0; i < 200; ++i) {
        const hipStream_t s = stream(i * 3 % 4);
        if (!shape_on(SHAPES[i * 7 % 6], s)) return false;
        for (auto &[other, n] : streams[s])
            if (other != s && n > 0) { std::printf("stream %d waits for another one\n", i * 3 % 4); return false; }
    }
    return true;
}
bool large_products_share_no_bytes_with_a_running_one() {
    struct Extent { int64_t first, end; Use use; };
    std::vector<Extent> taken;
    int64_t end = 0;
    for (int i = 0; i < 200; ++i) {
        const Shape &p = SHAPES[i * 7 % 6];
        const hipStream_t s = stream(i * 5 % STREAMS);
        if (!shape_on(p, s)) return false;
        const int64_t first = static_cast<unsigned char *>(last_first_arg) - image;
        for (const Extent &e : taken)
            if (first < e.end && e.first < first + partial_bytes(p) && streams[s][e.use.stream] < e.use.operations) {
                std::printf("bytes from %lld on are taken up while another stream may be using them\n", (long long)first);
                return false;
            }
        taken.push_back({first, first + partial_bytes(p), {s, streams[s][s]}});
        if (first + partial_bytes(p) > end) end = first + partial_bytes(p);
    }
    return end <= ARRAY_BYTES;
}
// An output of 256 MiB and more goes past the caches whole, in whichever launches it is made
bool streams_outputs_by_the_size_of_the_product() {
    struct Output { int64_t M, N, K; size_t launches; bool streamed; };
    constexpr Output OUTPUTS[] = {{8176, 16470, 3143, 2, true}, {7727, 17374, 4540, 2, true}, {8192, 50257, 768, 1, true}, {4096, 32768, 72, 1, true},
                                  {4095, 32776, 72, 1, false}, {1021, 50257, 768, 2, false}};
    keep_launches = true;
    for (const Output &o : OUTPUTS) {
        launched.clear();
        tio::k::gemm(stream(0), BF16, false, false, o.M, o.N, o.K, image, (o.K + 7) / 8 * 8, image, (o.K + 7) / 8 * 8, nullptr, nullptr, 0, image,
                     (o.N + 7) / 8 * 8, nullptr, nullptr, 1, false);
        if (launched.size() != o.launches) { std::printf("%d x %d x %d: %d launches\n", (int)o.M, (int)o.N, (int)o.K, (int)launched.size()); return false; }
        int64_t elements = 0;
        for (const Launched &l : launched) {
            elements += l.M * l.N;
            if (l.streamed != o.streamed) { std::printf("%d x %d of %d x %d: %d\n", (int)l.M, (int)l.N, (int)o.M, (int)o.N, l.streamed); return false; }
        }
        if (elements != o.M * o.N) { std::printf("%lld elements of %d x %d\n", (long long)elements, (int)o.M, (int)o.N); return false; }
    }
    return true;
}
// A product in two launches: the second has the operands' next rows or columns, with bias, residual, row sums and C beside them; where C is
// accumulated it is the residual of both, and the row sums of both add
bool a_second_launch_goes_on_where_the_first_ends() {
    struct Cut { int64_t M, N, K; bool a_km, b_km, rowsum, by_rows; };
    constexpr Cut CUTS[] = {{50257, 768, 1021, true, true, true, true},   {6200, 8449, 1000, true, false, false, true}, {4224, 12277, 1200, false, false, false, true},
                            {16001, 3130, 1161, true, true, true, false}, {1792, 9664, 1000, false, true, false, false}, {1021, 50257, 768, false, false, false, false}};
    constexpr uintptr_t A = 0x10000000000, B = 0x20000000000, C = 0x30000000000, BIAS = 0x40000000000, RESID = 0x50000000000, ROWSUM = 0x60000000000;
    auto at = [](uintptr_t p) { return reinterpret_cast<void *>(p); };
    auto up8 = [](int64_t n) { return (n + 7) / 8 * 8; };
    keep_launches = true;
    for (const Cut &c : CUTS)
        for (const bool accumulate : {false, true}) {
            const int64_t lda = up8(c.a_km ? c.M : c.K), ldb = up8(c.b_km ? c.N : c.K), ldc = up8(c.N) + 16, ldr = accumulate ? ldc : up8(c.N);
            launched.clear();
            tio::k::gemm(stream(0), BF16, c.a_km, c.b_km, c.M, c.N, c.K, at(A), lda, at(B), ldb, at(BIAS), accumulate ? nullptr : at(RESID),
                         accumulate ? 0 : ldr, at(C), ldc, c.rowsum ? at(ROWSUM) : nullptr, nullptr, 1, accumulate);
            if (launched.size() != 2) { std::printf("%d launches\n", (int)launched.size()); return false; }
            const Launched &f = launched[0], &s = launched[1];
            const int64_t rows = c.by_rows ? f.M : 0, cols = c.by_rows ? 0 : f.N;
            const uintptr_t resid = accumulate ? C : RESID, rowsum = c.rowsum ? ROWSUM : 0;
            const bool first = f.A == A && f.B == B && f.bias == BIAS && f.resid == resid && f.C == C && f.rowsum == rowsum;
            const bool sizes = c.by_rows ? f.N == c.N && s.N == c.N && f.M + s.M == c.M : f.M == c.M && s.M == c.M && f.N + s.N == c.N;
            const bool second = s.A == A + 2 * rows * (c.a_km ? 1 : lda) && s.B == B + 2 * cols * (c.b_km ? 1 : ldb) && s.bias == BIAS + 2 * cols &&
                                s.resid == resid + 2 * (rows * ldr + cols) && s.C == C + 2 * (rows * ldc + cols) &&
                                s.rowsum == (c.by_rows && c.rowsum ? ROWSUM + 2 * rows : 0);
            const bool same = f.ldr == ldr && s.ldr == ldr && f.ldc == ldc && s.ldc == ldc && f.rowsum_acc == accumulate && s.rowsum_acc == accumulate;
            if (!first || !sizes || !second || !same) {
                std::printf("%d x %d x %d, accumulate %d: first %d sizes %d second %d same %d\n", (int)c.M, (int)c.N, (int)c.K, accumulate, first, sizes, second, same);
                return false;
            }
        }
    return true;
}
}  // namespace

int main(int argc, char **argv) {
    const char *name = argc > 1 ? argv[1] : "";
    bool (*const tests[])() = {cuts_and_waits, refuses_accumulate_with_residual, a_failed_record_ends_the_sharing, leaves_streams_of_other_devices_alone,
                              large_products_of_four_streams_do_not_wait, large_products_share_no_bytes_with_a_running_one,
                              streams_outputs_by_the_size_of_the_product, a_second_launch_goes_on_where_the_first_ends};
    const char *const names[] = {"cuts_and_waits", "refuses_accumulate_with_residual", "a_failed_record_ends_the_sharing",
                                 "leaves_streams_of_other_devices_alone", "large_products_of_four_streams_do_not_wait",
                                 "large_products_share_no_bytes_with_a_running_one", "streams_outputs_by_the_size_of_the_product",
                                 "a_second_launch_goes_on_where_the_first_ends"};
    for (size_t i = 0; i < sizeof names / sizeof *names; ++i)
        if (!std::strcmp(name, names[i])) return tests[i]() ? 0 : 1;
    return 2;
}
