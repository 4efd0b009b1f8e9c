// Batch plans (qap_api.hip) on the stand-in runtime: the side streams a plan creates, and what is
// finished once the caller's stream is waited for.
#include "standin_hip.h"

#define __align__(x)
#define HIP_SYMBOL(x) (x)
#include "../paper_2307_11248_amd/csrc/qap_api.hip"

extern "C" {
hipError_t hipEventCreate(hipEvent_t *e) { return hipEventCreateWithFlags(e, 0); }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float *ms, hipEvent_t, hipEvent_t) { return *ms = 1, hipSuccess; }
hipError_t hipMallocAsync(void **p, size_t n, hipStream_t) { return hipMalloc(p, n); }
hipError_t hipFreeAsync(void *p, hipStream_t) { return std::free(p), hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *s) { return *p = const_cast<void *>(s), hipSuccess; }
}

namespace qapk {
hipError_t launch_table(const TableArgs &, hipStream_t s) { return put(s); }
hipError_t launch_cost(const TableArgs &, hipStream_t s) { return put(s); }
hipError_t launch_table_batch(const BatchArgs &b, size_t, hipStream_t s) { return b.count ? put(s) : hipSuccess; }
hipError_t launch_search(int, bool, const SearchArgs &, int, int, hipStream_t s) { return put(s); }
hipError_t launch_stream(bool, const SearchArgs &, int, hipStream_t s) { return put(s); }
hipError_t launch_block(bool, int, bool, size_t, const SearchArgs *, const BatchArgs *, int, hipStream_t s) { return put(s); }
hipError_t launch_wide_block(bool, const SearchArgs &, int, hipStream_t s) { return put(s); }
hipError_t launch_batch_group(int, const BatchArgs &, size_t, hipStream_t s) { return put(s); }
hipError_t launch_batch_freq(const BatchArgs &, size_t, hipStream_t s) { return put(s); }
int block_form(int n, int sym) { return 2 * ((n + 31) / 32 - 1) + (sym ? 1 : 0); }
int block_ok(int n, int, int blk, bool, int, int, size_t) { return blk && n <= WIDE_N; }
int wide_block_ok(bool, const SearchArgs &, size_t) { return 1; }
size_t block_smem_bytes(int, int, int, bool) { return 1024; }
size_t table_smem_bytes(int) { return 1024; }
size_t search_smem_bytes(int, int, int, int) { return 1024; }
size_t stream_smem_bytes(int, int) { return 1024; }
size_t freq_static_lds() { return 1024; }
int search_lanes(int, int, int, int) { return 512; }
int search_max_lanes(int) { return 512; }
int search_blocks_per_cu(int, int, bool, int, int) { return 1; }
int batch_variant(int n, int, bool stream, int, int) { return n > WIDE_N ? BV_WIDE : (stream ? BV_STREAM : BV_R4); }
int batch_variant_lanes(int) { return 512; }
int batch_shape_ok(int n, int, int, int) { return n <= WIDE_N; }
int batch_shape_ok_wide(int n, int, int, int) { return n <= WIDE_N; }
int stream_shape_ok(int, int, size_t) { return 1; }
}  // namespace qapk

namespace {

// A plan of one search for each size (odd ones symmetric), run once.  Returns the streams it
// created, -1 if something failed or was not finished with the caller's stream.  fail_at: the
// call of the run that fails, counted from 0.
int plan(const std::vector<int> &sizes, int iters, int copies = 1, int fail_at = -1) {
    std::vector<qap_handle> hs;
    std::vector<int32_t> k, lo, hi, perms;
    std::vector<uint64_t> seed;
    for (int n : sizes) {
        std::vector<int32_t> F((size_t)n * n, 1);
        if (n % 2 == 0) F[1] = 0;
        qap_handle h = nullptr;
        if (qap_create(F.data(), F.data(), n, &h)) return -1;
        hs.push_back(h);
        k.push_back(copies);
        lo.push_back(1);
        hi.push_back(5);
        seed.push_back(0);
    }
    const int before = (int)g_streams.size();
    hipStream_t st;
    (void)hipStreamCreateWithFlags(&st, 0);
    qap_batch_handle b = nullptr;
    if (qap_batch_create(hs.data(), (int)hs.size(), k.data(), iters, lo.data(), hi.data(), seed.data(), nullptr, &b))
        return -1;
    int64_t starts = 0, ints = 0;
    qap_batch_size(b, &starts, &ints);
    std::vector<int32_t> p(ints), done(starts);
    std::vector<int64_t> best(starts);
    g_calls = 0;
    g_failed = false;
    g_fail_at = fail_at;
    int rc = qap_batch_run_async(b, p.data(), best.data(), done.data(), st);
    g_fail_at = -1;
    if (g_failed) rc = rc == 0 ? -1 : 0;   // a failed call fails the run
    (void)hipStreamSynchronize(st);
    if (!idle()) rc = -1;
    qap_batch_destroy(b);
    for (qap_handle h : hs) qap_destroy(h);
    return rc ? -1 : (int)g_streams.size() - before - 1;
}

}  // namespace

// one line a plan: the side streams it created
int main() {
    std::printf("%d\n", plan({8}, 1000));                        // one kernel
    std::printf("%d\n", plan({8, 9}, 1));                        // two block forms, short
    std::printf("%d\n", plan({8, 9}, 40));
    std::printf("%d\n", plan({8, 9}, 200));                      // long: the caller's stream and one more
    std::printf("%d\n", plan({20, 31, 40, 51, 60}, 10));
    std::printf("%d\n", plan({20, 31, 40, 51, 60, 91, 200}, 10));   // 54 us beside the longest
    std::printf("%d\n", plan({20, 31, 40, 51, 60, 91, 200}, 2000));   // no more lanes than queues but one
    std::printf("%d\n", plan({8, 9}, 30, 1000));                 // many rounds over the compute units
    setenv("QAP_BATCH_LANES", "2", 1);
    std::printf("%d\n", plan({8, 9, 100}, 1));                   // as told
    unsetenv("QAP_BATCH_LANES");
    // every call of a run on three lanes failing in turn
    int bad = 0, fail = 0;
    for (;; ++fail) {
        const int r = plan({20, 31, 40, 51, 60, 91, 200, 300}, 2000, 1, fail);
        if (r < 0) ++bad, std::fprintf(stderr, "call %d failed\n", fail);
        if (!g_failed) break;
    }
    std::printf("%d\n%d\n", bad, fail);
    return 0;
}
