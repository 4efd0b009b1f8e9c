// The server's host code (qap_server.hip) on the stand-in runtime, one call of a step failing.
// Prints every failing call after which a stream was left with work nobody waited for.
#include "standin_hip.h"

#include "../paper_2307_11248_amd/csrc/qap_server.hip"

namespace qapk {
hipError_t launch_table(const TableArgs &, hipStream_t s) { return put(s); }
hipError_t launch_table_items(const Item *, int n, size_t, hipStream_t s) { return n ? put(s) : hipSuccess; }
hipError_t launch_resume(const Item *, int n, size_t, hipStream_t s) { return n ? put(s) : hipSuccess; }
hipError_t launch_resume_freq(const Item *, int n, size_t, hipStream_t s) { return n ? put(s) : hipSuccess; }
hipError_t launch_resume_wide(const Item *, int n, size_t, hipStream_t s) { return n ? put(s) : hipSuccess; }
hipError_t launch_resume_block(const Item *, int n, size_t, hipStream_t s) { return n ? put(s) : hipSuccess; }
size_t freq_static_lds() { return 1024; }
size_t table_smem_bytes(int) { return 1024; }
size_t search_smem_bytes(int, int, int, int) { return 1024; }
size_t stream_smem_bytes(int, int) { return 1024; }
size_t block_smem_bytes(int, int, int, bool) { return 1024; }
size_t block_ring_bytes(int) { return 128; }
int batch_shape_ok(int n, int, int, int) { return n <= WIDE_N; }
int stream_shape_ok(int, int, size_t) { return 1; }
int block_ok(int n, int, int blk, bool, int, int, size_t) { return blk && n <= WIDE_N; }
}  // namespace qapk

namespace qaph {
std::vector<int32_t> enumerate_tiles(int, int, int *inner) { return *inner = 1, std::vector<int32_t>(1); }
int pack_instance(const int32_t *F, const int32_t *, int n, std::vector<uint8_t> &pack, int *sym, int *blk) {
    pack.assign((size_t)4 * n * row_stride(n), 0);
    *sym = 0;
    *blk = F[0] ? 0 : 1;   // (the test's way to ask for tiles)
    return QAP_OK;
}
int dev_err_at(hipError_t, const char *) { return QAP_E_DEVICE; }
bool check_perms(const int32_t *, int, int) { return true; }
bool handle_view(const qap_ctx *h, const uint8_t **mats, int *n, int *sym, int *blk, int *device) {
    *mats = reinterpret_cast<const uint8_t *>(h);
    *n = 20;
    *sym = *blk = *device = 0;
    return true;
}
}  // namespace qaph

int main() {
    static int32_t F[300 * 300], G[300 * 300], start[300];
    G[0] = 1;
    int fail = 0;
    for (;; ++fail) {
        for (Stream *s : g_streams) delete s;
        g_streams.clear();
        g_finished.clear();
        g_fail_at = -1;
        qap_server_handle s = nullptr;
        int64_t t;
        if (qap_server_create(64 << 20, 16, 1.0, &s)) return 2;
        // one request of each kernel: block form, tiles, frequency memory, above n = 256
        if (qap_server_submit_matrices(s, F, F, 40, start, 10, 1, 2, 0, &t) ||
            qap_server_submit_matrices(s, G, F, 40, start, 10, 1, 2, 0, &t) ||
            qap_server_submit_freq(s, reinterpret_cast<qap_handle>(F), start, 10, 1, 2, 0, 0, 0, &t) ||
            qap_server_submit_matrices(s, F, F, 300, start, 10, 1, 2, 0, &t))
            return 2;
        g_calls = 0;
        g_failed = false;
        g_fail_at = fail;
        const int rc = qap_server_step(s, nullptr, nullptr);
        if (g_failed != (rc < 0)) ++g_bad, std::printf("call %d failed, step returned %d\n", fail, rc);
        if (!idle()) ++g_bad, std::printf("call %d failed, work left in flight\n", fail);
        const bool last = !g_failed;
        g_fail_at = -1;
        qap_server_destroy(s);
        if (last) break;
    }
    std::printf("calls %d bad %d\n", fail, g_bad);
    return g_bad ? 1 : 0;
}
