// Checks of the library's host code on a machine without a GPU, where every device
// allocation fails: one per argument, exit status 0 = passed.  Linked against
// libmapmaker.so by test_host_checks.py.
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <new>
#include <unistd.h>

#include "mm_internal.h"

namespace mm {
void pointing_p_slots_device(mm_ctx *ctx, mm_pointing *p, int32_t width, Scratch &sc,
                             const int32_t **dir_cnt);
}

namespace {
bool no_host_memory = false;
}
void *operator new(std::size_t n) {
    void *p = no_host_memory ? nullptr : std::malloc(n ? n : 1);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void *p) noexcept { std::free(p); }
void operator delete(void *p, std::size_t) noexcept { std::free(p); }

namespace {

int failures = 0;
#define EXPECT(c)                                                 \
    do {                                                          \
        if (!(c)) {                                               \
            std::printf("line %d: %s\n", __LINE__, #c);           \
            ++failures;                                           \
        }                                                         \
    } while (0)

// A buffer that a working device would have given (never dereferenced here).
void pretend(mm::DBuf &b, size_t bytes) {
    b.ptr = reinterpret_cast<void *>((uintptr_t)1 << 20);
    b.bytes = bytes;
}

// A pointing with a grid of three map copies, a tile order and a sliced P^T.
void gridded(mm_pointing &p) {
    p.n_samp = (int64_t)1 << 23;
    p.n_pix_total = p.n_obs = 16384;
    p.n_valid = p.n_samp;
    p.nc = 3;
    p.grid_width = 128;
    p.p_copies = 3;
    pretend(p.j, 4 * p.n_samp);
    pretend(p.p_j, 4 * p.n_samp);
    pretend(p.p_slot, 4 * 3 * p.n_obs);
    pretend(p.p_chunk_grp, 4 * (p.n_samp >> 12));
    pretend(p.seg_order, 4 * p.n_obs);
    p.sl_G = 256 * 3;
    p.sl_S = 5;
    p.sl_D = 3;
    for (mm::DBuf *b : {&p.sl_pix, &p.sl_base, &p.sl_perm, &p.sl_w}) pretend(*b, 1 << 20);
}

// Set-up of a new grid fails at its first allocation, or at the first one inside the
// map copies: what the applies look at afterwards is whole or absent, never a new
// count with old slots or an order that was not written.
void regrid() {
    {
        mm_ctx ctx;
        mm_pointing p;
        gridded(p);
        bool threw = false;
        try {
            mm::pointing_layout_device(&ctx, &p, 64);
        } catch (const mm::Error &e) {
            threw = e.code == MM_E_OOM;
        }
        EXPECT(threw);
        EXPECT(p.p_j.ptr == nullptr && p.p_copies == 0);
        EXPECT(p.seg_order.ptr == nullptr && p.grid_width == 0);
        EXPECT(p.sl_G == 0 && p.sl_S == 0 && p.sl_D == 1);
        EXPECT(mm::apply_PT_scratch_bytes(&p, 1) == 0);
    }
    {
        mm_ctx ctx;
        mm_pointing p;
        gridded(p);
        bool threw = false;
        try {
            mm::Scratch sc(&ctx);
            const int32_t *cnt = nullptr;
            mm::pointing_p_slots_device(&ctx, &p, 64, sc, &cnt);
        } catch (const mm::Error &e) {
            threw = e.code == MM_E_OOM;
        }
        EXPECT(threw);
        EXPECT(p.p_copies == 0 && p.p_j.ptr == nullptr);
        // one copy at the compact ids
        EXPECT(mm::apply_P_scratch_bytes(&p, 1) == 32 * (size_t)p.n_obs);
    }
}

// The P of 2 to 64 columns: every sample has a wave and the launch stays below 2^32
// threads, up to the most samples a pointing takes.
void p_launch() {
    for (int R = 2; R <= 64; R *= 2)
        for (int64_t n : {(int64_t)1, (int64_t)1000, (int64_t)1 << 28, ((int64_t)1 << 28) + 1,
                          ((int64_t)1 << 31) - 1})
            for (int64_t blocks : {0, 512, 8192}) {
                const int step = 256 / R;
                const int64_t per = mm::p_wave_samples(n, step, blocks);
                const int64_t grid = (n + 4 * per - 1) / (4 * per);
                EXPECT(per >= step && per % step == 0);
                EXPECT(grid * 4 * per >= n && grid * 256 < (int64_t)1 << 32);
                if (blocks > 0) EXPECT(grid <= blocks);
                else if (n * R < (int64_t)1 << 32) EXPECT(per == step);
                // a map beyond the L2s: longer runs, from 32 columns and 2^25 values on
                const int64_t far = mm::p_wave_samples(n, step, blocks, 25 << 20);
                EXPECT((n + 4 * far - 1) / (4 * far) * 256 < (int64_t)1 << 32);
                if (R == 64 && blocks == 0 && n == (int64_t)1 << 28) EXPECT(far >= 16 * step);
                if (R < 32 || blocks > 0 || n < 1 << 19) EXPECT(far == per);
            }
}

// The tile keys of every pixel fit in the bits that are sorted, at most 64.
void tile_keys() {
    for (int32_t tile : {8, 32})
        for (int32_t n_pix : {1, 1000, 1 << 20, 2147483647})
            for (int32_t width : {1, 7, 32, 33, 46341, 2147483616, 2147483617, 2147483647}) {
                const unsigned b = mm::tile_key_bits(n_pix, width, tile);
                EXPECT(b <= 64);
                const int64_t tiles_x = ((int64_t)width + tile - 1) / tile;
                for (int64_t g : {(int64_t)n_pix - 1, (int64_t)n_pix / 2, (int64_t)width - 1}) {
                    if (g >= n_pix) continue;
                    const uint64_t t = (uint64_t)(g / width / tile * tiles_x + g % width / tile);
                    EXPECT(((t << 24 | 0xffffff) >> (b - 1)) <= 1);
                }
            }
}

// Blocks of the map-domain reductions: never fewer for a larger map, at most 512, and
// no block without a row.
void reduction_blocks() {
    for (int R = 1; R <= 64; R *= 2) {
        int last = 1;
        for (int64_t n = 1; n * R <= 1000000; n += 1 + n / 97) {
            const int p = mm::reduction_parts(n, R);
            EXPECT(p >= last && p <= 512);
            if (R == 1) EXPECT(p <= n);
            last = p;
        }
    }
    EXPECT(mm::reduction_parts(49153, 1) >= 192 && mm::reduction_parts(65536, 1) >= 192);
}

// Another FFT block length fails half way: no apply may run its kernels with what is
// left of the tables of the old length.
void fft_block() {
    mm_ctx ctx;
    mm_noise nz;
    nz.method = MM_NOISE_FFT;
    nz.half_bw = 100;
    nz.n_samp = 100000;
    nz.n_int = 1;
    nz.n_filters = 1;
    nz.h_istart = {0, nz.n_samp};
    nz.fft_n = nz.fft.n = 16384;
    nz.fft.valid = 16384 - 200;
    nz.fft.n_blocks = 7;
    for (mm::DBuf *b : {&nz.fft.spec, &nz.fft.tw, &nz.fft.blocks}) pretend(*b, 1 << 20);
    auto code = [](auto f) {
        try {
            f();
        } catch (const mm::Error &e) {
            return (int)e.code;
        }
        return 0;
    };
    EXPECT(code([&] { mm::noise_fft_prepare(&ctx, &nz, 32768); }) == MM_E_OOM);
    EXPECT(nz.fft.n_blocks == 0 || nz.fft.n == 16384);
    EXPECT(code([&] { mm::noise_apply_dev(&ctx, &nz, 1, nullptr, nullptr); }) == MM_E_OOM);
}

// Buffers and contexts are released in destructors and behind a C interface, where no
// exception may leave: nothing there takes host memory.
void release_without_host_memory() {
    mm::dev_pool_ctx(0, 1);
    mm::DBuf *b = new mm::DBuf();
    pretend(*b, 4096);
    bool threw = false;
    no_host_memory = true;
    try {
        b->release();
        mm::dev_pool_ctx(0, -1);
    } catch (...) {
        threw = true;
    }
    no_host_memory = false;
    EXPECT(!threw);
    EXPECT(noexcept(mm::dev_free(nullptr, 0)) && noexcept(mm::dev_pool_trim(0)));
}

// A count of elements that overflowed is refused, not taken as one element.
void scratch_sizes() {
    for (int64_t n : {(int64_t)-1, (int64_t)-64, -((int64_t)1 << 37), (int64_t)1 << 61}) {
        mm_ctx ctx;
        pretend(ctx.build_ws, 1 << 20);
        bool threw = false;
        try {
            mm::Scratch sc(&ctx);
            (void)sc.get<double>(n);
        } catch (const mm::Error &e) {
            threw = e.code == MM_E_OOM;
        }
        EXPECT(threw);
        EXPECT(ctx.build_off == 0);
    }
}

// The P^T kernel of several columns: few hits per pixel do not fill the steps of the
// two-column kernel (65,536 samples on 4,096 pixels x 8 columns took 3.2 times as long
// there), nor a quarter of them those of a block per pixel.
void pt_forms() {
    using mm::PtForm;
    const auto f = [](int32_t n_obs, int64_t hits, int R) {
        return mm::pt_form(n_obs, hits * n_obs, R, 256);
    };
    EXPECT(f(4096, 16, 8) == PtForm::LANES && f(1024, 16, 8) == PtForm::LANES);
    EXPECT(f(65536, 16, 8) == PtForm::LANES && f(4096, 4, 32) == PtForm::LANES);
    EXPECT(f(1024, 10000, 4) == PtForm::LANES);
    EXPECT(f(4096, 16, 16) == PtForm::COLUMNS && f(1024, 64, 16) == PtForm::COLUMNS);
    EXPECT(f(4096, 256, 64) == PtForm::COLUMNS && f(65536, 2048, 64) == PtForm::COLUMNS);
    EXPECT(f(1024, 64, 64) == PtForm::BLOCK && f(1, 512, 8) == PtForm::BLOCK);
    for (int R = 1; R <= 64; R *= 2)  // more hits never go back to fewer waves
        for (int32_t n_obs : {1, 300, 2047, 2048, 100000}) {
            int last = 0;
            for (int64_t h = 1; h < 100000; h += 1 + h / 9) {
                const int v = (int)f(n_obs, h, R);
                EXPECT(v >= last);
                last = v;
            }
        }
}

// The sliced P^T of I and QU only with little padding (seven times slower at 4.4 times
// the entries, and of no bound in memory); IQU always.
void slices() {
    const int64_t n = (int64_t)1 << 23, m = (int64_t)1 << 25;
    for (int nc : {1, 2}) {
        EXPECT(mm::slices_pay(nc, n, n / 2, n / 2) && mm::slices_pay(nc, n, 1000, 1200));
        EXPECT(!mm::slices_pay(nc, n, 1000, 1201) && !mm::slices_pay(nc, n, n / 2, 3 * n));
        EXPECT(mm::slices_pay(nc, m, 1000, 2000) && !mm::slices_pay(nc, m, 1000, 2001));
    }
    EXPECT(mm::slices_pay(3, n, n, 64 * n));
}

}  // namespace

int main(int argc, char **argv) {
    int n = 0;
    if (hipGetDeviceCount(&n) == hipSuccess && n > 0) {
        std::printf("a GPU is here\n");
        return 77;
    }
    const char *what = argc > 1 ? argv[1] : "";
    if (!std::strcmp(what, "regrid")) regrid();
    else if (!std::strcmp(what, "p_launch")) p_launch();
    else if (!std::strcmp(what, "tile_keys")) tile_keys();
    else if (!std::strcmp(what, "slices")) slices();
    else if (!std::strcmp(what, "pt_forms")) pt_forms();
    else if (!std::strcmp(what, "scratch_sizes")) scratch_sizes();
    else if (!std::strcmp(what, "release")) release_without_host_memory();
    else if (!std::strcmp(what, "fft_block")) fft_block();
    else if (!std::strcmp(what, "reduction_blocks")) reduction_blocks();
    else {
        std::printf("no check named '%s'\n", what);
        return 2;
    }
    std::fflush(stdout);
    _exit(failures ? 1 : 0);
}
