/*
 * Driver of the CPU SIMT emulation build of the policy-gradient step.
 *
 * TEST INFRASTRUCTURE.  Compiled together with the library's own
 * csrc/parason.hip (the segment plan) and csrc/pg.hip for the host
 * (tests/simt/hip/hip_runtime.h stands in for the HIP runtime), under
 * AddressSanitizer and UndefinedBehaviorSanitizer.  Reads one batch from a
 * binary file, runs it through the C-ABI as a caller would (host memory plays
 * the device memory) and writes the outputs to another file.
 *
 * Input (little endian): int64 n, int64 n_tok, int32 group_size, int32 cus,
 * int32 shift, int32 in_place (the advantages are written over the rewards),
 * double clip_low, double clip_high, then float reward[n], float logp[n_tok],
 * float logp_old[n_tok], int64 starts[n], int32 lengths[n].
 * Output: int32 status, float advantage[n], float grad[n_tok] (1e30 where
 * nothing was written), double stats[4].
 */
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <vector>

#include <hip/hip_runtime.h>

#include "parason.h"

static void rd(FILE *f, void *p, size_t n)
{
    if (n && fread(p, 1, n, f) != n) {
        fprintf(stderr, "short read\n");
        exit(2);
    }
}

/* n floats at `shift` elements past a 256-byte boundary, in an allocation that
 * ends at the 16-byte vector holding the last of them (the kernels read whole
 * vectors, which never cross a page) */
static float *floats(int64_t n, int shift, char **mem)
{
    if (posix_memalign((void **)mem, 256, ((size_t)(n + shift) * 4 + 15) / 16 * 16 + 16) != 0) exit(2);
    return (float *)*mem + shift;
}

int main(int argc, char **argv)
{
    if (argc != 3) {
        fprintf(stderr, "usage: %s in out\n", argv[0]);
        return 2;
    }
    FILE *f = fopen(argv[1], "rb");
    if (!f) return 2;
    int64_t n, n_tok;
    int32_t G, cus, shift, in_place;
    double clip[2];
    rd(f, &n, 8);
    rd(f, &n_tok, 8);
    rd(f, &G, 4);
    rd(f, &cus, 4);
    rd(f, &shift, 4);
    rd(f, &in_place, 4);
    rd(f, clip, sizeof clip);
    char *mem[3];
    float *logp = floats(n_tok, shift, &mem[0]), *old = floats(n_tok, shift, &mem[1]), *grad = floats(n_tok, shift, &mem[2]);
    std::vector<float> reward(n), adv(n, -77.0f);
    std::vector<int64_t> starts(n);
    std::vector<int32_t> lengths(n);
    rd(f, reward.data(), (size_t)n * 4);
    rd(f, logp, (size_t)n_tok * 4);
    rd(f, old, (size_t)n_tok * 4);
    rd(f, starts.data(), (size_t)n * 8);
    rd(f, lengths.data(), (size_t)n * 4);
    fclose(f);
    for (int64_t i = 0; i < n_tok; ++i) grad[i] = 1e30f;
    simt::emulated_cus() = cus;

    const parason_pg_config cfg = {G, clip[0], clip[1]};
    double stats[PARASON_PG_STAT_COUNT] = {-77.0, -77.0, -77.0, -77.0};
    float *advantage = in_place ? reward.data() : adv.data();
    size_t bytes = 0;
    int rc = parason_pg_workspace_size(n, &bytes);
    if (rc == PARASON_OK) {
        /* exact size, filled with a pattern: the path must not rely on the
         * workspace's contents or read past its end */
        void *ws = nullptr;
        if (posix_memalign(&ws, 256, bytes) != 0) return 2;
        memset(ws, 0xA5, bytes);
        rc = parason_pg_run(&cfg, reward.data(), logp, old, starts.data(), lengths.data(), n, advantage, grad, stats, ws,
                            bytes, nullptr);
        free(ws);
    }
    FILE *o = fopen(argv[2], "wb");
    if (!o) return 2;
    fwrite(&rc, 4, 1, o);
    fwrite(advantage, 4, (size_t)n, o);
    fwrite(grad, 4, (size_t)n_tok, o);
    fwrite(stats, 1, sizeof stats, o);
    fclose(o);
    for (char *m : mem) free(m);
    fprintf(stderr, "simt: %llu wave operations\n", (unsigned long long)simt::st().collectives);
    return 0;
}
