/* Argument checks and scratch sizes of rmdf_mlp_grads, driven on a machine
 * without a GPU (see test_grads_sanitized.py): every call below has to come
 * back before it reaches the device. */
#include <stdint.h>
#include <stdio.h>

#include "rmdf.h"

static int bad = 0;

static void expect(const char *what, int got, int want) {
  if (got != want) {
    printf("%s: %d, not %d\n", what, got, want);
    bad = 1;
  }
}

int main(void) {
  size_t bytes = 0, last = 0;
  int i, n;
  char *room = (char *)(uintptr_t)0x100000;   /* an address that is looked at, never followed */
  const int refused[] = {-2147483647 - 1, -8, 0, 1, 7, 12, 4095, 2147483647};
  expect("work NULL", rmdf_mlp_grads_work(64, NULL), RMDF_E_INVAL);
  for (i = 0; i < (int)(sizeof(refused) / sizeof(refused[0])); ++i)
    expect("work n", rmdf_mlp_grads_work(refused[i], &bytes), RMDF_E_INVAL);
  /* up to the largest n there is: the intermediates alone take 640 bytes a sample */
  for (n = 8; ; n = n < 1073741824 ? 2 * n : 2147483640) {
    expect("work", rmdf_mlp_grads_work(n, &bytes), RMDF_OK);
    if (bytes < (size_t)n * 640 || bytes < last) {
      printf("n %d: %zu bytes\n", n, bytes);
      bad = 1;
    }
    last = bytes;
    if (n == 2147483640) break;
  }
  expect("work 4096", rmdf_mlp_grads_work(4096, &bytes), RMDF_OK);
  for (i = 0; i < 16; ++i) {                  /* each operand NULL, and each aligned one misaligned */
    char *p[16];
    int k;
    for (k = 0; k < 16; ++k) p[k] = room + 4096 * k;
    for (k = 0; k < 2; ++k) {
      if (k == 0) p[i] = NULL;
      else if (i == 0 || i == 2 || i == 4 || i == 15) p[i] = room + 4096 * i + 8;
      else continue;
      expect("grads", rmdf_mlp_grads(p[0], (float *)p[1], 4096, p[2], (float *)p[3], p[4], (float *)p[5], (float *)p[6],
                                     (float *)p[7], 1.f, 0.25f, (float *)p[8], (float *)p[9], (float *)p[10],
                                     (float *)p[11], (float *)p[12], (float *)p[13], (float *)p[14], p[15], bytes, NULL),
             RMDF_E_INVAL);
    }
  }
  {
    float *f = (float *)room;
    expect("scratch too small", rmdf_mlp_grads(room, f, 4096, room, f, room, f, f, f, 1.f, 0.25f, f, f, f, f, f, f, f,
                                               room, bytes - 1, NULL), RMDF_E_INVAL);
    expect("n", rmdf_mlp_grads(room, f, 4100, room, f, room, f, f, f, 1.f, 0.25f, f, f, f, f, f, f, f, room, bytes, NULL),
           RMDF_E_INVAL);
    expect("n max", rmdf_mlp_grads(room, f, 2147483640, room, f, room, f, f, f, 1.f, 0.25f, f, f, f, f, f, f, f, room, bytes,
                                   NULL), RMDF_E_INVAL);
  }
  if (!bad) printf("sanitized grads ok\n");
  return bad;
}
