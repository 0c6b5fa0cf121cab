// Montgomery form of the CRT halves of the 3072-bit size class.
#define PMK_CLASS_BITS 3072
#include "kmont.inc"
