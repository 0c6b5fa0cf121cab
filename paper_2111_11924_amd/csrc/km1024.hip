// Montgomery form of the CRT halves of the 1024-bit size class.
#define PMK_CLASS_BITS 1024
#include "kmont.inc"
